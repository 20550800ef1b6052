// layout.hip - conversions between the canonical site-major FP64 arrays and the
// block-tiled even-odd SoA layout (FP64, FP32 or FP16 with a per-site FP32 scale), and
// a STREAM-type copy kernel used to measure attainable HBM bandwidth.
#include "canon.hpp"
#include "kernels.hpp"

#include <algorithm>

namespace sapdd {

constexpr int LAYOUT_WG = 256;

template <int N, class S>
__global__ __launch_bounds__(LAYOUT_WG) void pack_kernel(Geom geo, const double *__restrict__ canon, S *out,
                                                         float *scale) {
    const int64_t t = (int64_t)blockIdx.x * LAYOUT_WG + threadIdx.x;
    if (t >= geo.V) return;
    const int f = blockIdx.y;
    const int64_t bp = t / geo.Vbh;
    const int s = (int)(t - bp * geo.Vbh);
    const double *src = canon + ((int64_t)f * geo.V + canon_index(geo, bp, s)) * N;
    double v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = src[k];
    store_site<double, N>(out + (int64_t)f * geo.V * N, scale ? scale + (int64_t)f * geo.V : nullptr, bp, s, geo.Vbh,
                          v);
}

template <int N, class S>
__global__ __launch_bounds__(LAYOUT_WG) void unpack_kernel(Geom geo, const S *in, const float *scale,
                                                           double *__restrict__ canon) {
    const int64_t t = (int64_t)blockIdx.x * LAYOUT_WG + threadIdx.x;
    if (t >= geo.V) return;
    const int f = blockIdx.y;
    const int64_t bp = t / geo.Vbh;
    const int s = (int)(t - bp * geo.Vbh);
    double v[N];
    load_site<double, N>(in + (int64_t)f * geo.V * N, scale ? scale + (int64_t)f * geo.V : nullptr, bp, s, geo.Vbh, v);
    double *dst = canon + ((int64_t)f * geo.V + canon_index(geo, bp, s)) * N;
#pragma unroll
    for (int k = 0; k < N; ++k) dst[k] = v[k];
}

// Spinors on 4^4 and 8x4^3 blocks: a workgroup turns a tile of 256 sites (a 4^4 block, or
// half of an 8x4^3 block: two time slices) in LDS, so that the canonical side is written in
// runs of four or eight sites (canon.hpp). Bound by HBM; against one thread per site storing
// its 192 bytes: 32^3 x 64, FP64, 6 fields 1365 -> 900 us (5.4 TB/s), FP32 140 -> 108 us, 16^3 x
// 32, FP64 13.6 -> 7.7 us. The opposite direction keeps one thread per site: its strided
// loads find the rest of their lines in the cache, and the same turn in LDS gained 6% on
// large fields and lost 50% on 16^3 x 32.
struct TileSite {
    int64_t bp;
    int s, n;  // n: lexicographic number inside the tile
    __device__ __forceinline__ TileSite(const Geom &geo) {
        const int h = LAYOUT_WG / 2, per = geo.Vbh / h;  // tiles per block
        const int p = threadIdx.x / h, part = blockIdx.x % per;
        bp = 2 * (int64_t)(blockIdx.x / per) + p;
        s = part * h + threadIdx.x % h;
        int l[4];
        local_coords(geo.B, p, s, l);
        n = l[0] + geo.B[0] * (l[1] + geo.B[1] * (l[2] + geo.B[2] * l[3])) - part * LAYOUT_WG;
    }
};
template <class S>
__global__ __launch_bounds__(LAYOUT_WG) void unpack_spinor_kernel(Geom geo, const S *in, const float *scale,
                                                                  double *canon) {
    __shared__ CanonSlot<S> lds[LAYOUT_WG];
    const int64_t f = blockIdx.y;
    const TileSite t(geo);
    CanonSlot<S> &slot = lds[t.n];
    const auto *p = reinterpret_cast<const typename Vec<S>::type *>(in + f * geo.V * 24);
    constexpr int W = Vec<S>::W;
#pragma unroll
    for (int v = 0; v < 24 / W; ++v) {
        const auto x = ld_vec<true>(p + vec_index<S, 24>(t.bp, v, t.s, geo.Vbh));
#pragma unroll
        for (int w = 0; w < W; w += 2) slot.c[(v * W + w) / 2] = typename CanonSlot<S>::v2{x[w], x[w + 1]};
    }
    if constexpr (Storage<S>::scaled) slot.scale = *gmem(scale + f * geo.V + t.bp * geo.Vbh + t.s);
    slot.idx = canon_index(geo, t.bp, t.s);
    __syncthreads();
    canon_put<LAYOUT_WG>(canon + f * geo.V * 24, lds);
}
static bool tiled_spinor(const Geom &geo, int ncomp) { return ncomp == 24 && geo.Vbh % (LAYOUT_WG / 2) == 0; }
template <int N, class S>
__global__ __launch_bounds__(LAYOUT_WG) void convert_kernel(Geom geo, const double *__restrict__ in, S *out,
                                                            float *scale) {
    const int64_t t = (int64_t)blockIdx.x * LAYOUT_WG + threadIdx.x;
    if (t >= geo.V) return;
    const int f = blockIdx.y;
    const int64_t bp = t / geo.Vbh;
    const int s = (int)(t - bp * geo.Vbh);
    double v[N];
    load_site<double, N>(in + (int64_t)f * geo.V * N, nullptr, bp, s, geo.Vbh, v);
    store_site<double, N>(out + (int64_t)f * geo.V * N, scale ? scale + (int64_t)f * geo.V : nullptr, bp, s, geo.Vbh,
                          v);
}

static dim3 site_grid(const Geom &geo, int nfield) {
    return dim3((unsigned)((geo.V + LAYOUT_WG - 1) / LAYOUT_WG), (unsigned)nfield);
}

template <int N>
static hipError_t pack_n(const Geom &geo, int nfield, const double *canon, Fld out, hipStream_t st) {
    const dim3 g = site_grid(geo, nfield);
    if (out.prec == P64) hipLaunchKernelGGL((pack_kernel<N, double>), g, dim3(LAYOUT_WG), 0, st, geo, canon, (double *)out.data, nullptr);
    else if (out.prec == P32) hipLaunchKernelGGL((pack_kernel<N, float>), g, dim3(LAYOUT_WG), 0, st, geo, canon, (float *)out.data, nullptr);
    else hipLaunchKernelGGL((pack_kernel<N, half_t>), g, dim3(LAYOUT_WG), 0, st, geo, canon, (half_t *)out.data, out.scale);
    return hipGetLastError();
}

template <int N>
static hipError_t unpack_n(const Geom &geo, int nfield, Fld in, double *canon, hipStream_t st) {
    const dim3 g = site_grid(geo, nfield);
    if (in.prec == P64) hipLaunchKernelGGL((unpack_kernel<N, double>), g, dim3(LAYOUT_WG), 0, st, geo, (const double *)in.data, nullptr, canon);
    else if (in.prec == P32) hipLaunchKernelGGL((unpack_kernel<N, float>), g, dim3(LAYOUT_WG), 0, st, geo, (const float *)in.data, nullptr, canon);
    else hipLaunchKernelGGL((unpack_kernel<N, half_t>), g, dim3(LAYOUT_WG), 0, st, geo, (const half_t *)in.data, in.scale, canon);
    return hipGetLastError();
}

template <int N>
static hipError_t convert_n(const Geom &geo, int nfield, const double *in, Fld out, hipStream_t st) {
    const dim3 g = site_grid(geo, nfield);
    if (out.prec == P64) return hipErrorInvalidValue;
    if (out.prec == P32) hipLaunchKernelGGL((convert_kernel<N, float>), g, dim3(LAYOUT_WG), 0, st, geo, in, (float *)out.data, nullptr);
    else hipLaunchKernelGGL((convert_kernel<N, half_t>), g, dim3(LAYOUT_WG), 0, st, geo, in, (half_t *)out.data, out.scale);
    return hipGetLastError();
}

hipError_t launch_pack(const Geom &geo, int ncomp, int nfield, const double *canon, Fld out, hipStream_t st) {
    if (nfield <= 0 || geo.V == 0) return hipSuccess;
    if (ncomp == 24) return pack_n<24>(geo, nfield, canon, out, st);
    if (ncomp == 72) return pack_n<72>(geo, nfield, canon, out, st);
    return hipErrorInvalidValue;
}

hipError_t launch_unpack(const Geom &geo, int ncomp, int nfield, Fld in, double *canon, hipStream_t st) {
    if (nfield <= 0 || geo.V == 0) return hipSuccess;
    if (tiled_spinor(geo, ncomp)) {
        const dim3 g((unsigned)(geo.V / LAYOUT_WG), (unsigned)nfield);
        if (in.prec == P64) hipLaunchKernelGGL(unpack_spinor_kernel<double>, g, dim3(LAYOUT_WG), 0, st, geo, (const double *)in.data, nullptr, canon);
        else if (in.prec == P32) hipLaunchKernelGGL(unpack_spinor_kernel<float>, g, dim3(LAYOUT_WG), 0, st, geo, (const float *)in.data, nullptr, canon);
        else hipLaunchKernelGGL(unpack_spinor_kernel<half_t>, g, dim3(LAYOUT_WG), 0, st, geo, (const half_t *)in.data, in.scale, canon);
        return hipGetLastError();
    }
    if (ncomp == 24) return unpack_n<24>(geo, nfield, in, canon, st);
    if (ncomp == 72) return unpack_n<72>(geo, nfield, in, canon, st);
    return hipErrorInvalidValue;
}

hipError_t launch_convert(const Geom &geo, int ncomp, int nfield, const double *in, Fld out, hipStream_t st) {
    if (nfield <= 0 || geo.V == 0) return hipSuccess;
    if (ncomp == 24) return convert_n<24>(geo, nfield, in, out, st);
    if (ncomp == 72) return convert_n<72>(geo, nfield, in, out, st);
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- copy (bandwidth probe)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// One 16-byte vector per thread over a grid that covers the whole buffer, with
// non-temporal hints: measured 6.2-6.5 TB/s on 2 GiB, where a grid capped at 16k
// workgroups that strides over the buffer stayed at 4.4-5.3 TB/s.
__global__ __launch_bounds__(256) void copy_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, int64_t n16,
                                                   int64_t base, const unsigned char *__restrict__ tsrc,
                                                   unsigned char *__restrict__ tdst, int tail) {
    const int64_t i = base + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n16) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
    if (base == 0 && blockIdx.x == 0 && (int)threadIdx.x < tail) tdst[threadIdx.x] = tsrc[threadIdx.x];
}

hipError_t launch_copy(const void *src, void *dst, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int64_t n16 = n / 16;
    const int tail = (int)(n - n16 * 16);
    const int64_t per = (int64_t)0x40000000;  // vectors per launch (2^22 workgroups of 256)
    for (int64_t base = 0; base == 0 || base < n16; base += per) {
        int64_t nb = (std::min(per, n16 - base) + 255) / 256;
        if (nb < 1) nb = 1;
        hipLaunchKernelGGL(copy_kernel, dim3((unsigned)nb), dim3(256), 0, st, (const u32x4 *)src, (u32x4 *)dst, n16,
                           base, (const unsigned char *)src + n16 * 16, (unsigned char *)dst + n16 * 16, tail);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace sapdd
