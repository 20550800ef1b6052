// blockgeo.hpp - compile-time Schwarz block shapes, per-thread site information inside a
// block, and the in-block hopping term evaluated through LDS.
//
// One workgroup owns one block (the GPU counterpart of the paper's one-domain-per-core
// assignment, Sec. 3.3/3.5). In the block operator thread tid < Vbh is the even site with
// half index tid and thread Vbh + s the odd site s, so the two parities occupy separate
// waves whenever Vbh >= 64; the Schwarz kernel has its own thread layout.
#pragma once
#include <utility>

#include "canon.hpp"
#include "core.hpp"

namespace sapdd {

template <int I, int N, class F> __device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

template <int BX, int BY, int BZ, int BT> struct Blk {
    static constexpr int bx = BX, by = BY, bz = BZ, bt = BT;
    static constexpr int Vb = BX * BY * BZ * BT;
    static constexpr int Vbh = Vb / 2;
    static constexpr int NT = Vb;                         // threads per workgroup
    __device__ static constexpr int ext(int mu) { return mu == 0 ? BX : mu == 1 ? BY : mu == 2 ? BZ : BT; }
};

struct SiteInfo {
    int p, s;
    int l[4];
    int nbf[4], nbb[4];  // half index of the in-block forward / backward neighbour
    unsigned fin, bin;   // bit mu set if that neighbour is inside the block
};

template <class BK> __device__ __forceinline__ SiteInfo site_info(int tid) {
    SiteInfo si;
    si.p = tid >= BK::Vbh;
    si.s = tid - si.p * BK::Vbh;
    const int B[4] = {BK::bx, BK::by, BK::bz, BK::bt};
    local_coords(B, si.p, si.s, si.l);
    si.fin = si.bin = 0;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        int lf[4] = {si.l[0], si.l[1], si.l[2], si.l[3]};
        int lb[4] = {si.l[0], si.l[1], si.l[2], si.l[3]};
        lf[mu] += 1;
        lb[mu] -= 1;
        si.nbf[mu] = si.nbb[mu] = 0;
        if (si.l[mu] < B[mu] - 1) {
            si.fin |= 1u << mu;
            si.nbf[mu] = local_half_index(B, lf);
        }
        if (si.l[mu] > 0) {
            si.bin |= 1u << mu;
            si.nbb[mu] = local_half_index(B, lb);
        }
    }
    return si;
}

// The four forward links of a thread's own site, held in registers as the
// storage-precision 16-byte vectors they were loaded in and converted on use.
template <class S, class R> struct SiteLinks {
    typedef typename Vec<S>::type VT;
    static constexpr int W = Vec<S>::W;
    VT u[72 / W];
    R sc;
    template <bool NT = false>
    __device__ __forceinline__ void init(const S *__restrict__ base, const float *__restrict__ scale,
                                         int64_t bp, int s, int Vbh) {
        const VT *p = reinterpret_cast<const VT *>(base);
#pragma unroll
        for (int v = 0; v < 72 / W; ++v) u[v] = ld_vec<NT>(p + vec_index<S, 72>(bp, v, s, Vbh));
        if constexpr (Storage<S>::scaled) sc = (R)*gmem(scale + bp * Vbh + s);
        else sc = (R)1;
    }
    // Link MU without the FP16 site scale (see scale()).
    template <int MU> __device__ __forceinline__ void get(R out[18]) const {
#pragma unroll
        for (int k = 0; k < 18; ++k) {
            const int q = 18 * MU + k;
            if constexpr (Storage<S>::scaled) out[k] = (R)(float)u[q / W][q % W];
            else out[k] = (R)u[q / W][q % W];
        }
    }
    __device__ __forceinline__ R scale() const {
        if constexpr (Storage<S>::scaled) return sc;
        else return (R)1;
    }
};

// Per-site packed clover (72 reals) in registers as the storage-precision vectors it was
// loaded in; entries are converted one at a time where they are used.
template <class S, class R> struct CloverRegs {
    typedef typename Vec<S>::type VT;
    static constexpr int W = Vec<S>::W;
    VT x[72 / W];
    R sc;
    template <bool NT = false>
    __device__ __forceinline__ void load(const S *__restrict__ base, const float *__restrict__ scale, int64_t bp,
                                         int s, int Vbh) {
        const VT *p = reinterpret_cast<const VT *>(base);
#pragma unroll
        for (int v = 0; v < 72 / W; ++v) x[v] = ld_vec<NT>(p + vec_index<S, 72>(bp, v, s, Vbh));
        if constexpr (Storage<S>::scaled) sc = (R)*gmem(scale + bp * Vbh + s);
        else sc = (R)1;
    }
    // Entry k without the FP16 site scale (clover_mul applies it).
    __device__ __forceinline__ R at(int k) const {
        if constexpr (Storage<S>::scaled) return (R)(float)x[k / W][k % W];
        else return (R)x[k / W][k % W];
    }
    __device__ __forceinline__ R scale() const {
        if constexpr (Storage<S>::scaled) return sc;
        else return (R)1;
    }
};

// out = in + kx * X in for the two packed Hermitian 6x6 blocks of X: X in is accumulated
// from the stored entries with FMAs and scaled once (kx times the site scale).
template <class XR, class R>
__device__ __forceinline__ void clover_mul(const XR &X, const R (&in)[24], R (&out)[24], R kx) {
    const R f = kx * X.scale();
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        const int o = 12 * blk;
        R t[12];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const R d = X.at(36 * blk + i);
            t[2 * i] = fmac(d, in[o + 2 * i], (R)0);
            t[2 * i + 1] = fmac(d, in[o + 2 * i + 1], (R)0);
        }
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = i + 1; j < 6; ++j) {
                const int q = 36 * blk + 6 + 2 * (i * 5 - i * (i - 1) / 2 + (j - i - 1));
                const R xr = X.at(q), xi = X.at(q + 1);
                t[2 * i] = fmac(xr, in[o + 2 * j], t[2 * i]);
                t[2 * i] = fmac(-xi, in[o + 2 * j + 1], t[2 * i]);
                t[2 * i + 1] = fmac(xr, in[o + 2 * j + 1], t[2 * i + 1]);
                t[2 * i + 1] = fmac(xi, in[o + 2 * j], t[2 * i + 1]);
                t[2 * j] = fmac(xr, in[o + 2 * i], t[2 * j]);
                t[2 * j] = fmac(xi, in[o + 2 * i + 1], t[2 * j]);
                t[2 * j + 1] = fmac(xr, in[o + 2 * i + 1], t[2 * j + 1]);
                t[2 * j + 1] = fmac(-xi, in[o + 2 * i], t[2 * j + 1]);
            }
#pragma unroll
        for (int k = 0; k < 12; ++k) out[o + k] = fmac(f, t[k], in[o + k]);
    }
}

// In-block hopping term between the two parities, via LDS.
//   Threads of parity `src` supply `in`. Threads of the other parity receive
//   out = sum_mu [ (1 - gamma_mu) U_mu(x) in(x + mu) + (1 + gamma_mu) U_mu(x - mu)^+ in(x - mu) ]
//   over the neighbours inside the block (hops leaving the block are dropped); source
//   threads leave `out` untouched.
// Source threads store their spinor (for the forward hops of their backward neighbours)
// and, for every in-block forward neighbour, the transported half spinor
// U_mu(x)^+ (1 + gamma_mu) in(x); the receiving threads then need only their own links.
// Every thread of the workgroup must call this; it contains two barriers. Face sites skip
// the hops that leave the block: their links are not loaded (the block operator, whose
// kernels use this, is bound by memory).
template <int MU, class BK, class R, class LK>
__device__ __forceinline__ void push_dir(const SiteInfo &si, const LK &U, const R (&in)[24], R *__restrict__ hb) {
    constexpr int Vbh = BK::Vbh;
    if (si.fin & (1u << MU)) {
        R h[12], uh[12], u[18];
        project<MU, +1>(in, h);
        U.template get<MU>(u);
        su3_dag_mul(u, h, uh);
        const R sc = U.scale();
#pragma unroll
        for (int k = 0; k < 12; ++k) hb[(MU * 12 + k) * Vbh + si.s] = sc * uh[k];
    }
}

template <int MU, class BK, class R, class LK>
__device__ __forceinline__ void pull_dir(const SiteInfo &si, const LK &U, R (&out)[24], const R *__restrict__ sp,
                                         const R *__restrict__ hb) {
    constexpr int Vbh = BK::Vbh;
    if (si.fin >> MU & 1u) {
        R chi[24], h[12], uh[12], u[18];
        const int n = si.nbf[MU];
#pragma unroll
        for (int k = 0; k < 24; ++k) chi[k] = sp[k * Vbh + n];
        project<MU, -1>(chi, h);
        U.template get<MU>(u);
        su3_mul(u, h, uh);
        accum_recon<MU, -1>(out, uh, U.scale());
    }
    if (si.bin >> MU & 1u) {
        R uh[12];
        const int n = si.nbb[MU];
#pragma unroll
        for (int k = 0; k < 12; ++k) uh[k] = hb[(MU * 12 + k) * Vbh + n];
        accum_recon<MU, +1>(out, uh, (R)1);
    }
}

// Reals of LDS that block_hop needs: a spinor and four transported half spinors per source
// site.
template <class BK> struct HopLds {
    static constexpr int PER = 72 * BK::Vbh;
};

template <class BK, class R, class LK>
__device__ __forceinline__ void block_hop(int src, const SiteInfo &si, const LK &U, const R (&in)[24], R (&out)[24],
                                          R *__restrict__ lds) {
    constexpr int Vbh = BK::Vbh;
    R *__restrict__ sp = lds;
    R *__restrict__ hb = lds + 24 * Vbh;
    if (si.p == src) {
#pragma unroll
        for (int k = 0; k < 24; ++k) sp[k * Vbh + si.s] = in[k];
        push_dir<0, BK>(si, U, in, hb);
        push_dir<1, BK>(si, U, in, hb);
        push_dir<2, BK>(si, U, in, hb);
        push_dir<3, BK>(si, U, in, hb);
    }
    __syncthreads();
    if (si.p != src) {
#pragma unroll
        for (int k = 0; k < 24; ++k) out[k] = 0;
        pull_dir<0, BK>(si, U, out, sp, hb);
        pull_dir<1, BK>(si, U, out, sp, hb);
        pull_dir<2, BK>(si, U, out, sp, hb);
        pull_dir<3, BK>(si, U, out, sp, hb);
    }
    __syncthreads();  // the next hop may only overwrite the buffer after every read
}

// LDS of a block operator kernel: the hops' exchange area, then the results on their way to
// the canonical array.
template <class BK, class S, class R> struct BlockLds {
    static constexpr int hop = HopLds<BK>::PER * (int)sizeof(R), out = BK::NT * (int)sizeof(CanonSlot<S>);
    static constexpr int bytes = hop > out ? hop : out;
};
template <class BK> __device__ __forceinline__ int64_t canon_index_bk(const Geom &geo, int64_t b, const int (&l)[4]) {
    int g[4];
    block_coords(geo.G, b, g);
    return g[0] * BK::bx + l[0] +
           (int64_t)geo.L[0] * (g[1] * BK::by + l[1] +
                                (int64_t)geo.L[1] * (g[2] * BK::bz + l[2] + (int64_t)geo.L[2] * (g[3] * BK::bt + l[3])));
}
// Block and right-hand side of workgroup w of Nd * nrhs (Nd a multiple of 8): workgroups run on XCD
// w mod 8, and the right-hand sides of one block follow each other there, so that all but the
// first read its links and clover from that XCD's L2. A call in us, all blocks of one
// right-hand side first / this order: 24 x 8 x 40 x 56, 4^4, 3 rhs FP64 413 / 350, FP32 204 / 181;
// 32^3 x 64, 8x4^3, 4 rhs FP64 3336 / 3179, FP32 1596 / 1317, FP16 1235 / 1160.
__device__ __forceinline__ int64_t block_and_rhs(int nrhs, int &rhs) {
    const int w = blockIdx.x, k = w >> 3;
    rhs = k % nrhs;
    return (int64_t)(k / nrhs) * 8 + (w & 7);
}
// The site at canonical index idx, in storage precision S.
template <class S, class R> __device__ __forceinline__ void block_load(const double *in, int64_t idx, R (&psi)[24]) {
    double e[24];
    canon_load(in, idx, e);
    round_site<S>(e, psi);
}
// Every thread's site (local coordinates l), rounded to storage precision S, to the canonical
// array. The last hop's barrier has freed the exchange area.
template <class BK, class S, class R>
__device__ __forceinline__ void block_store(double *out, int64_t idx, const int (&l)[4], const R (&res)[24], char *lds) {
    CanonSlot<S> *st = reinterpret_cast<CanonSlot<S> *>(lds);
    CanonSlot<S> &slot = st[l[0] + BK::bx * (l[1] + BK::by * (l[2] + BK::bz * l[3]))];
    slot.set(res);
    slot.idx = idx;
    __syncthreads();
    canon_put<BK::NT>(out, st);
}

}  // namespace sapdd
