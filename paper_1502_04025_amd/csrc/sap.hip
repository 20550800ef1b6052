// sap.hip - one colour half-sweep of the Schwarz alternating procedure (Sec. 3.1): for
// every block B of one colour, in parallel, one workgroup
//   1. forms the block residual rho_B: the stored even-site MR residual of B's previous
//      solve (odd sites: 0), or the input eta on the first cycle, plus the change the
//      other colour's last corrections made to it - a gather of the hops from the
//      neighbouring blocks' corrections delta into B's boundary sites;
//   2. solves M_B delta = rho_B approximately with even-odd preconditioning:
//      bhat_e = rho_e - K_eo A_o^-1 rho_o, nmr minimal-residual steps on
//      Dhat = A_e - K_eo A_o^-1 K_oe from zero, delta_o = A_o^-1 (rho_o - K_oe delta_e),
//      with K = -kappa * (in-block hopping);
//   3. adds delta to psi and keeps delta and the new even-site residual for the next
//      half-sweep.
// The block never leaves the workgroup during the MR iterations: spinors live in
// registers and LDS and the MR inner products are wave plus LDS reductions in a fixed
// order (so results do not depend on scheduling). Blocks of one colour share no site and
// no hop, so the gather form (each block reads its neighbours, nobody writes into another
// block) is race free.
//
// Two threads per pair of sites. Lane l < 32 of a wave and lane l + 32 share the even and
// the odd site with one half index. In a hop the lower lane does the four forward hops of
// the receiving site, the upper lane the four backward hops, both from the source
// parity's spinors in LDS; afterwards v_permlane32_swap exchanges the halves of the two
// partial sums, so that the lower lane holds spins 0-1 and the upper lane spins 2-3 of the
// result. The clover term is diagonal in that chirality, as are all vector updates, so
// between the hops every lane works on the 12 reals of its own chirality. Every wave is
// busy in every phase and a thread's state is half a spinor per vector.
// Both directions run one instruction stream: a backward hop is
//   (1 + gamma) U^+ psi = conj((1 + gamma*) U^T conj(psi)),
// the same product with the link transposed and conjugations that fold into the signs of
// the projection's and the reconstruction's FMAs.
//
// What bounds it: with FP16 links and clover the issue of vector instructions (each hop is
// 72 FMAs of SU(3) arithmetic per direction and lane, plus projection, reconstruction and
// the transposition); with FP32 and FP64 fields also the links and clover that every MR
// step re-reads through the caches (an 8x4^3 domain holds 295 KB of them in FP32, and 16 to
// 32 domains share an XCD's 4 MB L2).
// Two lanes per pair instead of one thread per pair or per site: the state of a lane is
// half as large, so FP16 and FP32 run 4 waves per SIMD in 128 registers and FP64 2 waves in
// 256 nearly without spills, no wave idles in one half of a hop, and the exchange costs 24
// register instructions instead of an LDS round trip. Measured per half-sweep (4 MR steps)
// against the one-thread-per-pair and one-thread-per-site kernels this replaced:
//   4^4 lattice, 2^4 domains, FP64, 1 rhs        74.8 -> 29.1 us
//   16^3 x 32, 8x4^3, FP32 / FP64, 1 rhs         68.8 -> 43.3 us / 442 -> 90.8 us
//   24^3 x 48, 4^4, FP16, 5 rhs                   564 -> 419 us
//   32^3 x 64, 8x4^3, FP16, 12 rhs               3860 -> 3097 us
//   32^3 x 64, 8x4^3, FP32, 4 rhs                2187 -> 1330 us
// At 32^3 x 64, 12 rhs the FP16 kernel issues 7970 vector instructions per wave and is
// issuing them 88% of the time.
//
// Odd sites (ODD_LAST in the kernel). With FP32 and FP64 links delta_o is formed once, from the
// final delta_e, by a closing hop and clover product. With FP16 links
// delta_o = A_o^-1 rho_o + kappa sum_i alpha_i A_o^-1 H_oe r_i is accumulated during the MR steps
// from the vectors A_o^-1 H_oe r_i they form anyway. The sum rounds delta_o in every step, which
// doubles its error (the next half-sweep takes the odd residual as zero). Relative error of a
// whole sweep and time of a call of 16 half-sweeps, 16^3 x 32, 8x4^3, accumulated / formed once:
//   FP64 (8^4, 4^4) 2.24e-16 / 2.09e-16, 1396 / 1506 us
//   FP32 1.221e-7 / 1.150e-7, 714 / 748 us
//   FP16 links, FP16 spinors 1.111e-4 / 1.111e-4, 712 / 761 us
//   FP16 links, FP32 spinors 9.840e-5 / 9.840e-5, 720 / 765 us
// The rounding of FP16 links hides the sum's, so there the cheaper form stays.
//
// Clover input X per rhs: X = kappa T on even sites (A_e = 1 + X) and
// X = A_o^-1 - 1 on odd sites (A_o^-1 = 1 + X).
#include <limits>

#include "blockgeo.hpp"
#include "kernels.hpp"
#include "lanes.hpp"

namespace sapdd {

template <class S, class SS, class P> struct SapArgs {  // S: links and clover, SS: spinors
    Geom geo;
    const S *links;
    const float *lscale;
    const S *const *X;
    const float *const *Xsc;
    const double *kappa;
    const double *eta;
    const double *eta_scale;
    int eta_scale_stride;
    int64_t eta_stride;  // doubles per rhs
    SS *rres;
    float *rres_sc;
    SS *delta;
    float *delta_sc;
    P *psi;
    int64_t psi_stride;  // elements per rhs
    const int *active;
    int nact;
    int colour, mode, write_state, nmr;
};

namespace {

// ------------------------------------------------------------------ lanes
// Sum over the lanes of one block (GROUP = 64: the whole wave; GROUP = 8: lanes 8 g .. 8 g
// + 7 and the same lanes + 32) in a fixed order, the same on each of them. Register to
// register: DPP adds inside rows of 16 lanes, then the rows' sums.
template <int GROUP, class R> __device__ __forceinline__ R lane_sum(R v) {
    v = v + dpp_move<0xB1>(v);  // quad_perm [1,0,3,2]
    v = v + dpp_move<0x4E>(v);  // quad_perm [2,3,0,1]
    if constexpr (GROUP == 64) {
        v = v + dpp_move<0x124>(v);  // row_ror:4
        v = v + dpp_move<0x128>(v);  // row_ror:8
        return ((lane_value(v, 0) + lane_value(v, 16)) + lane_value(v, 32)) + lane_value(v, 48);
    } else {
        v = v + dpp_move<0x141>(v);  // row_half_mirror: the other quad of 8 lanes
        R w = v;
        swap32(v, w);
        return v + w;
    }
}

// ------------------------------------------------------------------ tile of one workgroup
template <class BK, class R> struct Tile {
    static constexpr int Vbh = BK::Vbh;
    static constexpr int PER = Vbh < 32 ? 32 / Vbh : 1;  // (block, rhs) pairs per workgroup
    static constexpr int NCOL = Vbh * PER;               // columns: even/odd site pairs
    static constexpr int NT = 2 * NCOL;
    static constexpr int NW = NT / 64;
    static constexpr int CW = 16 / (int)sizeof(R);       // reals per 16-byte LDS vector
    static constexpr int OWN = 12 / CW;                  // vectors of one chirality
    static constexpr int BUF = 2 * OWN * NCOL;           // vectors per LDS buffer (one spinor per column)
    typedef R VR __attribute__((ext_vector_type(16 / sizeof(R))));
};

// A thread's place: column col (site half index s of its block), f = 0 lower lane (forward
// hops, spins 0-1) or 1 upper lane (backward hops, spins 2-3); c = 1 or -1 accordingly.
template <class BK, class R> struct Lane {
    int s, f, col, col0;  // col0: first column of this thread's block
    R c;
    // For the site of either parity: the half index of its neighbour (forward or backward by
    // f) in direction mu in byte mu of nb, s where that lies outside the block, and bit mu
    // of in set where it lies inside.
    unsigned nb[2], in[2];
    __device__ __forceinline__ Lane() {
        typedef Tile<BK, R> T;
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
        f = lane >> 5;
        col = 32 * wv + (lane & 31);
        s = T::PER > 1 ? col % BK::Vbh : col;
        col0 = T::PER > 1 ? col - s : 0;
        c = f ? (R)-1 : (R)1;
        const int B[4] = {BK::bx, BK::by, BK::bz, BK::bt};
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            int l[4];
            local_coords(B, p, s, l);
            in[p] = nb[p] = 0;
#pragma unroll
            for (int mu = 0; mu < 4; ++mu) {
                int m[4] = {l[0], l[1], l[2], l[3]};
                m[mu] += f ? -1 : 1;
                const bool inside = f ? l[mu] > 0 : l[mu] < B[mu] - 1;
                in[p] |= inside ? 1u << mu : 0u;
                nb[p] |= (unsigned)(inside ? local_half_index(B, m) : s) << (8 * mu);
            }
        }
    }
    // Neighbour index and weight (1 inside, 0 outside) of direction MU at parity PR. The
    // empty asm keeps what is computed from them out of the loop-invariant registers: as
    // loop invariants the addresses of a hop's loads alone would fill the register file.
    template <int PR, int MU> __device__ __forceinline__ int neighbour() const {
        unsigned v = nb[PR];
        asm volatile("" : "+v"(v));
        return (int)(v >> (8 * MU) & 255u);
    }
    template <int PR, int MU> __device__ __forceinline__ R weight() const {
        unsigned v = in[PR];
        asm volatile("" : "+v"(v));
        return (R)(int)(v >> MU & 1u);
    }
};

// ------------------------------------------------------------------ loads
// A block's part of a field: every load is a uniform base, a 32-bit offset per lane and a
// constant. UNI (one block per workgroup): buffer loads, which take exactly that form and
// return zeros past the block's end; else (2^4 blocks, several blocks per wave) plain
// global loads from a base per lane.
template <bool UNI> struct View;
template <> struct View<true> {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ void set(const void *p, int bytes) {
        r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
    }
};
template <> struct View<false> {
    const char *p;
    __device__ __forceinline__ void set(const void *q, int) { p = (const char *)q; }
};
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x3 __attribute__((ext_vector_type(3)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x3a __attribute__((ext_vector_type(3), aligned(4)));
// N dwords (1..4) at byte offset off + C.
template <int N> __device__ __forceinline__ void load_dwords(const View<true> &v, unsigned off, int C, unsigned *out) {
    if constexpr (N == 1) {
        out[0] = __builtin_amdgcn_raw_buffer_load_b32(v.r, (int)off, C, 0);
    } else if constexpr (N == 2) {
        const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(v.r, (int)off, C, 0);
        out[0] = x[0], out[1] = x[1];
    } else if constexpr (N == 3) {
        const u32x3 x = __builtin_amdgcn_raw_buffer_load_b96(v.r, (int)off, C, 0);
        out[0] = x[0], out[1] = x[1], out[2] = x[2];
    } else {
        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(v.r, (int)off, C, 0);
        out[0] = x[0], out[1] = x[1], out[2] = x[2], out[3] = x[3];
    }
}
template <int N> __device__ __forceinline__ void load_dwords(const View<false> &v, unsigned off, int C, unsigned *out) {
    const char *p = v.p + (size_t)off + C;
    if constexpr (N == 1) {
        out[0] = *gmem(reinterpret_cast<const unsigned *>(p));
    } else if constexpr (N == 2) {
        const u32x2 x = *gmem(reinterpret_cast<const u32x2 *>(p));
        out[0] = x[0], out[1] = x[1];
    } else if constexpr (N == 3) {
        const u32x3a x = *(const SAPDD_GLOBAL u32x3a *)p;
        out[0] = x[0], out[1] = x[1], out[2] = x[2];
    } else {
        const u32x4 x = *gmem(reinterpret_cast<const u32x4 *>(p));
        out[0] = x[0], out[1] = x[1], out[2] = x[2], out[3] = x[3];
    }
}
// Dwords D0 .. D0 + N - 1 of a site whose vectors of four dwords lie VS bytes apart, in
// loads of exactly those bytes.
template <int D0, int N, int VS, class VW>
__device__ __forceinline__ void load_site_dwords(const VW &v, unsigned off, unsigned *out) {
    if constexpr (N > 0) {
        constexpr int here = 4 - D0 % 4 < N ? 4 - D0 % 4 : N;
        load_dwords<here>(v, off, D0 / 4 * VS + D0 % 4 * 4, out);
        load_site_dwords<D0 + here, N - here, VS>(v, off, out + here);
    }
}
__device__ __forceinline__ float as_real(const unsigned *d, float) { return __builtin_bit_cast(float, d[0]); }
__device__ __forceinline__ double as_real(const unsigned *d, double) {
    return __builtin_bit_cast(double, (uint2){d[0], d[1]});
}
template <class VW> __device__ __forceinline__ float load_float(const VW &v, unsigned off) {
    unsigned x;
    load_dwords<1>(v, off, 0, &x);
    return __builtin_bit_cast(float, x);
}

// ------------------------------------------------------------------ links
// Link MU of the site whose vector 0 lies at byte offset off (vectors VS bytes apart),
// transposed if tr: nine complex entries in storage precision. FP64 entries are vectors of
// their own, so there the transposition is in the addresses; FP32 and FP16 entries change
// places in registers (use: after their arrival).
template <int MU, class S, int VS> struct Link;

template <int MU, int VS> struct Link<MU, double, VS> {
    unsigned d[36];
    template <class VW> __device__ __forceinline__ void load(const VW &v, unsigned off, bool tr) {
        const unsigned t = tr ? 2 * VS : 0, n = 2 * VS - t;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {  // entry (a, b) or (b, a), 2 |a - b| vectors apart
                const int lo = a < b ? 3 * a + b : 3 * b + a, dist = a < b ? b - a : a - b;
                load_dwords<4>(v, off + (unsigned)dist * (a < b ? t : n), (9 * MU + lo) * VS, d + 4 * (3 * a + b));
            }
    }
    __device__ __forceinline__ void arrive(bool) {}
    template <class R> __device__ __forceinline__ R re(int k) const { return (R)as_real(d + 4 * k, 0.0); }
    template <class R> __device__ __forceinline__ R im(int k) const { return (R)as_real(d + 4 * k + 2, 0.0); }
};

__device__ __forceinline__ void swap_if(bool tr, unsigned &a, unsigned &b) {
    const unsigned x = tr ? b : a, y = tr ? a : b;
    a = x;
    b = y;
}

template <int MU, int VS> struct Link<MU, float, VS> {
    unsigned d[18];
    template <class VW> __device__ __forceinline__ void load(const VW &v, unsigned off, bool) {
        load_site_dwords<18 * MU, 18, VS>(v, off, d);
    }
    __device__ __forceinline__ void arrive(bool tr) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            swap_if(tr, d[2 * 1 + q], d[2 * 3 + q]);
            swap_if(tr, d[2 * 2 + q], d[2 * 6 + q]);
            swap_if(tr, d[2 * 5 + q], d[2 * 7 + q]);
        }
    }
    template <class R> __device__ __forceinline__ R re(int k) const { return (R)as_real(d + 2 * k, 0.f); }
    template <class R> __device__ __forceinline__ R im(int k) const { return (R)as_real(d + 2 * k + 1, 0.f); }
};

typedef half_t half2v __attribute__((ext_vector_type(2)));
template <int MU, int VS> struct Link<MU, half_t, VS> {
    unsigned d[9];  // without the site scale
    template <class VW> __device__ __forceinline__ void load(const VW &v, unsigned off, bool) {
        load_site_dwords<9 * MU, 9, VS>(v, off, d);
    }
    __device__ __forceinline__ void arrive(bool tr) {
        swap_if(tr, d[1], d[3]);
        swap_if(tr, d[2], d[6]);
        swap_if(tr, d[5], d[7]);
    }
    template <class R> __device__ __forceinline__ R re(int k) const {
        return (R)(float)__builtin_bit_cast(half2v, d[k])[0];
    }
    template <class R> __device__ __forceinline__ R im(int k) const {
        return (R)(float)__builtin_bit_cast(half2v, d[k])[1];
    }
};

// A neighbour's spinor as it is read: component k as an R. FP16 sites keep their halves
// (without the site scale), which the projection's FMAs take as they are.
template <class R, class S> struct Chi {
    R v[24];
    __device__ __forceinline__ R operator()(int k) const { return v[k]; }
};
template <class R> struct Chi<R, half_t> {
    unsigned d[12];
    __device__ __forceinline__ R operator()(int k) const {
        return (R)(float)__builtin_bit_cast(half2v, d[k / 2])[k % 2];
    }
};

// One hop in direction MU by this lane, up to the reconstruction: (1 - gamma) U chi
// (forward, c = 1) or (1 + gamma) U^+ chi (backward, c = -1, u transposed). With sg = -c
// the projected half spinor is h = up + sg G lo; backward it is conjugated, so its
// imaginary part is c up - G lo in both cases (c sg = -1), and that of uh carries c.
template <int MU, class R, class CHI, class LK>
__device__ __forceinline__ void hop_half(const CHI &chi, const LK &u, R c, R (&uh)[12]) {
    R h[12];
    auto proj = [&](auto row) {
        constexpr int ROW = decltype(row)::value;
        constexpr int col = Grow<MU, ROW>::col, ph = Grow<MU, ROW>::ph;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            R re, im;
            iph<ph>(chi(2 * (3 * (2 + col) + a)), chi(2 * (3 * (2 + col) + a) + 1), re, im);
            h[2 * (3 * ROW + a)] = fmac(-c, re, chi(2 * (3 * ROW + a)));
            h[2 * (3 * ROW + a) + 1] = fmac(c, chi(2 * (3 * ROW + a) + 1), -im);
        }
    };
    proj(std::integral_constant<int, 0>{});
    proj(std::integral_constant<int, 1>{});
#pragma unroll
    for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            R re = fmac(u.template re<R>(3 * a), h[6 * sp], (R)0);
            R im = fmac(u.template re<R>(3 * a), h[6 * sp + 1], (R)0);
            re = fmac(-u.template im<R>(3 * a), h[6 * sp + 1], re);
            im = fmac(u.template im<R>(3 * a), h[6 * sp], im);
#pragma unroll
            for (int b = 1; b < 3; ++b) {
                const R ur = u.template re<R>(3 * a + b), ui = u.template im<R>(3 * a + b);
                re = fmac(ur, h[6 * sp + 2 * b], re);
                re = fmac(-ui, h[6 * sp + 2 * b + 1], re);
                im = fmac(ur, h[6 * sp + 2 * b + 1], im);
                im = fmac(ui, h[6 * sp + 2 * b], im);
            }
            uh[6 * sp + 2 * a] = re;
            uh[6 * sp + 2 * a + 1] = im;
        }
}
// The reconstruction: acc_up += w (re, c im), acc_lo += sg w i^ph (re, c im), wc = w c.
template <int MU, class R> __device__ __forceinline__ void hop_recon(const R (&uh)[12], R w, R wc, R (&acc)[24]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        acc[2 * k] = fmac(w, uh[2 * k], acc[2 * k]);
        acc[2 * k + 1] = fmac(wc, uh[2 * k + 1], acc[2 * k + 1]);
    }
    auto recon = [&](auto row) {
        constexpr int ROW = decltype(row)::value;
        constexpr int col = GDrow<MU, ROW>::col, ph = GDrow<MU, ROW>::ph;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const R re = uh[2 * (3 * col + a)], im = uh[2 * (3 * col + a) + 1];
            R &xr = acc[2 * (6 + 3 * ROW + a)], &xi = acc[2 * (6 + 3 * ROW + a) + 1];
            // sg i^ph (re, c im) = (-c) i^ph (re, c im)
            if constexpr (ph == 0) {
                xr = fmac(-wc, re, xr);
                xi = fmac(-w, im, xi);
            } else if constexpr (ph == 1) {
                xr = fmac(w, im, xr);
                xi = fmac(-wc, re, xi);
            } else if constexpr (ph == 2) {
                xr = fmac(wc, re, xr);
                xi = fmac(w, im, xi);
            } else {
                xr = fmac(-w, im, xr);
                xi = fmac(wc, re, xi);
            }
        }
    };
    recon(std::integral_constant<int, 0>{});
    recon(std::integral_constant<int, 1>{});
}
template <int MU, class R, class CHI, class LK>
__device__ __forceinline__ void hop_dir(const CHI &chi, const LK &u, R c, R w, R (&acc)[24]) {
    R uh[12];
    hop_half<MU>(chi, u, c, uh);
    hop_recon<MU>(uh, w, w * c, acc);
}

// The sum of the two lanes' partial spinors, each lane keeping its own chirality.
template <class R> __device__ __forceinline__ void fold(R (&acc)[24], R (&out)[12]) {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        swap32(acc[k], acc[12 + k]);
        out[k] = acc[k] + acc[12 + k];
    }
}

// ------------------------------------------------------------------ own-chirality storage
// The 12 reals of chirality f of site (bp, s) in a 24-real field, 16 bytes at a time (8 for
// FP16, whose site has three 16-byte vectors).
template <class R, class S>
__device__ __forceinline__ void load_half(const S *data, const float *scale, int64_t bp, int s, int f, int Vbh,
                                          R (&out)[12]) {
    if constexpr (Storage<S>::scaled) {
        typedef half_t h4 __attribute__((ext_vector_type(4)));
        const R sc = (R)*gmem(scale + bp * Vbh + s);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int q = 3 * f + i;
            const h4 x = *gmem(reinterpret_cast<const h4 *>(data) + 2 * ((bp * 3 + (q >> 1)) * Vbh + s) + (q & 1));
#pragma unroll
            for (int w = 0; w < 4; ++w) out[4 * i + w] = (R)(float)x[w] * sc;
        }
    } else {
        typedef typename Vec<S>::type VT;
        constexpr int W = Vec<S>::W;
#pragma unroll
        for (int v = 0; v < 12 / W; ++v) {
            const VT x = *gmem(reinterpret_cast<const VT *>(data) + (bp * (24 / W) + f * (12 / W) + v) * (int64_t)Vbh + s);
#pragma unroll
            for (int w = 0; w < W; ++w) out[v * W + w] = (R)x[w];
        }
    }
}
// Store them; FP16 divides by the site's max |value| over both lanes and rounds to nearest
// even (scale 0 stores zeros). Every lane of the wave calls this.
template <class R, class S>
__device__ __forceinline__ void store_half(S *data, float *scale, int64_t bp, int s, int f, int Vbh, const R (&in)[12]) {
    if constexpr (Storage<S>::scaled) {
        typedef half_t h4 __attribute__((ext_vector_type(4)));
        float m = 0.f;
#pragma unroll
        for (int k = 0; k < 12; ++k) m = fmaxf(m, fabsf((float)in[k]));
        float o = m;
        swap32(m, o);
        m = fmaxf(m, o);
        const float inv = fp16_site_inv(m);
        if (f == 0) *gmem(scale + bp * Vbh + s) = inv > 0.f ? m : 0.f;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int q = 3 * f + i;
            h4 x;
#pragma unroll
            for (int w = 0; w < 4; ++w) x[w] = (half_t)((float)in[4 * i + w] * inv);
            *gmem(reinterpret_cast<h4 *>(data) + 2 * ((bp * 3 + (q >> 1)) * Vbh + s) + (q & 1)) = x;
        }
    } else {
        typedef typename Vec<S>::type VT;
        constexpr int W = Vec<S>::W;
#pragma unroll
        for (int v = 0; v < 12 / W; ++v) {
            VT x;
#pragma unroll
            for (int w = 0; w < W; ++w) x[w] = (S)in[v * W + w];
            *gmem(reinterpret_cast<VT *>(data) + (bp * (24 / W) + f * (12 / W) + v) * (int64_t)Vbh + s) = x;
        }
    }
}

// The packed 6x6 block of one chirality: 36 reals in storage precision. FP16: nine 8-byte
// pieces, piece q of a site in the (q & 1) half of vector q >> 1.
template <class S, int VS> struct CloverHalf {
    static constexpr int W = Vec<S>::W, DW = (int)sizeof(S) / 4;
    unsigned d[36 * DW];
    template <class VW> __device__ __forceinline__ void load(const VW &v, unsigned off, int f) {
        const unsigned o = off + (f ? 36 / W * VS : 0);
#pragma unroll
        for (int q = 0; q < 36 / W; ++q) load_dwords<4>(v, o, q * VS, d + 4 * q);
    }
    template <class R> __device__ __forceinline__ R at(int k) const { return (R)as_real(d + DW * k, (S)0); }
    // To and from LDS: this thread's vectors, nt threads apart.
    __device__ __forceinline__ void put(u32x4 *lds, int nt) const {
#pragma unroll
        for (int q = 0; q < 9 * DW; ++q) lds[q * nt + threadIdx.x] = u32x4{d[4 * q], d[4 * q + 1], d[4 * q + 2], d[4 * q + 3]};
    }
    __device__ __forceinline__ void get(const u32x4 *lds, int nt) {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));  // read where it is used, not kept in registers across the MR loop
#pragma unroll
        for (int q = 0; q < 9 * DW; ++q) {
            const u32x4 x = lds[q * nt + t];
#pragma unroll
            for (int k = 0; k < 4; ++k) d[4 * q + k] = x[k];
        }
    }
};
template <int VS> struct CloverHalf<half_t, VS> {
    unsigned d[18];
    template <class VW> __device__ __forceinline__ void load(const VW &v, unsigned off, int f) {
        // piece 9 f + i: for f = 1 an even i starts in the upper half of vector 4 + i / 2,
        // an odd i in the lower half of vector 5 + i / 2
        const unsigned oe = off + (f ? 4 * VS + 8 : 0), oo = off + (f ? 5 * VS : 8);
#pragma unroll
        for (int i = 0; i < 9; ++i) load_dwords<2>(v, i & 1 ? oo : oe, i / 2 * VS, d + 2 * i);
    }
    template <class R> __device__ __forceinline__ R at(int k) const {
        return (R)(float)__builtin_bit_cast(half2v, d[k / 2])[k % 2];
    }
};

// out = in + fx X in for one chirality (fx: the FP16 site scale, else 1).
template <class XR, class R>
__device__ __forceinline__ void clover_half_mul(const XR &X, const R (&in)[12], R (&out)[12], R fx) {
    R t[12];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const R d = X.template at<R>(i);
        t[2 * i] = fmac(d, in[2 * i], (R)0);
        t[2 * i + 1] = fmac(d, in[2 * i + 1], (R)0);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = i + 1; j < 6; ++j) {
            const int q = 6 + 2 * (i * 5 - i * (i - 1) / 2 + (j - i - 1));
            const R xr = X.template at<R>(q), xi = X.template at<R>(q + 1);
            t[2 * i] = fmac(xr, in[2 * j], t[2 * i]);
            t[2 * i] = fmac(-xi, in[2 * j + 1], t[2 * i]);
            t[2 * i + 1] = fmac(xr, in[2 * j + 1], t[2 * i + 1]);
            t[2 * i + 1] = fmac(xi, in[2 * j], t[2 * i + 1]);
            t[2 * j] = fmac(xr, in[2 * i], t[2 * j]);
            t[2 * j] = fmac(xi, in[2 * i + 1], t[2 * j]);
            t[2 * j + 1] = fmac(xr, in[2 * i + 1], t[2 * j + 1]);
            t[2 * j + 1] = fmac(-xi, in[2 * i], t[2 * j + 1]);
        }
#pragma unroll
    for (int k = 0; k < 12; ++k) out[k] = fmac(fx, t[k], in[k]);
}

// ------------------------------------------------------------------ one block
// The resident fields of a thread's block.
template <class BK, class S, class R> struct BlockView {
    static constexpr bool UNI = Tile<BK, R>::PER == 1;
    static constexpr int VS = BK::Vbh * 16;           // bytes between a site's vectors
    static constexpr int NV = 72 / Vec<S>::W;         // vectors per link / clover site
    View<UNI> links, X, lsc, xsc;
    __device__ __forceinline__ static unsigned off(int p, int s) { return (unsigned)(p * NV * VS + s * 16); }
    __device__ __forceinline__ R lscale(int p, int s) const {
        if constexpr (Storage<S>::scaled) return (R)load_float(lsc, (unsigned)((p * BK::Vbh + s) * 4));
        else return (R)1;
    }
    __device__ __forceinline__ R xscale(int p, int s) const {
        if constexpr (Storage<S>::scaled) return (R)load_float(xsc, (unsigned)((p * BK::Vbh + s) * 4));
        else return (R)1;
    }
    // out = (1 + X) in at the site of parity P
    template <int P> __device__ __forceinline__ void clover(const Lane<BK, R> &ln, const R (&in)[12], R (&out)[12]) const {
        CloverHalf<S, VS> c;
        int s = ln.s;
        asm volatile("" : "+v"(s));
        c.load(X, off(P, s), ln.f);
        clover_half_mul(c, in, out, xscale(P, s));
    }
};

// One direction of an in-block hop into the sites of parity PR: the link and its weight
// (0 for a lane without the neighbour inside the block), loaded ahead of their use. The
// link sits at the receiving site (forward) or at the source (backward).
template <int PR, int MU, class BK, class S, class R> struct HopLink {
    Link<MU, S, BlockView<BK, S, R>::VS> u;
    R sc;
    __device__ __forceinline__ void load(const BlockView<BK, S, R> &bv, const Lane<BK, R> &ln) {
        const int n = ln.template neighbour<PR, MU>();
        const int lp = ln.f ? 1 - PR : PR, ls = ln.f ? n : ln.s;
        u.load(bv.links, bv.off(lp, ls), ln.f != 0);
        sc = bv.lscale(lp, ls);
    }
};
template <int PR, int MU, class BK, class S, class R>
__device__ __forceinline__ void hop_mu(HopLink<PR, MU, BK, S, R> &l, const Lane<BK, R> &ln,
                                       const typename Tile<BK, R>::VR *buf, R (&acc)[24]) {
    typedef Tile<BK, R> T;
    const int at = ln.col0 + ln.template neighbour<PR, MU>();
    Chi<R, R> chi;
#pragma unroll
    for (int q = 0; q < 2 * T::OWN; ++q) {
        const typename T::VR x = buf[q * T::NCOL + at];
#pragma unroll
        for (int k = 0; k < T::CW; ++k) chi.v[q * T::CW + k] = x[k];
    }
    l.u.arrive(ln.f != 0);
    hop_dir<MU>(chi, l.u, ln.c, ln.template weight<PR, MU>() * l.sc, acc);
}

// The in-block hops into the sites of parity PR from the spinors of the other parity in
// buf: out = own chirality of sum_mu [ (1 - gamma) U(x) chi(x + mu) + (1 + gamma) U^+(x - mu) chi(x - mu) ].
// Lanes without the neighbour take their own column's slot with weight zero: the face
// conditions differ between the lanes of a wave, so a branch would save no issue slot.
// l0: the link of direction 0, loaded by the caller. The scheduling barriers keep one
// direction's spinor in registers at a time, and one link or, with AHEAD, two: the next
// direction's is then on its way while this one's is used.
template <int PR, bool AHEAD, class BK, class S, class R>
__device__ __forceinline__ void block_hop_half(HopLink<PR, 0, BK, S, R> &l0, const BlockView<BK, S, R> &bv,
                                               const Lane<BK, R> &ln, const typename Tile<BK, R>::VR *buf,
                                               R (&out)[12]) {
    R acc[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = 0;
    HopLink<PR, 1, BK, S, R> l1;
    HopLink<PR, 2, BK, S, R> l2;
    HopLink<PR, 3, BK, S, R> l3;
    if constexpr (AHEAD) l1.load(bv, ln);
    hop_mu(l0, ln, buf, acc);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!AHEAD) l1.load(bv, ln);
    if constexpr (AHEAD) l2.load(bv, ln);
    hop_mu(l1, ln, buf, acc);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!AHEAD) l2.load(bv, ln);
    if constexpr (AHEAD) l3.load(bv, ln);
    hop_mu(l2, ln, buf, acc);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!AHEAD) l3.load(bv, ln);
    hop_mu(l3, ln, buf, acc);
    fold(acc, out);
}

template <class BK, class R>
__device__ __forceinline__ void put(typename Tile<BK, R>::VR *buf, const Lane<BK, R> &ln, const R (&v)[12]) {
    typedef Tile<BK, R> T;
#pragma unroll
    for (int q = 0; q < T::OWN; ++q) {
        typename T::VR x;
#pragma unroll
        for (int k = 0; k < T::CW; ++k) x[k] = v[q * T::CW + k];
        buf[(ln.f * T::OWN + q) * T::NCOL + ln.col] = x;
    }
}
template <class BK, class R>
__device__ __forceinline__ void get_own(const typename Tile<BK, R>::VR *buf, const Lane<BK, R> &ln, R (&v)[12]) {
    typedef Tile<BK, R> T;
#pragma unroll
    for (int q = 0; q < T::OWN; ++q) {
        const typename T::VR x = buf[(ln.f * T::OWN + q) * T::NCOL + ln.col];
#pragma unroll
        for (int k = 0; k < T::CW; ++k) v[q * T::CW + k] = x[k];
    }
}

// ------------------------------------------------------------------ gather
// The spinor of site (bp, s) for the face hops, without its FP16 scale.
template <class R, class SS>
__device__ __forceinline__ void load_chi(const SS *data, int64_t bp, int s, int Vbh, Chi<R, SS> &chi) {
    if constexpr (Storage<SS>::scaled) {
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            const u32x4 x = *gmem(reinterpret_cast<const u32x4 *>(data) + (bp * 3 + v) * (int64_t)Vbh + s);
#pragma unroll
            for (int k = 0; k < 4; ++k) chi.d[4 * v + k] = x[k];
        }
    } else {
        load_site<R, 24>(data, nullptr, bp, s, Vbh, chi.v);
    }
}
// The block beyond this lane's face in direction MU (forward for f = 0) and the sign of
// the hop into it.
template <int MU> __device__ __forceinline__ int64_t face_block(const Geom &geo, const int (&g)[4], int f, int &sg) {
    int gn[4] = {g[0], g[1], g[2], g[3]};
    sg = 1;
    gn[MU] += f ? -1 : 1;
    if (gn[MU] == geo.G[MU] || gn[MU] < 0) {
        gn[MU] = f ? geo.G[MU] - 1 : 0;
        if (MU == 3 && geo.antiperiodic) sg = -1;
    }
    return block_index(geo.G, gn);
}
// One hop across a face in direction MU into site sr of parity PR, from site sn of block
// nb, up to the reconstruction: uh with its weight w (kappa, the sign, the FP16 scales).
template <int PR, int MU, class BK, class S, class SS, class R, class P>
__device__ __forceinline__ R face_hop(const SapArgs<S, SS, P> &a, int64_t b, int64_t nb, int sr, int sn, int f, R c,
                                      R ksg, const SS *dlt, const float *dlt_sc, R (&uh)[12]) {
    constexpr int Vbh = BK::Vbh;
    constexpr int VS = Vbh * 16, NV = 72 / Vec<S>::W;
    const int64_t nbp = 2 * nb + (1 - PR);
    const int64_t lbp = f ? nbp : 2 * b + PR;  // the link sits at the receiver (forward) or the source
    const int ls = f ? sn : sr;
    View<false> lv;
    lv.set(reinterpret_cast<const char *>(a.links) + lbp * (NV * VS), 0);
    Link<MU, S, VS> u;
    u.load(lv, (unsigned)(ls * 16), f != 0);
    Chi<R, SS> chi;
    load_chi<R, SS>(dlt, nbp, sn, Vbh, chi);
    const R w = ksg * site_scale<R, S>(a.lscale, lbp, ls, Vbh) * site_scale<R, SS>(dlt_sc, nbp, sn, Vbh);
    u.arrive(f != 0);
    hop_half<MU>(chi, u, c, uh);
    return w;
}

// The face hops of one block and parity, shared out over the workgroup: a block has
// Vbh / B_mu receiving sites per face, 224 over the four directions on 8x4^3 and 128 on
// 4^4 blocks, at most one for every lane of either half (forward faces the lower lanes,
// backward the upper). Each direction takes whole waves, so a wave runs one direction's
// code for 32 sites a half; hopping where the sites sit instead would run all four
// directions in every wave with a quarter (an eighth in x) of its lanes (32^3 x 64, FP16,
// 12 rhs: 9070 against 7970 instructions per wave, 3270 against 3097 us on 8x4^3 and 3158
// against 2936 us on 4^4 blocks).
template <class BK> struct Faces {
    static constexpr int ext(int mu) { return BK::ext(mu); }
    static constexpr int count(int mu) { return BK::Vbh / BK::ext(mu); }
    static constexpr int first(int mu) { return mu == 0 ? 0 : first(mu - 1) + count(mu - 1); }
    static constexpr int total = first(3) + count(3);
    // the two directions other than t = MU that number the face's sites beside x (y for MU = 0)
    static constexpr int o1(int mu) { return mu == 0 ? 2 : mu == 1 ? 2 : 1; }
    static constexpr int o2(int mu) { return mu == 3 ? 2 : 3; }
    static_assert(BK::Vbh < 32 || (count(0) % 32 == 0 && count(1) % 32 == 0 && count(2) % 32 == 0 && count(3) % 32 == 0 &&
                                   total <= BK::Vbh), "whole waves per direction");
    // coordinates of receiving site j of parity p on the face l[MU] = at
    template <int MU> static __device__ __forceinline__ void site(int j, int p, int at, int (&l)[4]) {
        constexpr int h = MU == 0 ? BK::by / 2 : BK::bx / 2, e1 = BK::ext(o1(MU));
        const int k = j % h, r = j / h;
        l[MU] = at;
        l[o1(MU)] = r % e1;
        l[o2(MU)] = r / e1;
        constexpr int in = MU == 0 ? 1 : 0;  // the direction that the parity fixes to k
        const int q = (p + at + r % e1 + r / e1) & 1;
        l[in] = 2 * k + q;
    }
    template <int MU> static __device__ __forceinline__ int number(const int (&l)[4]) {
        constexpr int h = MU == 0 ? BK::by / 2 : BK::bx / 2, e1 = BK::ext(o1(MU));
        return (l[MU == 0 ? 1 : 0] >> 1) + h * (l[o1(MU)] + e1 * l[o2(MU)]);
    }
};

// This wave's face hops into the sites of parity PR: w uh of face site q (by first + j) and
// half f into vector column f * total + q of buf.
template <int PR, class BK, class S, class SS, class R, class P>
__device__ __forceinline__ void face_items(const SapArgs<S, SS, P> &a, const Lane<BK, R> &ln, const int (&g)[4], int64_t b,
                                           const SS *dlt, const float *dlt_sc, R kappa,
                                           typename Tile<BK, R>::VR *buf) {
    typedef Tile<BK, R> T;
    typedef Faces<BK> F;
    const int B[4] = {BK::bx, BK::by, BK::bz, BK::bt};
    const int q0 = 32 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    static_for<0, 4>([&](auto m) {
        constexpr int MU = decltype(m)::value;
        if (q0 >= F::first(MU) && q0 < F::first(MU) + F::count(MU)) {  // uniform
            const int q = q0 + (threadIdx.x & 31);
            int lr[4], lb[4], sgf, sgb;
            F::template site<MU>(q - F::first(MU), PR, ln.f ? 0 : B[MU] - 1, lr);
#pragma unroll
            for (int d = 0; d < 4; ++d) lb[d] = lr[d];
            lb[MU] = ln.f ? B[MU] - 1 : 0;
            const int64_t bf = face_block<MU>(a.geo, g, 0, sgf), bb = face_block<MU>(a.geo, g, 1, sgb);
            R uh[12];
            const R w = face_hop<PR, MU, BK>(a, b, ln.f ? bb : bf, local_half_index(B, lr), local_half_index(B, lb), ln.f,
                                             ln.c, kappa * (R)(ln.f ? sgb : sgf), dlt, dlt_sc, uh);
#pragma unroll
            for (int v = 0; v < T::OWN; ++v) {
                typename T::VR x;
#pragma unroll
                for (int k = 0; k < T::CW; ++k) x[k] = w * uh[v * T::CW + k];
                buf[v * (2 * F::total) + ln.f * F::total + q] = x;
            }
        }
    });
}
// rho += the face hops into this thread's site of parity PR, from buf.
template <int PR, class BK, class R>
__device__ __forceinline__ void face_sum(const Lane<BK, R> &ln, const typename Tile<BK, R>::VR *buf, R (&rho)[12]) {
    typedef Tile<BK, R> T;
    typedef Faces<BK> F;
    const int B[4] = {BK::bx, BK::by, BK::bz, BK::bt};
    int l[4];
    local_coords(B, PR, ln.s, l);
    R acc[24], sum[12];
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = 0;
    static_for<0, 4>([&](auto m) {
        constexpr int MU = decltype(m)::value;
        if (!(ln.in[PR] >> MU & 1u)) {
            const int q = F::first(MU) + F::template number<MU>(l);
            R uh[12];
#pragma unroll
            for (int v = 0; v < T::OWN; ++v) {
                const typename T::VR x = buf[v * (2 * F::total) + ln.f * F::total + q];
#pragma unroll
                for (int k = 0; k < T::CW; ++k) uh[v * T::CW + k] = x[k];
            }
            hop_recon<MU>(uh, (R)1, ln.c, acc);
        }
    });
    fold(acc, sum);
#pragma unroll
    for (int k = 0; k < 12; ++k) rho[k] += sum[k];
}
// The same without LDS, every lane hopping into its own site (2^4 blocks, where half of
// the sites lie on any direction's face): rho += the face hops into the site of parity PR.
template <int PR, class BK, class S, class SS, class R, class P>
__device__ __forceinline__ void gather_half(const SapArgs<S, SS, P> &a, const Lane<BK, R> &ln, const int (&g)[4],
                                            int64_t b, const SS *dlt, const float *dlt_sc, R kappa, R (&rho)[12]) {
    const int B[4] = {BK::bx, BK::by, BK::bz, BK::bt};
    int l[4];
    local_coords(B, PR, ln.s, l);
    R acc[24], sum[12];
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = 0;
    static_for<0, 4>([&](auto m) {
        constexpr int MU = decltype(m)::value;
        if (!(ln.in[PR] >> MU & 1u)) {
            int lm[4] = {l[0], l[1], l[2], l[3]}, sg;
            lm[MU] = ln.f ? B[MU] - 1 : 0;
            const int64_t nb = face_block<MU>(a.geo, g, ln.f, sg);
            R uh[12];
            const R w = face_hop<PR, MU, BK>(a, b, nb, ln.s, local_half_index(B, lm), ln.f, ln.c, kappa * (R)sg, dlt,
                                             dlt_sc, uh);
            hop_recon<MU>(uh, w, w * ln.c, acc);
        }
    });
    fold(acc, sum);
#pragma unroll
    for (int k = 0; k < 12; ++k) rho[k] += sum[k];
}

// Sum three values over the threads of one block in a fixed order; every thread gets the
// sums. red: 3 * NW reals, 16-byte aligned.
template <class BK, class R> __device__ __forceinline__ void block_sum3(R &a, R &b, R &c, R *red) {
    typedef Tile<BK, R> T;
    constexpr int GROUP = T::PER > 1 ? BK::Vbh : 64;
    a = lane_sum<GROUP>(a);
    b = lane_sum<GROUP>(b);
    c = lane_sum<GROUP>(c);
    if constexpr (T::NW > 1) {
        constexpr int NW = T::NW;
        const int wv = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) {
            red[wv] = a;
            red[NW + wv] = b;
            red[2 * NW + wv] = c;
        }
        __syncthreads();
        R ra[NW], rb[NW], rc[NW];  // wide loads, all issued before the first add
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            ra[q] = red[q];
            rb[q] = red[NW + q];
            rc[q] = red[2 * NW + q];
        }
        a = ra[0];
        b = rb[0];
        c = rc[0];
#pragma unroll
        for (int q = 1; q < NW; ++q) {
            a += ra[q];
            b += rb[q];
            c += rc[q];
        }
    } else {
        __syncthreads();
    }
}

// Waves per SIMD the kernel is compiled for, and whether a hop loads the next direction's
// link ahead. WIDE chooses between two forms of the FP32 kernel on 8x4^3 blocks, whose
// workgroups have two waves per SIMD: one workgroup per CU with the look-ahead and, in LDS, the
// even sites' clover, or two without them in 128 registers. One workgroup per CU leaves fewer
// blocks to an XCD's L2, which counts when each is used by one or two right-hand sides only.
// Half-sweep times in us, wide / narrow:
//   16^3 x 32, 1 rhs (128 workgroups)    43.1 / 48.9     2 rhs  48.5 / 53.1     3 rhs  80.9 / 72.9
//   16 x 24^2 x 32, 1 rhs (288)         108.7 / 117.7    2 rhs 136.0 / 137.9    4 rhs   218 / 200
//   32^3 x 64, 1 rhs (2048)               621 / 777      2 rhs   756 / 820      3 rhs  1075 / 1048
//   48 x 32^2 x 64, 1 rhs (3072)          931 / 1169     2 rhs  1124 / 1233     4 rhs       / 1967
// (The wide form without the clover in LDS: 42.6, 123.7, 721 and 1075 us with one right-hand side,
// 745 at 32^3 x 64 with two.) On 4^4 blocks (one wave per SIMD and workgroup) the look-ahead
// in 140 registers wins throughout (16^3 x 32, 1 rhs: 39.7 / 44.9; 32^3 x 64, 4 rhs: 1267 / 1320);
// FP16 links need 128 registers either way; FP64 is faster without it (16^3 x 32, 8x4^3: 90.6 against
// 92.7 us with; 32^3 x 64, 4^4, 2 rhs: 1584 against 1621). The forms differ in where operands
// wait, not in any operation, so a right-hand side gets the same bits from both.
template <class BK, class S, class R> constexpr bool sap_two_forms() {
    return sizeof(S) == 4 && sizeof(R) == 4 && BK::Vbh == 256;
}
template <class BK, class S, class R, bool WIDE> constexpr int sap_waves_per_eu() {
    if (BK::Vbh < 32) return sizeof(R) == 8 ? 1 : 2;  // 2^4 blocks: one wave per workgroup
    if (sizeof(R) == 8 || (WIDE && sap_two_forms<BK, S, R>())) return 2;
    return sizeof(S) == 4 && WIDE ? 3 : 4;
}
template <class BK, class S, class R, bool WIDE> constexpr bool sap_look_ahead() {
    return sizeof(R) == 4 && (WIDE || !sap_two_forms<BK, S, R>());
}
// LDS to request beside the kernel's own. A single right-hand side with FP32 links on 4^4 blocks
// re-reads each block's 147 KB from the L2 in every MR step: with three workgroups per CU the 96
// blocks of an XCD miss its 4 MB and the fabric's rate counts. Where there are two workgroups per
// CU or more, they then get a CU each in turn. Half-sweep times in us, three per CU / one:
//   16^2 x 24 x 32 (384 workgroups)  61.0 / 68.7    16^2 x 32^2 (512)   97.2 / 76.8
//   16 x 24^2 x 32 (576)              116 / 102     24^3 x 48 (1296)     265 / 214
//   32^3 x 64 (4096)                  769 / 575     48^3 x 64 (13824)   2633 / 1888
// With two right-hand sides per block it loses (32^3 x 64: 761 / 1010), on FP16 it is not needed.
template <class BK, class S, class R> int sap_extra_lds(int nact, int64_t nwg) {
    constexpr int own = 2 * Tile<BK, R>::BUF * 16;
    if (sizeof(S) == 4 && sizeof(R) == 4 && BK::Vbh == 128 && nact == 1 && nwg >= 512) return 84 * 1024 - own;
    return 0;
}

}  // namespace

template <class BK, class S, class SS, class R, class P, bool WIDE>
__global__ __launch_bounds__((Tile<BK, R>::NT)) __attribute__((amdgpu_waves_per_eu(sap_waves_per_eu<BK, S, R, WIDE>())))
void sap_kernel(SapArgs<S, SS, P> a) {
    constexpr int Vbh = BK::Vbh;
    constexpr bool AHEAD = sap_look_ahead<BK, S, R, WIDE>();
    constexpr bool ODD_LAST = !Storage<S>::scaled;
    typedef Tile<BK, R> T;
    typedef typename T::VR VR;
    __shared__ VR lds[2 * T::BUF];
    __shared__ __align__(16) R red[3 * T::NW];
    constexpr bool XL = WIDE && sap_two_forms<BK, S, R>();
    __shared__ u32x4 xl[XL ? 9 * T::NT : 1];  // each thread's half of its even site's clover
    VR *buf0 = lds, *buf1 = lds + T::BUF;  // even-site vectors r, odd-site vectors

    const Geom &geo = a.geo;
    const Lane<BK, R> ln;
    int slot;
    int64_t kb;
    // The block grid is even in every direction, so the count of blocks of one colour is a
    // multiple of 8 and no workgroup is partly filled.
    if constexpr (T::PER > 1) {  // several (block, rhs) pairs per wave
        const int64_t q = (int64_t)blockIdx.x * T::PER + ln.col / Vbh;
        slot = (int)(q % a.nact);
        kb = q / a.nact;
    } else {
        // Workgroup w runs on XCD w mod 8. Number the (block, rhs) pairs so that the nact
        // right-hand sides of one block follow each other on the same XCD: the block's
        // links and clover are then re-read from that XCD's L2 instead of HBM.
        const int64_t w = blockIdx.x;
        const int64_t kq = w >> 3;
        slot = (int)(kq % a.nact);
        kb = (kq / a.nact) * 8 + (w & 7);
    }
    const int64_t b = colour_block(geo.G, a.colour, kb);
    const int rhs = a.active[slot];
    const R kappa = (R)a.kappa[rhs];
    const int64_t V = geo.V;

    BlockView<BK, S, R> bv;
    constexpr int BB = 2 * Vbh * 72 * (int)sizeof(S);  // bytes of links or clover per block
    bv.links.set(a.links + 2 * b * 72 * Vbh, BB);
    bv.X.set(a.X[rhs] + 2 * b * 72 * Vbh, BB);
    if constexpr (Storage<S>::scaled) {
        bv.lsc.set(a.lscale + 2 * b * Vbh, 2 * Vbh * 4);
        bv.xsc.set(a.Xsc[rhs] + 2 * b * Vbh, 2 * Vbh * 4);
    }

    SS *dlt = a.delta + (int64_t)rhs * V * 24;
    float *dlt_sc = a.delta_sc ? a.delta_sc + (int64_t)rhs * V : nullptr;
    SS *rr = a.rres + (int64_t)rhs * V * 12;
    float *rr_sc = a.rres_sc ? a.rres_sc + (int64_t)rhs * (V / 2) : nullptr;

    // own chirality of: A = even rho, then the MR residual r; B = MR solution x; O = odd
    // rho (ODD_LAST: to the end of the MR steps), then delta_o; H, Q scratch
    R A[12], B[12], O[12], H[12], Q[12];

    if constexpr (XL) {
        CloverHalf<S, BlockView<BK, S, R>::VS> c;
        c.load(bv.X, bv.off(0, ln.s), ln.f);
        c.put(xl, T::NT);
    }

    // ---- 1. block residual rho (even into A, odd into O)
    if (a.mode < 2) {
        const double *eta = a.eta + rhs * a.eta_stride;
        const double f = a.eta_scale ? a.eta_scale[(int64_t)rhs * a.eta_scale_stride] : 1.0;
        double e[12];
        load_half<double, double>(eta, nullptr, 2 * b, ln.s, ln.f, Vbh, e);
#pragma unroll
        for (int k = 0; k < 12; ++k) A[k] = (R)(e[k] * f);
        load_half<double, double>(eta, nullptr, 2 * b + 1, ln.s, ln.f, Vbh, e);
#pragma unroll
        for (int k = 0; k < 12; ++k) O[k] = (R)(e[k] * f);
    } else {
        load_half<R, SS>(rr, rr_sc, b, ln.s, ln.f, Vbh, A);
#pragma unroll
        for (int k = 0; k < 12; ++k) O[k] = 0;
    }
    if (a.mode >= 1) {
        int g[4];
        block_coords(geo.G, b, g);
        if constexpr (T::PER > 1) {
            gather_half<1, BK, S, SS, R>(a, ln, g, b, dlt, dlt_sc, kappa, O);
            gather_half<0, BK, S, SS, R>(a, ln, g, b, dlt, dlt_sc, kappa, A);
        } else {
            face_items<1, BK, S, SS, R>(a, ln, g, b, dlt, dlt_sc, kappa, buf0);
            face_items<0, BK, S, SS, R>(a, ln, g, b, dlt, dlt_sc, kappa, buf1);
            __syncthreads();
            face_sum<1>(ln, buf0, O);
            face_sum<0>(ln, buf1, A);
            __syncthreads();  // buf1 is written below
        }
    }

    // ---- 2. Q = A_o^-1 rho_o, bhat_e = rho_e + kappa H_eo A_o^-1 rho_o
    bv.template clover<1>(ln, O, Q);
    if constexpr (!ODD_LAST) {
#pragma unroll
        for (int k = 0; k < 12; ++k) O[k] = Q[k];
    }
    HopLink<0, 0, BK, S, R> le;
    HopLink<1, 0, BK, S, R> lo;
    le.load(bv, ln);
    put<BK, R>(buf1, ln, Q);
    __syncthreads();
    block_hop_half<0, AHEAD>(le, bv, ln, buf1, H);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        A[k] = fmac(kappa, H[k], A[k]);
        B[k] = 0;
    }

    // ---- 3. MR on Dhat = A_e - kappa^2 H_eo A_o^-1 H_oe
    // Three barriers a step: r in buf0, A_o^-1 H_oe r in buf1, the inner products. A buffer
    // is written again only after a later barrier than its last reads.
    const R k2 = kappa * kappa;
    P *ps = a.psi + rhs * a.psi_stride;
    for (int it = 0; it < a.nmr; ++it) {
        lo.load(bv, ln);
        put<BK, R>(buf0, ln, A);
        __syncthreads();
        block_hop_half<1, AHEAD>(lo, bv, ln, buf0, H);  // odd: H_oe r
        bv.template clover<1>(ln, H, Q);         // odd: Q = A_o^-1 H_oe r
        le.load(bv, ln);
        put<BK, R>(buf1, ln, Q);
        __syncthreads();
        block_hop_half<0, AHEAD>(le, bv, ln, buf1, H);  // even: H_eo Q
        if constexpr (XL) {                      // even: A_e r, then p = A_e r - kappa^2 H
            CloverHalf<S, BlockView<BK, S, R>::VS> c;
            c.get(xl, T::NT);
            clover_half_mul(c, A, Q, (R)1);
        } else {
            bv.template clover<0>(ln, A, Q);
        }
        R pr_re = 0, pr_im = 0, pp = 0;
#pragma unroll
        for (int k = 0; k < 12; ++k) Q[k] = fmac(-k2, H[k], Q[k]);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            pr_re = fmac(Q[2 * k], A[2 * k], pr_re);
            pr_re = fmac(Q[2 * k + 1], A[2 * k + 1], pr_re);
            pr_im = fmac(Q[2 * k], A[2 * k + 1], pr_im);
            pr_im = fmac(-Q[2 * k + 1], A[2 * k], pr_im);
            pp = fmac(Q[2 * k], Q[2 * k], pp);
            pp = fmac(Q[2 * k + 1], Q[2 * k + 1], pp);
        }
        block_sum3<BK, R>(pr_re, pr_im, pp, red);
        // alpha = <p, r> / <p, p> with one division for both parts. Far from a point source <p, p>
        // can be so small that its reciprocal overflows: both products are scaled first then, by a
        // power of two, so that every other quotient keeps its bits.
        R ar = 0, ai = 0;
        if (pp > 0) {
            const R up = pp < 4 * std::numeric_limits<R>::min() ? (R)0x1p64 : (R)1;
            const R inv = (R)1 / (pp * up);
            ar = pr_re * up * inv;
            ai = pr_im * up * inv;
        }
        if constexpr (!ODD_LAST) {
            get_own<BK, R>(buf1, ln, H);  // this step's A_o^-1 H_oe r
            const R kr = kappa * ar, ki = kappa * ai;
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const R tr = H[2 * k], ti = H[2 * k + 1];
                O[2 * k] = fmac(kr, tr, fmac(-ki, ti, O[2 * k]));
                O[2 * k + 1] = fmac(kr, ti, fmac(ki, tr, O[2 * k + 1]));
            }
        }
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const R rr_ = A[2 * k], ri = A[2 * k + 1];
            const R qr = Q[2 * k], qi = Q[2 * k + 1];
            B[2 * k] = fmac(ar, rr_, fmac(-ai, ri, B[2 * k]));
            B[2 * k + 1] = fmac(ar, ri, fmac(ai, rr_, B[2 * k + 1]));
            A[2 * k] = fmac(-ar, qr, fmac(ai, qi, rr_));
            A[2 * k + 1] = fmac(-ar, qi, fmac(-ai, qr, ri));
        }
    }

    // ---- 4. delta_o = A_o^-1 (rho_o + kappa H_oe delta_e)
    if constexpr (ODD_LAST) {
        lo.load(bv, ln);
        put<BK, R>(buf0, ln, B);  // last read before the last two barriers
        __syncthreads();
        block_hop_half<1, AHEAD>(lo, bv, ln, buf0, H);
#pragma unroll
        for (int k = 0; k < 12; ++k) H[k] = fmac(kappa, H[k], O[k]);
        bv.template clover<1>(ln, H, O);
    }

    // ---- 5. outputs: psi += delta (even B, odd O), keep delta and the even-site residual
    R old[12];
    if (a.mode == 2) {
        load_half<R, P>(ps, nullptr, 2 * b, ln.s, ln.f, Vbh, H);
        load_half<R, P>(ps, nullptr, 2 * b + 1, ln.s, ln.f, Vbh, old);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            H[k] += B[k];
            old[k] += O[k];
        }
        store_half<R, P>(ps, nullptr, 2 * b, ln.s, ln.f, Vbh, H);
        store_half<R, P>(ps, nullptr, 2 * b + 1, ln.s, ln.f, Vbh, old);
    } else {
        store_half<R, P>(ps, nullptr, 2 * b, ln.s, ln.f, Vbh, B);
        store_half<R, P>(ps, nullptr, 2 * b + 1, ln.s, ln.f, Vbh, O);
    }
    if (a.write_state) {
        store_half<R, SS>(dlt, dlt_sc, 2 * b, ln.s, ln.f, Vbh, B);
        store_half<R, SS>(dlt, dlt_sc, 2 * b + 1, ln.s, ln.f, Vbh, O);
        store_half<R, SS>(rr, rr_sc, b, ln.s, ln.f, Vbh, A);
    }
}

template <class BK, class S, class SS, class R, class P>
static hipError_t sap_typed(const Geom &geo, const SapArgsHost &h, int colour, int mode, int ws, hipStream_t st) {
    SapArgs<S, SS, P> a;
    a.geo = geo;
    a.links = (const S *)h.links.data;
    a.lscale = h.links.scale;
    a.X = (const S *const *)h.X;
    a.Xsc = h.Xsc;
    a.kappa = h.kappa;
    a.eta = h.eta;
    a.eta_scale = h.eta_scale;
    a.eta_scale_stride = h.eta_scale_stride;
    a.eta_stride = (int64_t)h.eta_stride_rhs * geo.V * 24;
    a.rres = (SS *)h.rres.data;
    a.rres_sc = h.rres.scale;
    a.delta = (SS *)h.delta.data;
    a.delta_sc = h.delta.scale;
    a.psi = (P *)h.psi;
    a.psi_stride = (int64_t)h.psi_stride_rhs * geo.V * 24;
    a.active = h.active;
    a.nact = h.nact;
    a.colour = colour;
    a.mode = mode;
    a.write_state = ws;
    a.nmr = h.nmr;
    typedef Tile<BK, R> T;
    const int64_t nblk = geo.Nd / 2, nwg = nblk * h.nact / T::PER;
    if (nblk % 8 != 0 || nwg > 0x7fffffff) return hipErrorInvalidValue;
    if constexpr (sap_two_forms<BK, S, R>()) {
        if (nwg > 256 && h.nact > 2) {  // more than one workgroup per CU, and blocks shared by three or more
            hipLaunchKernelGGL((sap_kernel<BK, S, SS, R, P, false>), dim3((unsigned)nwg), dim3(T::NT), 0, st, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((sap_kernel<BK, S, SS, R, P, true>), dim3((unsigned)nwg), dim3(T::NT),
                       (sap_extra_lds<BK, S, R>(h.nact, nwg)), st, a);
    return hipGetLastError();
}

// Storage combinations: (links and clover, Schwarz spinors, output psi). FP16 links and
// clover with FP32 spinors is the paper's half-precision mode (Sec. 3.3); FP16 spinors as
// well halve the spinor traffic; FP64 output serves the preconditioned vectors of
// deflated restarts.
template <class BK>
static hipError_t sap_shape(const Geom &geo, const SapArgsHost &h, int colour, int mode, int ws, hipStream_t st) {
    const int lp = h.links.prec, sp = h.rres.prec, pp = h.psi_prec;
    if (h.delta.prec != sp) return hipErrorInvalidValue;
    if (lp == P64 && sp == P64 && pp == P64)
        return sap_typed<BK, double, double, double, double>(geo, h, colour, mode, ws, st);
    if (lp == P32 && sp == P32 && pp == P32) return sap_typed<BK, float, float, float, float>(geo, h, colour, mode, ws, st);
    if (lp == P16 && sp == P16 && pp == P32)
        return sap_typed<BK, half_t, half_t, float, float>(geo, h, colour, mode, ws, st);
    if (lp == P16 && sp == P32 && pp == P32)
        return sap_typed<BK, half_t, float, float, float>(geo, h, colour, mode, ws, st);
    if (lp == P32 && sp == P32 && pp == P64)
        return sap_typed<BK, float, float, float, double>(geo, h, colour, mode, ws, st);
    if (lp == P16 && sp == P16 && pp == P64)
        return sap_typed<BK, half_t, half_t, float, double>(geo, h, colour, mode, ws, st);
    if (lp == P16 && sp == P32 && pp == P64)
        return sap_typed<BK, half_t, float, float, double>(geo, h, colour, mode, ws, st);
    return hipErrorInvalidValue;
}

hipError_t launch_sap_half(const Geom &geo, const SapArgsHost &a, int colour, int mode, int write_state,
                           hipStream_t st) {
    if (a.nact <= 0) return hipSuccess;
    if (geo.B[0] == 2 && geo.B[1] == 2 && geo.B[2] == 2 && geo.B[3] == 2)
        return sap_shape<Blk<2, 2, 2, 2>>(geo, a, colour, mode, write_state, st);
    if (geo.B[0] == 4 && geo.B[1] == 4 && geo.B[2] == 4 && geo.B[3] == 4)
        return sap_shape<Blk<4, 4, 4, 4>>(geo, a, colour, mode, write_state, st);
    if (geo.B[0] == 8 && geo.B[1] == 4 && geo.B[2] == 4 && geo.B[3] == 4)
        return sap_shape<Blk<8, 4, 4, 4>>(geo, a, colour, mode, write_state, st);
    return hipErrorInvalidValue;
}

}  // namespace sapdd
