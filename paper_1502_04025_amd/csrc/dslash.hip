// dslash.hip - the Wilson-clover operator M on the whole lattice and its block-diagonal
// part M_B (the domain-internal operator of the Schwarz splitting, Sec. 3.1).
//
// Full operator: one thread per (site, right-hand side); neighbours come from the workgroup's
// tile in LDS (SpinorTile) or from global memory. Workgroups are numbered so that the chunks of one block and right-hand
// side, then the block's right-hand sides, follow each other on the same XCD (workgroup w
// runs on XCD w mod 8): neighbour spinors, links and clover are then re-read from that XCD's
// L2 rather than through the fabric. Blocks are dealt to the XCDs one by one or, for few
// right-hand sides, in eight contiguous ranges (dslash_xcd_ranges).
//
// Block operator: one workgroup per (block, rhs), the block's spinor staged in LDS and
// the hops through the block faces masked off.
#include "blockgeo.hpp"
#include "canon.hpp"
#include "kernels.hpp"

namespace sapdd {

template <class T> struct CF {  // typed const field view
    const T *data;
    const float *scale;
};
template <class T> struct MF {
    T *data;
    float *scale;
};

template <class BK> struct GeoC {  // geometry with compile-time block extents
    static __device__ __forceinline__ void site(const Geom &geo, const int x[4], int64_t &bp, int &s) {
        const int B[4] = {BK::bx, BK::by, BK::bz, BK::bt};
        int g[4], l[4];
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            g[mu] = x[mu] / B[mu];
            l[mu] = x[mu] - g[mu] * B[mu];
        }
        bp = block_index(geo.G, g) * 2 + ((l[0] + l[1] + l[2] + l[3]) & 1);
        s = local_half_index(B, l);
    }
    static __device__ __forceinline__ void coords(const Geom &geo, int64_t bp, int s, int x[4]) {
        const int B[4] = {BK::bx, BK::by, BK::bz, BK::bt};
        int g[4], l[4];
        block_coords(geo.G, bp >> 1, g);
        local_coords(B, (int)(bp & 1), s, l);
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) x[mu] = g[mu] * B[mu] + l[mu];
    }
};

constexpr int DSLASH_WG = 256;

// Lexicographic number of a site inside its block.
template <class BK> __device__ __forceinline__ int canon_slot_of(const int (&x)[4]) {
    return x[0] % BK::bx + BK::bx * (x[1] % BK::by + BK::by * (x[2] % BK::bz + BK::bz * (x[3] % BK::bt)));
}

// Chunks of DSLASH_WG sites that make up one block (with a tile the earlier, then the later half
// of its time slices, else its even, then its odd half): they run next to each other on one
// XCD, so the hops between them are read from that XCD's L2.
template <class BK> constexpr int full_chunks_per_block() {
    return 2 * BK::Vbh > DSLASH_WG ? 2 * BK::Vbh / DSLASH_WG : 1;
}

// How blocks go to the XCDs. In eight contiguous ranges, the next blocks in x (and y) are on
// the same XCD at about the same time and the face spinors come from its L2, as long as few
// right-hand sides lie between them; with many, a block's own right-hand sides fill the L2
// and dealing the blocks out one by one keeps the fabric's traffic even. Ranges gain 7 to 16% for
// one right-hand side and 1 to 10% for two to four; from five on they gain 1% on small lattices
// and lose 2 to 5% on large ones. FP64 operator in us, one by one / ranges:
//   16^3 x 32, 8x4^3, 1 rhs     56.0 / 46.9     4 rhs   123 / 118    8 rhs   234 / 231
//   24^3 x 48, 4^4, 2 rhs        393 / 355      5 rhs   775 / 766
//   32^3 x 64, 8x4^3, 1 rhs      848 / 746      6 rhs  2720 / 2845   12 rhs  5290 / 5400
//   48^3 x 96, 8x4^3, 1 rhs     4250 / 3950     2 rhs  5485 / 5445
//   32^3 x 64, 4^4, 2 rhs       1120 / 1093     12 rhs 5180 / 5401
static bool dslash_xcd_ranges(int nact) { return nact <= 4; }

// On 4^4 and 8x4^3 blocks a workgroup's 256 sites (both parities of a block, or of two of its
// time slices) put their spinors into LDS, in storage precision: each is used there nine
// times, and only the hops out of the tile, a quarter of them, read memory. Read straight
// from global memory they keep the L1 busy (216 reads of 16 bytes a site in FP64); a third
// wave per SIMD gained nothing. Operator alone, global / tile, in us:
//   16^3 x 32, 8x4^3, 1 rhs      FP64 52.2 / 47.2, FP32 25.3 / 24.7
//   24^3 x 48, 4^4, 5 rhs        FP64 966 / 772, FP32 545 / 448
//   32^3 x 64, 8x4^3, 6 rhs      FP64 3640 / 2720, FP32 2150 / 1600
//   32^3 x 64, 4^4, 12 rhs       FP64 6450 / 5170, FP32 3840 / 3150
//   48^3 x 96, 8x4^3, 2 rhs      FP64 6770 / 5500, FP32 3690 / 2990
// On 2^4 blocks half of all hops leave the block: they keep the reads from global memory. So
// do FP16 spinors, not for speed (they would gain as much): behind the tile's branches the
// compiler fuses their site scale into the projection in another order, and the rounding to
// FP16 storage then gives other results. It would take a projection of explicit FMAs in the
// present order.
template <class BK, class TI, bool CIN> struct SpinorTile {
    static constexpr bool ON = BK::Vbh % (DSLASH_WG / 2) == 0 && !Storage<TI>::scaled;
    static constexpr int W = Vec<TI>::W, NV = 24 / W, H = DSLASH_WG / 2;
    static constexpr int PITCH = CIN ? DSLASH_WG + 1 : DSLASH_WG;  // neighbouring lanes write a site's vectors
    static constexpr int BYTES = ON ? PITCH * NV * 16 : 0;
    typedef typename Vec<TI>::type VT;
    VT *lds;
    __device__ __forceinline__ static VT load(const TI *d, int64_t bp, int q, int s) {
        return ld_vec<false>(reinterpret_cast<const VT *>(d) + vec_index<TI, 24>(bp, q, s, BK::Vbh));
    }
    __device__ __forceinline__ void stage(const TI *d, int64_t bp, int s) const {
#pragma unroll
        for (int q = 0; q < NV; ++q) lds[q * PITCH + threadIdx.x] = load(d, bp, q, s);
    }
    // The tile of block b from sites s0 on of both parities, from the operator API's canonical
    // array: whole rows in x by neighbouring lanes, rounded to storage precision as a pass of
    // its own would. That pass moves every spinor once more; without it a call takes, in us,
    //   16^3 x 32, 1 rhs FP64 74 -> 57, FP32 45 -> 41    32^3 x 64, 6 rhs FP64 3524 -> 2705
    //   32^3 x 64, 4^4, 1 rhs FP32 523 -> 479            24 x 8 x 40 x 56, 3 rhs FP32 253 -> 233
    // FP16 sites need their maximum first, and 2^4 blocks have no tile: they keep the pass.
    __device__ __forceinline__ void stage_canon(const Geom &geo, const double *d, int64_t b, int s0) const {
        constexpr int ROW = 12 * BK::bx;
        const int B[4] = {BK::bx, BK::by, BK::bz, BK::bt};
        int g[4];
        block_coords(geo.G, b, g);
        const int t0 = 2 * s0 / (BK::bx * BK::by * BK::bz);
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            const int j = i * DSLASH_WG + threadIdx.x, row = j / ROW, q = j % 12;
            const int l[4] = {j % ROW / 12, row % BK::by, row / BK::by % BK::bz, row / (BK::by * BK::bz) + t0};
            const int64_t idx = g[0] * BK::bx + l[0] +
                                (int64_t)geo.L[0] * (g[1] * BK::by + l[1] +
                                                     (int64_t)geo.L[1] * (g[2] * BK::bz + l[2] + (int64_t)geo.L[2] * (g[3] * BK::bt + l[3])));
            const dv2g x = ((const SAPDD_GLOBAL dv2g *)d)[idx * 12 + q];
            const int n = ((l[0] + l[1] + l[2] + l[3]) & 1) * H + local_half_index(B, l) - s0;
            TI *to = (TI *)(lds + 2 * q / W * PITCH + n) + 2 * q % W;
            to[0] = (TI)x.x, to[1] = (TI)x.y;
        }
    }
    // The spinor in slot n of the tile, or of site (bp, s), canonical index idx, if it lies outside.
    template <class R>
    __device__ __forceinline__ void get(bool inside, int n, const TI *d, int64_t bp, int s, const double *canon,
                                        int64_t idx, R (&out)[24]) const {
        VT x[NV];
        asm volatile("" : "+v"(n) : : "memory");  // the read stays behind the previous hop
        if (inside) {
#pragma unroll
            for (int q = 0; q < NV; ++q) x[q] = lds[q * PITCH + n];
        } else {
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                if constexpr (CIN) {
#pragma unroll
                    for (int k = 0; k < W; k += 2) {
                        const dv2g e = ((const SAPDD_GLOBAL dv2g *)canon)[idx * 12 + (q * W + k) / 2];
                        x[q][k] = (TI)e.x, x[q][k + 1] = (TI)e.y;
                    }
                } else {
                    x[q] = load(d, bp, q, s);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < NV; ++q)
#pragma unroll
            for (int w = 0; w < W; ++w) out[q * W + w] = (R)x[q][w];
    }
};

// Keeps a hop's arithmetic where it is written: the compiler otherwise moves that of all eight
// hops behind the last of the tile's branches, and spills their spinors and links.
template <class R> __device__ __forceinline__ void pin(R (&v)[24]) {
#pragma unroll
    for (int k = 0; k < 24; ++k) asm volatile("" : "+v"(v[k]));
}

template <class BK, class S, class TI, class TO, class R, bool CANON, bool CIN = false>
__global__ __launch_bounds__(DSLASH_WG) void dslash_full_kernel(Geom geo, CF<S> links, CF<S> tclov, R kappa,
                                                                 CF<TI> in, MF<TO> out, double *canon,
                                                                 const double *sub,
                                                                 double *part, const int *active, int nact,
                                                                 int nchunk, int ranges, int ins_, int outs_,
                                                                 int subs_, const double *kap) {
    constexpr int Vbh = BK::Vbh;
    constexpr int G = full_chunks_per_block<BK>();
    const int w = blockIdx.x;
    const int xcd = w & 7;
    const int k = w >> 3;
    const int slot = k / G % nact;
    const int q = k / G / nact;  // group of G chunks within the XCD's share
    const int share = (nchunk / G + 7) / 8;
    const int chunk = (ranges ? xcd * share + q : q * 8 + xcd) * G + k % G;
    const int rhs = active ? active[slot] : slot;
    const int64_t site = (int64_t)chunk * DSLASH_WG + threadIdx.x;
    const bool valid = chunk < nchunk && site < geo.V;
    typedef SpinorTile<BK, TI, CIN> ST;
    constexpr int CB = CANON ? DSLASH_WG * (int)sizeof(CanonSlot<TO>) : 16;
    __shared__ __align__(16) char smem[ST::BYTES > CB ? ST::BYTES : CB];
    CanonSlot<TO> *lds = reinterpret_cast<CanonSlot<TO> *>(smem);
    const ST tile{reinterpret_cast<typename ST::VT *>(smem)};
    double nrm = 0.0;
    // the workgroup's sites: with a tile, sites s0 .. s0 + 127 of both parities of a block
    int64_t bp;
    int s, s0 = 0;
    if constexpr (ST::ON) {
        s0 = chunk % G * ST::H;
        bp = 2 * (int64_t)(chunk / G) + threadIdx.x / ST::H;
        s = s0 + threadIdx.x % ST::H;
    } else {
        bp = site / Vbh;
        s = (int)(site - bp * Vbh);
    }
    const TI *ind = in.data + (int64_t)rhs * ins_ * geo.V * 24;
    const double *cin = CIN ? (const double *)in.data + (int64_t)rhs * geo.V * 24 : nullptr;
    const float *ins = in.scale ? in.scale + (int64_t)rhs * ins_ * geo.V : nullptr;
    if constexpr (ST::ON) {  // a chunk is whole or past the lattice
        if (valid) {
            if constexpr (CIN) tile.stage_canon(geo, cin, bp >> 1, s0);
            else tile.stage(ind, bp, s);
        }
        __syncthreads();
    }
    int x[4] = {0, 0, 0, 0};
    if (valid) {
        GeoC<BK>::coords(geo, bp, s, x);
        if (kap) kappa = (R)kap[rhs];
        const int64_t ooff = (int64_t)rhs * outs_ * geo.V * 24;
        // the spinor of site (nbp, ns)
        auto spinor = [&](int64_t nbp, int ns, const int (&y)[4], R (&chi)[24]) {
            if constexpr (ST::ON) {
                const bool inside = (nbp >> 1) == (bp >> 1) && (unsigned)(ns - s0) < (unsigned)ST::H;
                tile.get(inside, (int)(nbp & 1) * ST::H + ns - s0, ind, nbp, ns, cin,
                         y[0] + (int64_t)geo.L[0] * (y[1] + (int64_t)geo.L[1] * (y[2] + (int64_t)geo.L[2] * y[3])), chi);
            } else {
                load_site<R, 24>(ind, ins, nbp, ns, Vbh, chi);
            }
        };
        R acc[24];
#pragma unroll
        for (int c = 0; c < 24; ++c) acc[c] = 0;
        static_for<0, 4>([&](auto m) {
            constexpr int MU = decltype(m)::value;
            const int L = geo.L[MU];
            {  // forward hop: (1 - gamma) U_mu(x) psi(x + mu)
                int y[4] = {x[0], x[1], x[2], x[3]};
                R sg = 1;
                if (++y[MU] == L) {
                    y[MU] = 0;
                    if (MU == 3 && geo.antiperiodic) sg = -1;
                }
                int64_t nbp;
                int ns;
                GeoC<BK>::site(geo, y, nbp, ns);
                R chi[24], h[12], u[18], uh[12];
                spinor(nbp, ns, y, chi);
                project<MU, -1>(chi, h);
                load_reals<R, 72, 18 * MU, 18, S, true>(links.data, nullptr, bp, s, Vbh, u);
                su3_mul(u, h, uh);
                accum_recon<MU, -1>(acc, uh, sg * site_scale<R, S>(links.scale, bp, s, Vbh));
                if constexpr (ST::ON) pin(acc);
            }
            {  // backward hop: (1 + gamma) U_mu(x - mu)^+ psi(x - mu)
                int y[4] = {x[0], x[1], x[2], x[3]};
                R sg = 1;
                if (--y[MU] < 0) {
                    y[MU] = L - 1;
                    if (MU == 3 && geo.antiperiodic) sg = -1;
                }
                int64_t nbp;
                int ns;
                GeoC<BK>::site(geo, y, nbp, ns);
                R chi[24], h[12], u[18], uh[12];
                spinor(nbp, ns, y, chi);
                project<MU, +1>(chi, h);
                load_reals<R, 72, 18 * MU, 18, S, true>(links.data, nullptr, nbp, ns, Vbh, u);
                su3_dag_mul(u, h, uh);
                accum_recon<MU, +1>(acc, uh, sg * site_scale<R, S>(links.scale, nbp, ns, Vbh));
                if constexpr (ST::ON) pin(acc);
            }
        });
        R psi[24], res[24];
        spinor(bp, s, x, psi);
        CloverRegs<S, R> cl;
        cl.load(tclov.data, tclov.scale, bp, s, Vbh);
        clover_mul(cl, psi, res, kappa);  // (1 + kappa T) psi
#pragma unroll
        for (int c = 0; c < 24; ++c) res[c] = fmac(-kappa, acc[c], res[c]);
        if (sub) {
            double sb[24];
            load_site<double, 24>(sub + (int64_t)rhs * subs_ * geo.V * 24, nullptr, bp, s, Vbh, sb);
#pragma unroll
            for (int c = 0; c < 24; ++c) res[c] = (R)sb[c] - res[c];
        }
        if constexpr (CANON) {
            // The operator API's result goes to the caller's array from here: against a pass
            // of its own the calls were 2 to 15% faster, with spinors still read from global
            // memory and packed first (32^3 x 64, 8x4^3, 4 rhs, FP64 3568 -> 3079 us, FP32 2078 ->
            // 1903 us, FP16 1524 -> 1493 us; 16^3 x 32, 1 rhs, FP64 80.7 -> 73.5 us).
            // slots in canonical order where the chunk holds both parities of its blocks
            int n = threadIdx.x;
            if constexpr (ST::ON) n = canon_slot_of<BK>(x) - 2 * s0;
            else if constexpr (2 * Vbh <= DSLASH_WG)
                n = canon_slot_of<BK>(x) + (int)(bp / 2 % (DSLASH_WG / (2 * Vbh))) * 2 * Vbh;
            if constexpr (ST::ON) __syncthreads();  // the tile has been read
            lds[n].set(res);
            lds[n].idx = x[0] + (int64_t)geo.L[0] * (x[1] + (int64_t)geo.L[1] * (x[2] + (int64_t)geo.L[2] * x[3]));
        } else {
            store_site<R, 24>(out.data + ooff, out.scale ? out.scale + (int64_t)rhs * outs_ * geo.V : nullptr, bp, s,
                              Vbh, res);
        }
        if (part) {
#pragma unroll
            for (int c = 0; c < 24; ++c) nrm += (double)res[c] * (double)res[c];
        }
    }
    if constexpr (CANON) {  // a chunk is whole or past the lattice
        __syncthreads();
        if (valid) canon_put<DSLASH_WG>(canon + (int64_t)rhs * geo.V * 24, lds);
    }
    if (part) {  // fixed-order workgroup reduction of |out|^2
        __shared__ double red[DSLASH_WG / 64];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = nrm;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0;
            for (int q = 0; q < DSLASH_WG / 64; ++q) t += red[q];
            const int nwg = (nchunk + 7) / 8 * 8;
            if (chunk < nwg) part[(int64_t)slot * nwg + chunk] = t;
        }
    }
}

int dslash_full_partials(const Geom &geo) {
    const int nchunk = (int)((geo.V + DSLASH_WG - 1) / DSLASH_WG);
    return (nchunk + 7) / 8 * 8;
}

template <class BK, class S, class TI, class TO, class R, bool CANON, bool CIN = false>
static hipError_t full_typed(const Geom &geo, Fld links, Fld tclov, double kappa, const DslashIO &io,
                             hipStream_t st) {
    const int nchunk = (int)((geo.V + DSLASH_WG - 1) / DSLASH_WG);
    constexpr int G = full_chunks_per_block<BK>();
    // groups of G chunks dealt round-robin to the 8 XCDs; every chunk index below
    // dslash_full_partials gets a workgroup (those past the lattice write zero partials)
    const int ng8 = ((nchunk + G - 1) / G + 7) / 8 * 8;
    const int64_t nwg = (int64_t)ng8 * G * io.nact;
    if (nwg == 0) return hipSuccess;
    // the block grid is even in every direction: the lattice is whole chunks
    if (nwg > 0x7fffffff || geo.V % DSLASH_WG != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL((dslash_full_kernel<BK, S, TI, TO, R, CANON, CIN>), dim3((unsigned)nwg), dim3(DSLASH_WG), 0, st, geo,
                       CF<S>{(const S *)links.data, links.scale}, CF<S>{(const S *)tclov.data, tclov.scale},
                       (R)kappa, CF<TI>{(const TI *)io.in.data, io.in.scale}, MF<TO>{(TO *)io.out.data, io.out.scale},
                       io.canon, io.sub, io.part, io.active, io.nact, nchunk, dslash_xcd_ranges(io.nact) ? 1 : 0, io.in_stride, io.out_stride, io.sub_stride,
                       io.kappa);
    return hipGetLastError();
}

template <class BK>
static hipError_t full_shape(const Geom &geo, Fld links, Fld tclov, double kappa, const DslashIO &io,
                             hipStream_t st) {
    // supported combinations: FP64 links with FP64 or FP32 input and block-tiled FP64 output
    // (the outer solver), and uniform FP64 / FP32 / FP16 storage with canonical output (the
    // operator API).
    if (io.canon) {
        if (io.in.prec != links.prec || io.sub || io.part) return hipErrorInvalidValue;
        if (io.canon_in) {
            if constexpr (SpinorTile<BK, float, true>::ON) {
                if (links.prec == P64) return full_typed<BK, double, double, double, double, true, true>(geo, links, tclov, kappa, io, st);
                if (links.prec == P32) return full_typed<BK, float, float, float, float, true, true>(geo, links, tclov, kappa, io, st);
            }
            return hipErrorInvalidValue;
        }
        if (links.prec == P64) return full_typed<BK, double, double, double, double, true>(geo, links, tclov, kappa, io, st);
        if (links.prec == P32) return full_typed<BK, float, float, float, float, true>(geo, links, tclov, kappa, io, st);
        return full_typed<BK, half_t, half_t, half_t, float, true>(geo, links, tclov, kappa, io, st);
    }
    if (links.prec != P64 || io.out.prec != P64) return hipErrorInvalidValue;
    if (io.in.prec == P64) return full_typed<BK, double, double, double, double, false>(geo, links, tclov, kappa, io, st);
    if (io.in.prec == P32) return full_typed<BK, double, float, double, double, false>(geo, links, tclov, kappa, io, st);
    return hipErrorInvalidValue;
}

// Call F<Blk<...>>(args...) for the supported block shapes.
template <template <class> class F, class... A>
static hipError_t by_shape(const Geom &geo, A &&...args) {
    if (geo.B[0] == 2 && geo.B[1] == 2 && geo.B[2] == 2 && geo.B[3] == 2) return F<Blk<2, 2, 2, 2>>::run(args...);
    if (geo.B[0] == 4 && geo.B[1] == 4 && geo.B[2] == 4 && geo.B[3] == 4) return F<Blk<4, 4, 4, 4>>::run(args...);
    if (geo.B[0] == 8 && geo.B[1] == 4 && geo.B[2] == 4 && geo.B[3] == 4) return F<Blk<8, 4, 4, 4>>::run(args...);
    return hipErrorInvalidValue;
}

template <class BK> struct FullRun {
    static hipError_t run(const Geom &geo, Fld links, Fld tclov, double kappa, const DslashIO &io, hipStream_t st) {
        return full_shape<BK>(geo, links, tclov, kappa, io, st);
    }
};

bool dslash_reads_canon(const Geom &geo, int prec) { return prec != P16 && geo.Vbh % (DSLASH_WG / 2) == 0; }

hipError_t launch_dslash_full(const Geom &geo, Fld links, Fld tclov, double kappa, const DslashIO &io,
                              hipStream_t st) {
    return by_shape<FullRun>(geo, geo, links, tclov, kappa, io, st);
}

// ---------------------------------------------------------------- block operator
// From the canonical array to the canonical array: every site is read and written by one
// thread only, so the conversion to the storage precision and back happens in registers and
// needs no pass of its own. Bound by HBM: 384 bytes of spinor a site beside the links and
// clover. 32^3 x 64, 4^4 blocks, one call with its conversions, against separate passes before
// and after: FP32 545 -> 362 us, FP16 412 -> 270 us, FP64 949 -> 704 us; the kernel alone moves
// 5.3 TB/s in FP32 and 5.1 TB/s in FP16.
template <class BK, class S, class R, bool ONE>
__global__ __launch_bounds__(BK::NT) void dslash_block_kernel(Geom geo, CF<S> links, CF<S> tclov, R kappa,
                                                               const double *in, double *out, int nrhs) {
    constexpr int Vbh = BK::Vbh;
    // one area for the hops (one LDS buffer: this memory-bound kernel gains more from
    // occupancy than from the barrier a second buffer would save) and then for the result
    __shared__ __align__(16) char lds[BlockLds<BK, S, R>::bytes];
    const SiteInfo si = site_info<BK>(threadIdx.x);
    int rhs;
    const int64_t b = block_and_rhs(ONE ? 1 : nrhs, rhs);
    const int64_t bp = 2 * b + si.p;
    const int64_t idx = canon_index_bk<BK>(geo, b, si.l);
    // links held in registers between the two half-hops (re-reading them from L1/L2 to
    // reach 4 waves per SIMD measured slower: 3.65 vs 4.53 TB/s in FP16)
    // With one right-hand side every byte of links and clover is used by one workgroup only:
    // non-temporal hints (measured 4.71 -> 5.52 TB/s in FP32, 4.49 -> 4.80 TB/s in FP16 on 32^3x64). Issuing
    // the clover loads before the hops instead of after measured slower.
    constexpr bool NT = ONE;
    SiteLinks<S, R> U;
    U.template init<NT>(links.data, links.scale, bp, si.s, Vbh);
    R psi[24], hop[24];
    block_load<S>(in + (int64_t)rhs * geo.V * 24, idx, psi);
    block_hop<BK>(0, si, U, psi, hop, (R *)lds);  // odd sites receive
    block_hop<BK>(1, si, U, psi, hop, (R *)lds);  // even sites receive
    R res[24];
    CloverRegs<S, R> cl;
    cl.template load<NT>(tclov.data, tclov.scale, bp, si.s, Vbh);
    clover_mul(cl, psi, res, kappa);
#pragma unroll
    for (int c = 0; c < 24; ++c) res[c] = fmac(-kappa, hop[c], res[c]);
    block_store<BK, S>(out + (int64_t)rhs * geo.V * 24, idx, si.l, res, lds);
}

template <class BK, class S, class R>
static hipError_t block_typed(const Geom &geo, Fld links, Fld tclov, double kappa, const double *in, double *out,
                              int nrhs, hipStream_t st) {
    const int64_t nwg = geo.Nd * nrhs;
    if (geo.Nd % 8 != 0 || nwg > 0x7fffffff) return hipErrorInvalidValue;
    const CF<S> l{(const S *)links.data, links.scale}, t{(const S *)tclov.data, tclov.scale};
    if (nrhs == 1)
        hipLaunchKernelGGL((dslash_block_kernel<BK, S, R, true>), dim3((unsigned)nwg), dim3(BK::NT), 0, st, geo, l, t, (R)kappa, in, out, nrhs);
    else
        hipLaunchKernelGGL((dslash_block_kernel<BK, S, R, false>), dim3((unsigned)nwg), dim3(BK::NT), 0, st, geo, l, t, (R)kappa, in, out, nrhs);
    return hipGetLastError();
}
template <class BK>
static hipError_t block_shape(const Geom &geo, Fld links, Fld tclov, double kappa, const double *in, double *out,
                              int nrhs, hipStream_t st) {
    if (tclov.prec != links.prec) return hipErrorInvalidValue;
    if (links.prec == P64) return block_typed<BK, double, double>(geo, links, tclov, kappa, in, out, nrhs, st);
    if (links.prec == P32) return block_typed<BK, float, float>(geo, links, tclov, kappa, in, out, nrhs, st);
    return block_typed<BK, half_t, float>(geo, links, tclov, kappa, in, out, nrhs, st);
}

template <class BK> struct BlockRun {
    static hipError_t run(const Geom &geo, Fld links, Fld tclov, double kappa, const double *in, double *out,
                          int nrhs, hipStream_t st) {
        return block_shape<BK>(geo, links, tclov, kappa, in, out, nrhs, st);
    }
};

hipError_t launch_dslash_block(const Geom &geo, Fld links, Fld tclov, double kappa, const double *in, double *out,
                               int nrhs, hipStream_t st) {
    if (nrhs <= 0 || geo.Nd == 0) return hipSuccess;
    return by_shape<BlockRun>(geo, geo, links, tclov, kappa, in, out, nrhs, st);
}

}  // namespace sapdd
