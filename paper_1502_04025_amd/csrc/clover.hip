// clover.hip - the Sheikholeslami-Wohlert clover term of the Wilson-clover operator
// (Sec. 3.1) and the per-site matrices the Schwarz sweep needs.
//
// T(x) = -c_sw sum_{mu<nu} gamma_mu gamma_nu (x) F_mu,nu(x), F = (Q - Q^+)/8 minus its
// trace / 3, Q = sum of the four plaquettes in the (mu, nu) plane that start and end at
// x, all traversed mu-then-nu. In the chiral basis gamma_mu gamma_nu is block diagonal:
// G_mu G_nu^+ on spins 0-1 and G_mu^+ G_nu on spins 2-3, so T is two 6x6 Hermitian
// blocks (72 reals, packed as described in core.hpp). All of it is FP64 and one-time
// per gauge field (T) or per kappa (the inverse).
#include "blockgeo.hpp"
#include "kernels.hpp"

namespace sapdd {

constexpr int CLOVER_WG = 128;

struct Cx {
    double r, i;
};
__device__ __forceinline__ Cx cmul(Cx a, Cx b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
__device__ __forceinline__ Cx cconj(Cx a) { return {a.r, -a.i}; }

struct M3 {
    Cx e[3][3];
};

__device__ __forceinline__ M3 mmul(const M3 &a, const M3 &b) {
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            Cx s = {0, 0};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const Cx p = cmul(a.e[i][k], b.e[k][j]);
                s.r += p.r;
                s.i += p.i;
            }
            c.e[i][j] = s;
        }
    return c;
}

__device__ __forceinline__ M3 mdag(const M3 &a) {
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) c.e[i][j] = cconj(a.e[j][i]);
    return c;
}

// U_mu at global coordinates x (periodic wrap), from the block-tiled FP64 links.
__device__ M3 link_at(const Geom &geo, const double *links, const int xin[4], int mu) {
    int x[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) x[d] = ((xin[d] % geo.L[d]) + geo.L[d]) % geo.L[d];
    int64_t bp;
    int s;
    site_of(geo, x, bp, s);
    M3 u;
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            u.e[a][b].r = links[real_index<double, 72>(bp, 18 * mu + 2 * (3 * a + b), s, geo.Vbh)];
            u.e[a][b].i = links[real_index<double, 72>(bp, 18 * mu + 2 * (3 * a + b) + 1, s, geo.Vbh)];
        }
    return u;
}

// Chiral-block factor of gamma_mu: G[mu][row][col] (DeGrand-Rossi basis).
__device__ __forceinline__ Cx gmat(int mu, int r, int c) {
    // G_x = [[0, i], [i, 0]], G_y = [[0, -1], [1, 0]], G_z = [[i, 0], [0, -i]], G_t = 1
    switch (mu) {
    case 0: return r != c ? Cx{0, 1} : Cx{0, 0};
    case 1: return r != c ? (r == 0 ? Cx{-1, 0} : Cx{1, 0}) : Cx{0, 0};
    case 2: return r == c ? (r == 0 ? Cx{0, 1} : Cx{0, -1}) : Cx{0, 0};
    default: return r == c ? Cx{1, 0} : Cx{0, 0};
    }
}

// 2x2 spin factor of gamma_mu gamma_nu on chiral block k: G_mu G_nu^+ (k = 0), G_mu^+ G_nu (k = 1).
__device__ __forceinline__ Cx spin_factor(int k, int mu, int nu, int s, int t) {
    Cx acc = {0, 0};
    for (int q = 0; q < 2; ++q) {
        Cx p;
        if (k == 0) p = cmul(gmat(mu, s, q), cconj(gmat(nu, t, q)));
        else p = cmul(cconj(gmat(mu, q, s)), gmat(nu, q, t));
        acc.r += p.r;
        acc.i += p.i;
    }
    return acc;
}

__device__ __forceinline__ int upper_index(int a, int b) { return a * 5 - a * (a - 1) / 2 + (b - a - 1); }

// Pack a Hermitian 6x6 block (only the diagonal's real part and the upper triangle are kept).
__device__ __forceinline__ void pack6(const Cx m[6][6], double *out36) {
    for (int i = 0; i < 6; ++i) out36[i] = m[i][i].r;
    for (int i = 0; i < 6; ++i)
        for (int j = i + 1; j < 6; ++j) {
            out36[6 + 2 * upper_index(i, j)] = m[i][j].r;
            out36[6 + 2 * upper_index(i, j) + 1] = m[i][j].i;
        }
}

__global__ __launch_bounds__(CLOVER_WG) void clover_build_kernel(Geom geo, const double *links, double csw,
                                                                 double *tclov) {
    const int64_t t = (int64_t)blockIdx.x * CLOVER_WG + threadIdx.x;
    if (t >= geo.V) return;
    const int64_t bp = t / geo.Vbh;
    const int s = (int)(t - bp * geo.Vbh);
    int x[4];
    coords_of(geo, bp, s, x);
    Cx T[2][6][6];
    for (int k = 0; k < 2; ++k)
        for (int i = 0; i < 6; ++i)
            for (int j = 0; j < 6; ++j) T[k][i][j] = {0, 0};
    for (int mu = 0; mu < 4; ++mu)
        for (int nu = mu + 1; nu < 4; ++nu) {
            int xm[4], xn[4], xmn[4], xmp[4], xpm[4], xmm[4], xpn[4];
            for (int d = 0; d < 4; ++d) xm[d] = xn[d] = xmn[d] = xmp[d] = xpm[d] = xmm[d] = xpn[d] = x[d];
            xpm[mu] += 1;                   // x + mu
            xpn[nu] += 1;                   // x + nu
            xm[mu] -= 1;                    // x - mu
            xn[nu] -= 1;                    // x - nu
            xmp[mu] -= 1; xmp[nu] += 1;     // x - mu + nu
            xmn[mu] += 1; xmn[nu] -= 1;     // x + mu - nu
            xmm[mu] -= 1; xmm[nu] -= 1;     // x - mu - nu
            const M3 um = link_at(geo, links, x, mu), un = link_at(geo, links, x, nu);
            // x -> x+mu -> x+mu+nu -> x+nu -> x
            M3 q = mmul(mmul(mmul(um, link_at(geo, links, xpm, nu)), mdag(link_at(geo, links, xpn, mu))), mdag(un));
            // x -> x+nu -> x+nu-mu -> x-mu -> x
            const M3 umm = link_at(geo, links, xm, mu);
            M3 l2 = mmul(mmul(mmul(un, mdag(link_at(geo, links, xmp, mu))), mdag(link_at(geo, links, xm, nu))), umm);
            // x -> x-mu -> x-mu-nu -> x-nu -> x
            const M3 unn = link_at(geo, links, xn, nu);
            M3 l3 = mmul(mmul(mmul(mdag(umm), mdag(link_at(geo, links, xmm, nu))), link_at(geo, links, xmm, mu)), unn);
            // x -> x-nu -> x-nu+mu -> x+mu -> x
            M3 l4 = mmul(mmul(mmul(mdag(unn), link_at(geo, links, xn, mu)), link_at(geo, links, xmn, nu)), mdag(um));
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b) {
                    q.e[a][b].r += l2.e[a][b].r + l3.e[a][b].r + l4.e[a][b].r;
                    q.e[a][b].i += l2.e[a][b].i + l3.e[a][b].i + l4.e[a][b].i;
                }
            M3 f;
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b) {
                    f.e[a][b].r = (q.e[a][b].r - q.e[b][a].r) * 0.125;
                    f.e[a][b].i = (q.e[a][b].i + q.e[b][a].i) * 0.125;
                }
            const double tri = (f.e[0][0].i + f.e[1][1].i + f.e[2][2].i) / 3.0;  // trace is imaginary
            for (int a = 0; a < 3; ++a) f.e[a][a].i -= tri;
            for (int k = 0; k < 2; ++k)
                for (int sp = 0; sp < 2; ++sp)
                    for (int tp = 0; tp < 2; ++tp) {
                        const Cx g = spin_factor(k, mu, nu, sp, tp);
                        if (g.r == 0.0 && g.i == 0.0) continue;
                        for (int a = 0; a < 3; ++a)
                            for (int b = 0; b < 3; ++b) {
                                const Cx p = cmul(g, f.e[a][b]);
                                T[k][3 * sp + a][3 * tp + b].r -= csw * p.r;
                                T[k][3 * sp + a][3 * tp + b].i -= csw * p.i;
                            }
                    }
        }
    double packed[72];
    pack6(T[0], packed);
    pack6(T[1], packed + 36);
    store_site<double, 72>(tclov, nullptr, bp, s, geo.Vbh, packed);
}

__global__ __launch_bounds__(CLOVER_WG) void clover_pack_kernel(Geom geo, const double *canon, double *tclov) {
    const int64_t t = (int64_t)blockIdx.x * CLOVER_WG + threadIdx.x;
    if (t >= geo.V) return;
    const int64_t bp = t / geo.Vbh;
    const int s = (int)(t - bp * geo.Vbh);
    int x[4];
    coords_of(geo, bp, s, x);
    const int64_t ci = x[0] + (int64_t)geo.L[0] * (x[1] + (int64_t)geo.L[1] * (x[2] + (int64_t)geo.L[2] * x[3]));
    const double *src = canon + ci * 288;  // 12 x 12 complex
    double packed[72];
    for (int k = 0; k < 2; ++k) {
        Cx m[6][6];
        for (int i = 0; i < 6; ++i)
            for (int j = 0; j < 6; ++j) {
                const int r = 6 * k + i, c = 6 * k + j;
                m[i][j] = {src[2 * (12 * r + c)], src[2 * (12 * r + c) + 1]};
            }
        pack6(m, packed + 36 * k);
    }
    store_site<double, 72>(tclov, nullptr, bp, s, geo.Vbh, packed);
}

__device__ __forceinline__ void exchange(bool take, Cx &x, Cx &y) {
    const Cx u = {take ? y.r : x.r, take ? y.i : x.i}, v = {take ? x.r : y.r, take ? x.i : y.i};
    x = u;
    y = v;
}

// In-place Gauss-Jordan inverse with partial pivoting; returns false if a pivot
// magnitude falls below 1e-12. Every index is a compile-time constant (the rows to
// exchange are found by comparison), so the matrix stays in registers. The product is formed
// before it is subtracted: each update then rounds an entry once, where two chained FMAs
// round it twice (an inverse near 1 is off by 1.35e-16 instead of 1.83e-16).
__device__ __forceinline__ bool invert6(Cx (&a)[6][6]) {
    bool ok = true;
    int piv[6];
    static_for<0, 6>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        int pv = c;
        double best = a[c][c].r * a[c][c].r + a[c][c].i * a[c][c].i;
        static_for<c + 1, 6>([&](auto rr) {
            constexpr int r = decltype(rr)::value;
            const double m = a[r][c].r * a[r][c].r + a[r][c].i * a[r][c].i;
            if (m > best) {
                best = m;
                pv = r;
            }
        });
        piv[c] = pv;
        if (!(best >= 1e-24)) ok = false;
        if (pv != c)
            static_for<c + 1, 6>([&](auto rr) {
                constexpr int r = decltype(rr)::value;
                static_for<0, 6>([&](auto j) { exchange(pv == r, a[c][decltype(j)::value], a[r][decltype(j)::value]); });
            });
        const Cx p = a[c][c];
        const double den = p.r * p.r + p.i * p.i;
        const Cx pinv = {p.r / den, -p.i / den};
        static_for<0, 6>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            a[c][j] = j == c ? pinv : cmul(a[c][j], pinv);
        });
        static_for<0, 6>([&](auto rr) {
            constexpr int r = decltype(rr)::value;
            if constexpr (r != c) {
                const Cx f = a[r][c];
                static_for<0, 6>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    const Cx x = cmul(f, a[c][j]);
                    const Cx b = j == c ? Cx{0.0, 0.0} : a[r][j];
                    a[r][j] = {b.r - x.r, b.i - x.i};
                });
            }
        });
    });
    // undo the row exchanges as column exchanges, last first
    static_for<0, 6>([&](auto cc) {
        constexpr int c = 5 - decltype(cc)::value;
        if (piv[c] != c)
            static_for<c + 1, 6>([&](auto rr) {
                constexpr int r = decltype(rr)::value;
                static_for<0, 6>([&](auto j) { exchange(piv[c] == r, a[decltype(j)::value][c], a[decltype(j)::value][r]); });
            });
    });
    return ok;
}

// The 36 reals of chirality f of a 72-real site; FP16 with the scale of the whole site,
// whose other half lies in lane ^ 32. Every lane of a wave calls this.
template <class S>
__device__ __forceinline__ void store_chirality(S *out, float *scale, int64_t bp, int s, int f, int Vbh,
                                                const double (&v)[36]) {
    if constexpr (Storage<S>::scaled) {
        typedef half_t h4 __attribute__((ext_vector_type(4)));
        float m = 0.f;
#pragma unroll
        for (int k = 0; k < 36; ++k) m = fmaxf(m, fabsf((float)v[k]));
        m = fmaxf(m, __shfl_xor(m, 32, 64));
        const float inv = fp16_site_inv(m);
        if (f == 0) *gmem(scale + bp * Vbh + s) = inv > 0.f ? m : 0.f;
        h4 *p = reinterpret_cast<h4 *>(out);
#pragma unroll
        for (int i = 0; i < 9; ++i) {  // 8-byte piece q of the site: half q & 1 of vector q >> 1
            const int q = 9 * f + i;
            h4 x;
#pragma unroll
            for (int w = 0; w < 4; ++w) x[w] = (half_t)((float)v[4 * i + w] * inv);
            *gmem(p + 2 * ((bp * 9 + (q >> 1)) * (int64_t)Vbh + s) + (q & 1)) = x;
        }
    } else {
        typedef typename Vec<S>::type VT;
        constexpr int W = Vec<S>::W;
        VT *p = reinterpret_cast<VT *>(out);
#pragma unroll
        for (int i = 0; i < 36 / W; ++i) {
            VT x;
#pragma unroll
            for (int w = 0; w < W; ++w) x[w] = (S)v[W * i + w];
            *gmem(p + (bp * (72 / W) + f * (36 / W) + i) * (int64_t)Vbh + s) = x;
        }
    }
}

// Two lanes per site (lane and lane ^ 32), one chirality each: the 6x6 matrix then fits in
// registers, where one thread per site kept both blocks and their inverses in scratch
// memory: a kappa new to the field costs 0.21 instead of 3.97 ms on 24^3 x 48 (FP16), 0.44
// instead of 11.8 ms on 32^3 x 64, which is near the time of reading T and writing X.
template <class S>
__global__ __launch_bounds__(CLOVER_WG) void sap_clover_kernel(Geom geo, const double *tclov, double kappa, S *out,
                                                               float *scale, int *singular) {
    const int lane = threadIdx.x & 63, f = lane >> 5;
    const int64_t t = (int64_t)blockIdx.x * (CLOVER_WG / 2) + 32 * (threadIdx.x >> 6) + (lane & 31);
    const int64_t bp = t / geo.Vbh;
    const int s = (int)(t - bp * geo.Vbh);
    typedef Vec<double>::type v2;
    const v2 *src = reinterpret_cast<const v2 *>(tclov) + (bp * 36 + 18 * f) * (int64_t)geo.Vbh + s;
    double v[36];
#pragma unroll
    for (int i = 0; i < 18; ++i) {
        const v2 x = *gmem(src + (int64_t)i * geo.Vbh);
        v[2 * i] = kappa * x.x;
        v[2 * i + 1] = kappa * x.y;
    }
    if (bp & 1) {
        Cx a[6][6];
        static_for<0, 6>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            a[i][i] = {1.0 + v[i], 0.0};
            static_for<i + 1, 6>([&](auto jj) {
                constexpr int j = decltype(jj)::value, q = 6 + 2 * (i * 5 - i * (i - 1) / 2 + (j - i - 1));
                a[i][j] = {v[q], v[q + 1]};
                a[j][i] = {v[q], -v[q + 1]};
            });
        });
        if (!invert6(a)) *singular = 1;
        // Hermitian by construction; average the two triangles against rounding
        static_for<0, 6>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            v[i] = a[i][i].r - 1.0;
            static_for<i + 1, 6>([&](auto jj) {
                constexpr int j = decltype(jj)::value, q = 6 + 2 * (i * 5 - i * (i - 1) / 2 + (j - i - 1));
                v[q] = 0.5 * (a[i][j].r + a[j][i].r);
                v[q + 1] = 0.5 * (a[i][j].i - a[j][i].i);
            });
        });
    }
    store_chirality(out, scale, bp, s, f, geo.Vbh, v);
}

static dim3 cgrid(const Geom &geo) { return dim3((unsigned)((geo.V + CLOVER_WG - 1) / CLOVER_WG)); }

hipError_t launch_clover_build(const Geom &geo, const double *links, double csw, double *tclov, hipStream_t st) {
    if (geo.V == 0) return hipSuccess;
    hipLaunchKernelGGL(clover_build_kernel, cgrid(geo), dim3(CLOVER_WG), 0, st, geo, links, csw, tclov);
    return hipGetLastError();
}

hipError_t launch_clover_pack(const Geom &geo, const double *canon, double *tclov, hipStream_t st) {
    if (geo.V == 0) return hipSuccess;
    hipLaunchKernelGGL(clover_pack_kernel, cgrid(geo), dim3(CLOVER_WG), 0, st, geo, canon, tclov);
    return hipGetLastError();
}

hipError_t launch_sap_clover(const Geom &geo, const double *tclov, double kappa, Fld out, int *singular,
                             hipStream_t st) {
    if (geo.V == 0) return hipSuccess;
    // the lattice is a multiple of 256 sites: block extents and block grid are even in every direction
    if (geo.V % (CLOVER_WG / 2) != 0) return hipErrorInvalidValue;
    const dim3 g((unsigned)(geo.V / (CLOVER_WG / 2)));
    if (out.prec == P64)
        hipLaunchKernelGGL((sap_clover_kernel<double>), g, dim3(CLOVER_WG), 0, st, geo, tclov, kappa,
                           (double *)out.data, nullptr, singular);
    else if (out.prec == P32)
        hipLaunchKernelGGL((sap_clover_kernel<float>), g, dim3(CLOVER_WG), 0, st, geo, tclov, kappa,
                           (float *)out.data, nullptr, singular);
    else
        hipLaunchKernelGGL((sap_clover_kernel<half_t>), g, dim3(CLOVER_WG), 0, st, geo, tclov, kappa,
                           (half_t *)out.data, out.scale, singular);
    return hipGetLastError();
}

}  // namespace sapdd
