// canon.hpp - spinors between a workgroup's threads (one site each) and the canonical
// site-major FP64 array.
//
// A canonical site is 24 doubles, 192 contiguous bytes. Stores by one thread per site would
// touch 64 cache lines with every 16-byte store of a wave, so a workgroup turns its sites in
// LDS and stores 16-byte units with neighbouring lanes on neighbouring addresses. The sites
// wait in LDS in storage precision and become doubles on the way out. Loads by one thread
// per site find the rest of their lines in the cache and stay as they are.
#pragma once
#include "core.hpp"

namespace sapdd {

typedef double dv2g __attribute__((ext_vector_type(2), aligned(8)));  // in the caller's array of doubles

// Canonical site index (x fastest) of block-tiled site (bp, s).
__device__ __forceinline__ int64_t canon_index(const Geom &geo, int64_t bp, int s) {
    int x[4];
    coords_of(geo, bp, s, x);
    return x[0] + (int64_t)geo.L[0] * (x[1] + (int64_t)geo.L[1] * (x[2] + (int64_t)geo.L[2] * x[3]));
}

// The 24 doubles of canonical site idx.
__device__ __forceinline__ void canon_load(const double *canon, int64_t idx, double (&v)[24]) {
    const SAPDD_GLOBAL dv2g *src = (const SAPDD_GLOBAL dv2g *)canon + idx * 12;
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        const dv2g x = src[c];
        v[2 * c] = x.x;
        v[2 * c + 1] = x.y;
    }
}

// The FP16 values and scale that store_site gives a site.
template <class T> __device__ __forceinline__ float fp16_site(const T (&in)[24], half_t (&h)[24]) {
    float m = 0.f;
#pragma unroll
    for (int k = 0; k < 24; ++k) m = fmaxf(m, fabsf((float)in[k]));
    const float inv = fp16_site_inv(m);
#pragma unroll
    for (int k = 0; k < 24; ++k) {
        float t = (float)in[k] * inv;
        asm("" : "+v"(t));  // rounded to FP32 first, as store_site's vectors are (no mixed FMA)
        h[k] = (half_t)t;
    }
    return inv > 0.f ? m : 0.f;
}
// A site in storage precision S, as arithmetic type R: what store_site and load_site would
// leave of the 24 values.
template <class S, class R> __device__ __forceinline__ void round_site(const double (&in)[24], R (&out)[24]) {
    if constexpr (Storage<S>::scaled) {
        half_t h[24];
        const R sc = (R)fp16_site(in, h);
#pragma unroll
        for (int k = 0; k < 24; ++k) out[k] = (R)(float)h[k] * sc;
    } else {
#pragma unroll
        for (int k = 0; k < 24; ++k) out[k] = (R)(S)in[k];
    }
}

// A site's slot in LDS: 12 complex components in storage precision S, its canonical index
// and, for FP16, its scale. The FP64 and FP32 strides (208 and 104 bytes) spread neighbouring
// slots over the banks; the FP16 slot has 64 bytes, so that every fourth starts on the same bank.
template <class S> struct CanonSlot;
template <> struct CanonSlot<double> {
    typedef double v2 __attribute__((ext_vector_type(2)));
    v2 c[12];
    int64_t idx, pad;
    __device__ __forceinline__ void set(const double (&in)[24]) {
#pragma unroll
        for (int k = 0; k < 12; ++k) c[k] = v2{in[2 * k], in[2 * k + 1]};
    }
    __device__ __forceinline__ dv2g at(int k) const { return (dv2g)c[k]; }
};
template <> struct CanonSlot<float> {
    typedef float v2 __attribute__((ext_vector_type(2)));
    v2 c[12];
    int64_t idx;
    __device__ __forceinline__ void set(const float (&in)[24]) {
#pragma unroll
        for (int k = 0; k < 12; ++k) c[k] = v2{in[2 * k], in[2 * k + 1]};
    }
    __device__ __forceinline__ dv2g at(int k) const { return dv2g{(double)c[k].x, (double)c[k].y}; }
};
template <> struct CanonSlot<half_t> {
    typedef half_t v2 __attribute__((ext_vector_type(2)));
    int64_t idx;
    v2 c[12];
    float scale, pad;
    __device__ __forceinline__ void set(const float (&in)[24]) {
        half_t h[24];
        scale = fp16_site(in, h);
#pragma unroll
        for (int k = 0; k < 12; ++k) c[k] = v2{h[2 * k], h[2 * k + 1]};
    }
    __device__ __forceinline__ dv2g at(int k) const {
        const double sc = scale;
        return dv2g{(double)(float)c[k].x * sc, (double)(float)c[k].y * sc};
    }
};
// All NT sites from LDS to the canonical field (after a barrier).
template <int NT, class S> __device__ __forceinline__ void canon_put(double *canon, const CanonSlot<S> *lds) {
    SAPDD_GLOBAL dv2g *dst = (SAPDD_GLOBAL dv2g *)canon;
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        const int u = threadIdx.x + NT * j, n = u / 12, c = u - 12 * n;
        __builtin_nontemporal_store(lds[n].at(c), dst + lds[n].idx * 12 + c);
    }
}

}  // namespace sapdd
