// lanes.hpp - values exchanged between the lanes of a wave, register to register.
#pragma once
#include <hip/hip_runtime.h>

namespace sapdd {

// Other lane's register contents: the DPP control moves inside rows of 16 lanes.
template <int CTRL> __device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ __forceinline__ double dpp_move(double v) {
    int2 x = __builtin_bit_cast(int2, v);
    x.x = __builtin_amdgcn_update_dpp(0, x.x, CTRL, 0xF, 0xF, false);
    x.y = __builtin_amdgcn_update_dpp(0, x.y, CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, x);
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    int2 x = __builtin_bit_cast(int2, v);
    x.x = __builtin_amdgcn_readlane(x.x, lane);
    x.y = __builtin_amdgcn_readlane(x.y, lane);
    return __builtin_bit_cast(double, x);
}

// (a, b) -> a = { a of lanes 0-31, b of lanes 0-31 }, b = { a of lanes 32-63, b of lanes
// 32-63 }: the upper half of a and the lower half of b change places.
__device__ __forceinline__ void swap32(unsigned &a, unsigned &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void swap32(float &a, float &b) {
    unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
    swap32(x, y);
    a = __builtin_bit_cast(float, x);
    b = __builtin_bit_cast(float, y);
}
__device__ __forceinline__ void swap32(double &a, double &b) {
    uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    swap32(x.x, y.x);
    swap32(x.y, y.y);
    a = __builtin_bit_cast(double, x);
    b = __builtin_bit_cast(double, y);
}

// The same between neighbouring rows of 16 lanes: row 1 of a with row 0 of b, row 3 of a with
// row 2 of b.
__device__ __forceinline__ void swap16(double &a, double &b) {
    uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    const auto r = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
    const auto t = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    a = __builtin_bit_cast(double, make_uint2(r[0], t[0]));
    b = __builtin_bit_cast(double, make_uint2(r[1], t[1]));
}

// Sums of N values (a power of two) over the lanes of each half of a wave (N = 1..16) or over
// the whole wave (N = 2..32), in a fixed order that does not depend on N: every step halves the
// values a lane carries and doubles the lanes behind each, so that N values cost about N
// adds instead of 5 or 6 N. Afterwards v[0] of lane l is the total of value
// half_scatter_index<N>(l) (of l's half) or wave_scatter_index<N>(l); the 32 / N or 64 / N
// lanes that differ in the low bits alone hold the same.
template <int CTRL, int H, class V> __device__ __forceinline__ void scatter_dpp(V &v, bool upper) {
    if constexpr (H == 0) {  // one value left: every lane adds its partner's
        v[0] += dpp_move<CTRL>(v[0]);
    } else {
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const double keep = upper ? v[k + H] : v[k], give = upper ? v[k] : v[k + H];
            v[k] = keep + dpp_move<CTRL>(give);
        }
    }
}
template <int N, class V> __device__ __forceinline__ void half_scatter(V &v) {
    const int l = threadIdx.x & 63;
    if constexpr (N == 1) {
        double a = v[0], b = v[0];
        swap16(a, b);
        v[0] = a + b;
    }
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
        swap16(v[k], v[k + N / 2]);
        v[k] += v[k + N / 2];
    }
    // the partner lanes: rotation by 8 in a row, mirror in 8 lanes, lane ^ 2, lane ^ 1
    scatter_dpp<0x128, N / 4>(v, l & 8);
    scatter_dpp<0x141, N / 8>(v, l & 4);
    scatter_dpp<0x4E, N / 16>(v, l & 2);
    scatter_dpp<0xB1, 0>(v, false);
}
template <int N> __device__ __forceinline__ int half_scatter_index(int l) {
    return (l & 31) / (32 / N);  // the upper bits of l, the highest first
}
template <int N, class V> __device__ __forceinline__ void wave_scatter(V &v) {
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
        swap32(v[k], v[k + N / 2]);
        v[k] += v[k + N / 2];
    }
    half_scatter<N / 2>(v);
}
template <int N> __device__ __forceinline__ int wave_scatter_index(int l) { return (l & 63) / (64 / N); }

}  // namespace sapdd
