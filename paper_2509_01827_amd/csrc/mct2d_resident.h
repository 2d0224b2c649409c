// Reductions of accepted candidates in the resident steps (device code).
#pragma once

#include <climits>

#include "mct2d_device.h"

namespace mct {
namespace res {

constexpr int kPickWaves = 4;  // wavefronts that take the slots: one slot per lane

// The best accepted candidate of a set and its smallest accepted G.
template <class T>
struct Best {
    T G, Gmin;
    int e, a, k;
};

template <class T>
__device__ __forceinline__ void best_none(Best<T> &b) {
    b.G = T(-1);
    b.Gmin = T(__builtin_inff());
    b.e = INT_MAX;
    b.a = 4;
    b.k = 0;
}

template <class T>
__device__ __forceinline__ void best_merge(Best<T> &b, T G, T Gmin, int e, int a, int k) {
    if (dev::better(G, e, a, b.G, b.e, b.a)) {
        b.G = G;
        b.e = e;
        b.a = a;
        b.k = k;
    }
    if (Gmin < b.Gmin) b.Gmin = Gmin;
}

__device__ __forceinline__ float from_lane(float x, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ __forceinline__ double from_lane(double x, int l) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The value of lane N of this lane's four.
template <int N>
__device__ __forceinline__ float quad_lane(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), N * 0x55, 0xf, 0xf, true));
}
template <int N>
__device__ __forceinline__ double quad_lane(double x) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)b, N * 0x55, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(b >> 32), N * 0x55, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The value of the other lane of this lane's pair.
__device__ __forceinline__ double pair_lane(double x) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)b, 0xB1, 0xf, 0xf, true);  // quad_perm 1 0 3 2
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(b >> 32), 0xB1, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The best of a wavefront, in every lane; has: lanes that hold a candidate
// (few in most steps: they are read one by one, which is shorter than the six
// exchange rounds of a butterfly).
template <class T>
__device__ __forceinline__ void best_wave(Best<T> &b, uint64_t has) {
    if (__popcll(has) <= 4) {
        Best<T> g;
        best_none(g);
        const int ak = (b.a << 2) | b.k;
        while (has) {
            const int l = __builtin_ctzll(has);
            has &= has - 1;
            const int x = __builtin_amdgcn_readlane(ak, l);
            best_merge(g, from_lane(b.G, l), from_lane(b.Gmin, l), __builtin_amdgcn_readlane(b.e, l), x >> 2, x & 3);
        }
        b = g;
        return;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const T G = __shfl_xor(b.G, off, 64), Gm = __shfl_xor(b.Gmin, off, 64);
        const int e = __shfl_xor(b.e, off, 64), ak = __shfl_xor((b.a << 2) | b.k, off, 64);
        best_merge(b, G, Gm, e, ak >> 2, ak & 3);
    }
}

}  // namespace res
}  // namespace mct
