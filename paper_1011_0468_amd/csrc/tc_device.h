// Device-side helpers for gfx950 (wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tc {

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// bits of lanes strictly below this lane
__device__ __forceinline__ uint64_t lanes_below() {
    const int l = __lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

__device__ __forceinline__ uint64_t ballot64(int pred) { return __ballot(pred); }

// inclusive wave scan (sum)
template <typename T>
__device__ __forceinline__ T wave_inclusive_sum(T v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        T o = __shfl_up(v, d, 64);
        if (__lane_id() >= d) v += o;
    }
    return v;
}

// The same for 32-bit integers with DPP lane moves (no LDS crossbar round
// trips): prefixes within each row of 16 lanes by shifts of 1, 2, 4 and 8,
// then the last lane of row 0 is added to row 1 and that of row 2 to row 3,
// and the last lane of row 1 to rows 2 and 3.  Whole wave.
__device__ __forceinline__ int32_t wave_inclusive_sum(int32_t v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2, 3
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        T o = __shfl_xor(v, d, 64);
        v = o > v ? o : v;
    }
    return v;
}

// Exclusive scan over a block of NT threads (NT multiple of 64, <= 1024).
// `tmp` must hold NT/64 + 1 elements of LDS.  Returns the exclusive prefix of
// this thread and writes the block total to *total.
template <int NT, typename T>
__device__ __forceinline__ T block_exclusive_sum(T v, T* tmp, T* total) {
    constexpr int NW = NT / 64;
    const int w = threadIdx.x >> 6;
    T inc = wave_inclusive_sum(v);
    if (__lane_id() == 63) tmp[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        T acc = 0;
        for (int i = 0; i < NW; ++i) { T t = tmp[i]; tmp[i] = acc; acc += t; }
        tmp[NW] = acc;
    }
    __syncthreads();
    T r = tmp[w] + inc - v;
    *total = tmp[NW];
    __syncthreads();
    return r;
}

// SplitMix64 output function (Steele, Lea, Flood 2014).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

// mix64's first step, linear over xor: fold(a ^ b) = fold(a) ^ fold(b)
__device__ __forceinline__ uint64_t mix_fold(uint64_t z) { return z ^ (z >> 30); }

// (mix64(x) >> 11) < thr for z = mix_fold(x) and thr <= 2^53.  The top 31 bits
// of mix64 are those of its last product, whose high word takes three of the
// four partial products: they decide (*below) unless they equal thr's (true is
// returned, and folded_below_exact decides).
__device__ __forceinline__ bool folded_top(uint64_t z, uint64_t thr, bool* below) {
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    const uint32_t lo = (uint32_t)z, hi = (uint32_t)(z >> 32);
    const uint32_t top = (__umulhi(lo, 0x133111EBu) + lo * 0x94D049BBu + hi * 0x133111EBu) >> 1;
    *below = top < (uint32_t)(thr >> 22);
    return top == (uint32_t)(thr >> 22);
}

__device__ __forceinline__ bool folded_below_exact(uint64_t z, uint64_t thr) {
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    return ((z ^ (z >> 31)) >> 11) < thr;
}

// The seed-independent part of the coin of edge {u,v}, a hash of (min, max).
__device__ __forceinline__ uint64_t edge_mix(uint32_t u, uint32_t v) {
    const uint64_t lo = u < v ? u : v;
    const uint64_t hi = u < v ? v : u;
    return mix64((lo << 32) | hi);
}

// Keep decision of the undirected edge {u,v}: section 3.1's independent coin,
// realised as a hash of (min, max) salted by the seed.
__device__ __forceinline__ bool edge_kept(uint32_t u, uint32_t v, uint64_t salt, uint64_t thr) {
    return (mix64(edge_mix(u, v) ^ salt) >> 11) < thr;
}

// (deg, id) rank order
__device__ __forceinline__ bool rank_below(int32_t du, int32_t u, int32_t dv, int32_t v) {
    return du < dv || (du == dv && u < v);
}

// A byte that orders degrees: the degree itself below 16, above it 8 steps
// per octave (exponent and the three bits after the leading one), so
// class(d) < class(d') implies d < d', and equal classes below 16 mean equal
// degrees.  At most 16 + 8 * 26 + 7 = 231.
__host__ __device__ __forceinline__ uint32_t deg_class(int32_t d) {
    if (d < 16) return d > 0 ? (uint32_t)d : 0u;
    const int e = 31 - __builtin_clz((uint32_t)d);  // >= 4
    return 16u + 8u * (uint32_t)(e - 4) + (((uint32_t)d >> (e - 3)) & 7u);
}

// The largest degree of class c.
__device__ __forceinline__ int32_t class_max_degree(uint32_t c) {
    if (c < 16) return (int32_t)c;
    const uint32_t e = (c - 16) / 8 + 4;
    return (int32_t)(((8u + ((c - 16) & 7u) + 1u) << (e - 3)) - 1u);
}

}  // namespace tc
