// Device search of a position in a non-decreasing prefix through a bucket
// index, shared by the estimators that draw elements by position.
#pragma once

#include "tc_device.h"

namespace tc {

namespace {

// log2 of the buckets of an index over n items: at least as many as items
// (between 2^10 and 2^26)
inline int index_bits(int64_t n) {
    int k = 10;
    while (k < 26 && ((int64_t)1 << k) < n) ++k;
    return k;
}

// A non-decreasing prefix pre[0..n] (pre[0] = 0, pre[n] = total) with an
// index of 2^k buckets: bucket b starts at position floor(b total / 2^k), and
// idx[b] is the item u whose range [pre[u], pre[u+1]) holds that position.
// The item of a position r in bucket b lies between idx[b] and idx[b+1], so
// its search takes a few steps instead of log2 n dependent loads.
template <typename T>
struct PrefixIndex {
    const T* pre;         // n + 1 entries on the device; total = pre[n]
    const int32_t* idx;   // 2^k entries; null: none, every search is over all items
    int64_t n;
    int k;
};

// Bucket starts floor(b total / 2^k) = b q + floor(b rem / 2^k) with
// q = total >> k and rem = total mod 2^k: b, rem < 2^26, so b rem < 2^52.
struct Buckets {
    uint64_t q, rem;
    int k;
    __device__ __forceinline__ Buckets(uint64_t total, int k_) : q(total >> k_), rem(total & ((1ull << k_) - 1)), k(k_) {}
    __device__ __forceinline__ uint64_t start(uint64_t b) const { return b * q + ((b * rem) >> k); }
};

// the last bucket starting at or before r (r < total)
__device__ __forceinline__ int64_t bucket_of(uint64_t r, uint64_t total, int k) {
    const Buckets bs(total, k);
    const int64_t B = (int64_t)1 << k;
    int64_t b = (int64_t)((double)r / (double)total * (double)B);  // then made exact
    b = b < 0 ? 0 : (b > B - 1 ? B - 1 : b);
    while (b > 0 && bs.start((uint64_t)b) > r) --b;
    while (b + 1 < B && bs.start((uint64_t)(b + 1)) <= r) ++b;
    return b;
}

// the first bucket starting at or after x (B if none)
__device__ __forceinline__ int64_t first_bucket_at(uint64_t x, uint64_t total, int k) {
    const Buckets bs(total, k);
    const int64_t B = (int64_t)1 << k;
    int64_t b = (int64_t)ceil((double)x / (double)total * (double)B);  // then made exact
    b = b < 0 ? 0 : (b > B ? B : b);
    while (b > 0 && bs.start((uint64_t)(b - 1)) >= x) --b;
    while (b < B && bs.start((uint64_t)b) < x) ++b;
    return b;
}

// the item u with pre[u] <= r < pre[u+1] (the last u with pre[u] <= r), 0 <= r < total
template <typename T>
__device__ __forceinline__ int64_t find_item(const PrefixIndex<T>& P, int64_t r) {
    int64_t lo = 0, hi = P.n - 1;
    if (P.idx) {
        const int64_t B = (int64_t)1 << P.k;
        const int64_t b = bucket_of((uint64_t)r, (uint64_t)P.pre[P.n], P.k);
        lo = P.idx[b];
        if (b + 1 < B) hi = P.idx[b + 1];
    }
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo + 1) >> 1);
        if ((int64_t)P.pre[mid] <= r) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// idx of a prefix: every bucket start lies in exactly one non-empty range, and
// the item of that range writes it.  Items with at most 8 buckets write their
// own; the wave writes those of longer ranges together, one item at a time.
template <typename T>
__global__ void __launch_bounds__(256) k_bucket_index(int64_t n, const T* __restrict__ pre, int k,
                                                      int32_t* __restrict__ idx) {
    const uint64_t total = (uint64_t)pre[n];
    if (total == 0) return;
    const Buckets bs(total, k);
    const int lane = __lane_id();
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t u0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63); u0 < n; u0 += step) {
        // u0 is the wave's first item (wave-uniform), u this lane's
        const int64_t u = u0 + lane;
        int64_t b0 = 0, b1 = 0;
        if (u < n) {
            const uint64_t a = (uint64_t)pre[u], e = (uint64_t)pre[u + 1];
            if (a != e) {
                b0 = first_bucket_at(a, total, k);
                b1 = first_bucket_at(e, total, k);
            }
        }
        const bool mine = b1 - b0 <= 8;
        if (mine)
            for (int64_t b = b0; b < b1; ++b) idx[b] = (int32_t)u;
        uint64_t longs = ballot64(!mine);
        while (longs) {
            const int src = __ffsll((long long)longs) - 1;
            longs &= longs - 1;
            const int64_t lb0 = __shfl(b0, src, 64), lb1 = __shfl(b1, src, 64);
            for (int64_t b = lb0 + lane; b < lb1; b += 64) idx[b] = (int32_t)(u0 + src);
        }
    }
}

}  // namespace

}  // namespace tc
