// Shared by the estimators that draw elements by position: the search of a
// position in a non-decreasing prefix through a bucket index, the partition of
// the draws into the order of the elements, the lookup of an edge, the sums.
#pragma once

#include "tc_internal.h"
#include "tc_device.h"

#include <algorithm>

namespace tc {

namespace {

// p[0] and p[1] in one request.  Dword alignment is all that a global load of
// two dwords needs; a list's two ends share a line, but as two loads they are
// two requests (2^25 triples on R-MAT s22: 3.70 -> 3.54 ms).
__device__ __forceinline__ int2 two_at(const int32_t* __restrict__ p) {
    int2 r;
    __builtin_memcpy(&r, p, sizeof(r));
    return r;
}

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
// The range of a hub can hold nearly all of the buckets: groups of kIndexGroup
// buckets that lie in one range are left to the first `gblocks` blocks, a thread
// per group, which searches its item (one wave for all 2^20 buckets of a star of
// 2^20 vertices took 500 us).
constexpr int64_t kIndexGroup = 256;

template <typename T>
__global__ void __launch_bounds__(256) k_bucket_index(int64_t n, const T* __restrict__ pre, int k, int gblocks,
                                                      int32_t* __restrict__ idx) {
    const uint64_t total = (uint64_t)pre[n];
    if (total == 0) return;
    const Buckets bs(total, k);
    const int lane = __lane_id();
    if ((int)blockIdx.x < gblocks) {  // block-uniform
        const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x, groups = ((int64_t)1 << k) / kIndexGroup;
        int64_t u = 0;
        bool whole = false;
        if (g < groups) {
            u = find_item(PrefixIndex<T>{pre, nullptr, n, k}, (int64_t)bs.start((uint64_t)(g * kIndexGroup)));
            whole = bs.start((uint64_t)(g * kIndexGroup + kIndexGroup - 1)) < (uint64_t)pre[u + 1];
        }
        for (uint64_t rest = ballot64(whole); rest; rest &= rest - 1) {
            const int src = __builtin_ctzll(rest);
            const int64_t b0 = (g - lane + src) * kIndexGroup;
            const int32_t v = __shfl((int32_t)u, src, 64);
            for (int64_t b = b0 + lane; b < b0 + kIndexGroup; b += 64) idx[b] = v;
        }
        return;
    }
    const int64_t step = (int64_t)(gridDim.x - gblocks) * blockDim.x;
    for (int64_t u0 = (int64_t)(blockIdx.x - gblocks) * blockDim.x + (threadIdx.x & ~63); u0 < n; u0 += step) {
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
            int64_t g0 = (lb0 + kIndexGroup - 1) / kIndexGroup * kIndexGroup, g1 = lb1 / kIndexGroup * kIndexGroup;
            if (!gblocks || g0 >= g1) g0 = g1 = lb1;  // [g0, g1): whole groups, written above
            for (int64_t b = lb0 + lane; b < g0; b += 64) idx[b] = (int32_t)(u0 + src);
            for (int64_t b = g1 + lane; b < lb1; b += 64) idx[b] = (int32_t)(u0 + src);
        }
    }
}

// The index idx of the prefix pre of n items, 2^k buckets (k >= 10).  Below 2^16
// buckets one wave writes the longest range in the time of a group's search.
template <typename T>
inline void bucket_index(const char* name, int64_t n, const T* pre, int k, int32_t* idx, hipStream_t s) {
    const int gblocks = k >= 16 ? (int)(((int64_t)1 << k) / kIndexGroup / 256) : 0;
    const unsigned items = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 65536));
    TC_LAUNCH(name, k_bucket_index<T>, dim3(gblocks + items), dim3(256), 0, s, n, pre, k, gblocks, idx);
}

// y in the sorted list col[lo .. end) of ids below n (scale = 1 / n).  Every
// step of a binary search of a long list reads another cache line, so lists
// past one line are entered where y would be if their ids were spread evenly
// (as relabelled graphs' are: off by about the root of the length) and the
// range is widened from there by doubling: 2^25 triples on R-MAT s22 took 6.6 ->
// 5.5 ms, and it is at most twice the steps on any list.  Ids: a pointer, or
// what stands for a list in a check on the host.
template <typename Ids>
__host__ __device__ __forceinline__ bool in_list(Ids col, int32_t lo, int32_t end, int32_t y, float scale) {
    int32_t hi = end;
    if (end - lo > 32) {
        // the length rounds up past 2^24: held below it before lo, near 2^31 in the largest graphs, is added
        const int32_t at = (int32_t)((float)(end - lo) * ((float)y * scale));
        const int32_t g = lo + (at < end - lo - 1 ? at : end - lo - 1);
        int32_t step = 16;
        if (col[g] < y) {
            lo = g + 1;
            while (hi - lo > step && col[lo + step] < y) {
                lo += step + 1;
                step *= 2;
            }
            hi = hi - lo > step ? lo + step : hi;
        } else {
            hi = g;
            while (hi - lo > step && col[hi - 1 - step] >= y) {
                hi -= step + 1;
                step *= 2;
            }
            if (hi - lo > step) lo = hi - step;
        }
        // the first entry >= y lies in [lo, hi]
    }
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (col[mid] < y) lo = mid + 1;
        else hi = mid;
    }
    return lo < end && col[lo] == y;
}

__device__ __forceinline__ bool adjacent(const int32_t* __restrict__ rp, const int32_t* __restrict__ col, int32_t x,
                                         int32_t y, float scale) {
    const int2 xr = two_at(rp + x), yr = two_at(rp + y);
    return xr.y - xr.x <= yr.y - yr.x ? in_list(col, xr.x, xr.y, y, scale) : in_list(col, yr.x, yr.y, x, scale);
}

// the 64-bit hash of sample i: its element of U is the high half of h * |U|
__device__ __forceinline__ uint64_t sample_hash(int64_t i, uint64_t salt) { return mix64(mix64((uint64_t)i) ^ salt); }

// ---- partition of the samples ---------------------------------------------
// Samples in hash order touch prefixes, lists and list prefixes all over the
// graph (a new cache line per search step); after the partition a wave's
// samples lie in one 256th of U.  Counts per part, their bases, then the
// sample numbers (relative to i0) at their places, in any order inside a part.
constexpr int kParts = 256, kPartTile = 8192;

// Part of a sample: the top byte of its hash, hence of its position in U.
struct HashParts {
    __device__ __forceinline__ void load() {}
    __device__ __forceinline__ int32_t operator()(uint64_t hash) const { return (int32_t)(hash >> 56); }
};

template <typename Part>
__global__ void __launch_bounds__(256) k_part_count(int64_t i0, int64_t s, uint64_t salt, Part part_of,
                                                     int32_t* __restrict__ cnt) {
    __shared__ int32_t c[kParts];
    part_of.load();
    c[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < s; i += (int64_t)gridDim.x * 256)
        atomicAdd(&c[part_of(sample_hash(i0 + i, salt))], 1);
    __syncthreads();
    if (c[threadIdx.x]) atomicAdd(&cnt[threadIdx.x], c[threadIdx.x]);
}

// at[p]: the start of part p, raised to its end
template <typename Part>
__global__ void __launch_bounds__(256) k_part_place(int64_t i0, int64_t s, uint64_t salt, Part part_of,
                                                     int32_t* __restrict__ at, int32_t* __restrict__ order) {
    __shared__ int32_t c[kParts];
    part_of.load();
    for (int64_t t0 = (int64_t)blockIdx.x * kPartTile; t0 < s; t0 += (int64_t)gridDim.x * kPartTile) {
        c[threadIdx.x] = 0;
        __syncthreads();
        int32_t part[kPartTile / 256], rank[kPartTile / 256];
#pragma unroll
        for (int k = 0; k < kPartTile / 256; ++k) {
            const int64_t i = t0 + 256 * k + threadIdx.x;
            part[k] = i < s ? part_of(sample_hash(i0 + i, salt)) : -1;
            rank[k] = i < s ? atomicAdd(&c[part[k]], 1) : 0;
        }
        __syncthreads();
        const int32_t mine = c[threadIdx.x];
        c[threadIdx.x] = mine ? atomicAdd(&at[threadIdx.x], mine) : 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPartTile / 256; ++k)
            if (part[k] >= 0) order[c[part[k]] + rank[k]] = (int32_t)(t0 + 256 * k + threadIdx.x);
        __syncthreads();
    }
}

// Sums of the samples, spread over lines of 128 bytes.
constexpr int kAccLines = 64, kAccStride = 16;

// Samples of one block of the kernels that read them: contiguous ones, one per
// thread, so that the resident blocks work close together and none starts a long
// share when the others end (R-MAT s22, against 2048 blocks striding through
// all: 2^25 triples 5.5 -> 4.3 ms, 2^24 draws of the stream 2.0 -> 1.6).
constexpr int64_t kDrawsPerBlock = 256;

// Blocks for c >= 1 samples, a multiple of the XCDs; past 2^28 samples their
// shares grow (a grid holds fewer than 2^32 threads).
inline unsigned draw_blocks(int64_t c) {
    const int64_t per_xcd = (c - 1) / (8 * kDrawsPerBlock) + 1;
    return 8 * (unsigned)std::min<int64_t>(per_xcd, (int64_t)1 << 17);
}

// Samples partitioned together, and the calls whose samples are.  Triples: R-MAT
// s22 with 2^25 samples took 16.3 -> 6.4 ms; from 2^21 samples it is 1.0 to 1.1
// times faster on R-MAT s17 to s21 and from 2^23 1.2 to 1.4 times; at 2^20 and
// below the two more launches cost what the locality gains (0.9 to 1.0 times),
// and graphs below s17 fit the caches (0.9 times).
constexpr int64_t kPartChunk = (int64_t)1 << 26;
constexpr int64_t kPartSamples = (int64_t)1 << 21;
constexpr int64_t kPartEntries = (int64_t)1 << 22;

inline bool samples_partitioned(int64_t samples, int64_t m) { return samples >= kPartSamples && 2 * m >= kPartEntries; }

// order[0 .. c) = the numbers i < c of the samples i0 + i by their parts; at[p]
// = the end of part p (kParts + 1 words)
template <typename Part>
inline void partition_samples(int64_t i0, int64_t c, uint64_t salt, const Part& part_of, int32_t* at, int32_t* order,
                              hipStream_t s) {
    fill_i32(at, 0, kParts, s);
    TC_LAUNCH("part_count", k_part_count<Part>, dim3((unsigned)num_cus() * 8), dim3(256), 0, s, i0, c, salt, part_of,
              at);
    scan_exclusive_i32(at, at, kParts, s);
    TC_LAUNCH("part_place", k_part_place<Part>, dim3(ceil_div(c, kPartTile)), dim3(256), 0, s, i0, c, salt, part_of,
              at, order);
}

// Adds the block's sums (256 threads) of a and b to words 0 and 1 of a line of
// acc (kAccLines lines of kAccStride words): one atomic per block and sum; per
// wave on one line they took 200 of 330 us at 2^19 triples on R-MAT s15.
__device__ __forceinline__ void add_to_lines(int64_t a, int64_t b, unsigned long long* __restrict__ acc) {
    __shared__ int64_t red[4][2];
    a = wave_sum(a);
    b = wave_sum(b);
    if (__lane_id() == 0) {
        red[threadIdx.x >> 6][0] = a;
        red[threadIdx.x >> 6][1] = b;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const int64_t t = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
        if (t) atomicAdd(&acc[(blockIdx.x % kAccLines) * kAccStride + threadIdx.x], (unsigned long long)t);
    }
}

}  // namespace

}  // namespace tc
