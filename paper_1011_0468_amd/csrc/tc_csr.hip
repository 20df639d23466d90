// CSR construction: the simple undirected graph of the pairs, every neighbour
// list sorted ascending (section 4.1 and the sorted neighbour-list format of
// section 4.2).
//
// Each pair (u, v), u != v, gives the keys (u, v) and (v, u) of nb bits a
// half.  They are sorted and made unique by windows of consecutive rows:
//
//   1. hist   : keys per window (the top W bits of u, some thousand keys each);
//   2. part   : the keys scattered to their windows, in any order, by one
//               pass over the pairs (W <= 8), or by one over the top W - 8
//               bits and one over the next 8.  A key leaves its window's bits
//               behind, and the windows hold 4-byte keys where 2 nb - W <= 32 (W
//               grows with the pairs: R-MAT s22 29 bits; 2^20 vertices and 30000
//               pairs 33);
//   3. sort   : each window sorted and made unique in LDS, its rows' degrees
//               stored;
//   4. big    : windows of more than kWindowCap keys (the hubs' windows of a
//               skewed graph) sorted by stable radix passes over their tiles;
//   5. emit   : columns, rows and the neighbours' degree classes at the places
//               that the counts' prefix gives.
//
// All of it is bound by memory: every pass reads and writes each key once, and
// here that is 40 bytes a key where six LSD passes over 8-byte keys, flags and
// positions took 160.  R-MAT s22 (2^26 pairs): 10.5 -> 4.4 ms.
#include "tc_internal.h"
#include "tc_device.h"

#include <algorithm>

namespace tc {

namespace {

constexpr int kDigit = 8;             // bits of a partition or radix digit
constexpr int kRadix = 1 << kDigit;
constexpr int kMaxWindowBits = 15;    // 2^15 counters take 128 KB of LDS
// Keys aimed at per window: as few as one pass of 256 windows gives, since the
// windows are then cheap and their hubs' rows stay below the cap; more where
// every further bit lengthens the second pass's tables.
constexpr int kOnePassKeys = 512, kWindowKeys = 2048;
// Most keys that a window sorts in LDS: 1024 threads of 8 keys, two blocks per
// CU; in a build of one pass, whose windows leave CUs idle, of 16 (4-byte keys).
constexpr int kWindowCap = 8192;
constexpr int kTile = 4096;           // keys per tile of a larger window
constexpr int kPartThreads = 512;
constexpr int kPartKeys = 8192;       // keys per tile of the partition (64 KB of LDS: 2 blocks per CU)
constexpr int kMaxPartBlocks = 512;   // persistent blocks of the pass over the pairs
constexpr int kHistThreads = 1024;

// Device-side facts of a build, read back together.
enum Info { kBad = 0, kUnits, kBigTiles, kTotal, kMaxDeg, kListed, kInfoN };

// How a build is cut: nb bits per id, W window bits (top of u), of which the
// first pass takes b1.  Keys keep rest = 2 nb - W bits inside a window.
struct CsrPlan {
    int nb, W, b1, rest;
    int64_t bins, parts;
    int64_t tiles;       // tiles of kPartKeys / 2 pairs
    int gpart, ghist;    // blocks of the pass over the pairs and of the histogram
};

CsrPlan csr_plan(int64_t n, int64_t P) {
    CsrPlan c{};
    c.nb = 1;
    while (c.nb < 31 && ((int64_t)1 << c.nb) < n) ++c.nb;
    c.W = 1;
    while (c.W < kMaxWindowBits && c.W < c.nb && ((int64_t)(c.W < kDigit ? kOnePassKeys : kWindowKeys) << c.W) < 2 * P)
        ++c.W;
    c.b1 = c.W > kDigit ? c.W - kDigit : c.W;
    c.rest = 2 * c.nb - c.W;
    c.bins = (int64_t)1 << c.W;
    c.parts = (int64_t)1 << c.b1;
    c.tiles = (P + kPartKeys / 2 - 1) / (kPartKeys / 2);
    c.gpart = (int)std::max<int64_t>(1, std::min<int64_t>(c.tiles, kMaxPartBlocks));
    c.ghist = std::max(1, (c.gpart + 1) / 2);
    return c;
}

struct Seg {              // a window above the cap
    int32_t bin, start, len, tile0, concat, pad;
};

__device__ __forceinline__ int32_t tiles_of(int32_t len, int32_t tile) {
    return (int32_t)(((int64_t)len + tile - 1) / tile);
}

// Both keys of a pair: false for a loop or an id outside [0, n) (bad is set).
__device__ __forceinline__ bool pair_ok(int32_t u, int32_t v, int64_t n, int32_t* bad) {
    const bool ok = u >= 0 && v >= 0 && (int64_t)u < n && (int64_t)v < n;
    if (!ok) *bad = 1;
    return ok && u != v;
}

// Keys per window.  Block h counts the tiles of the partition blocks h and
// h + ghist into one LDS table (row h of binrows), and after each of the two
// the keys per part of the first pass (row g of partrows, g that block), so
// that the partition knows every block's places without an atomic.
__global__ void __launch_bounds__(kHistThreads) k_csr_hist(const int32_t* __restrict__ src,
                                                            const int32_t* __restrict__ dst, int64_t P, int64_t n,
                                                            int shift, int bins, int parts, int64_t tiles, int gpart,
                                                            int32_t* __restrict__ binrows,
                                                            int32_t* __restrict__ partrows,
                                                            int32_t* __restrict__ info) {
    extern __shared__ int32_t cnt[];  // bins counters, then parts (the first block's)
    int32_t* before = cnt + bins;
    const int t = threadIdx.x;
    for (int i = t; i < bins; i += kHistThreads) cnt[i] = 0;
    for (int i = t; i < parts; i += kHistThreads) before[i] = 0;
    __syncthreads();
    const int per = bins / parts;
    int32_t bad = 0;
    for (int g = blockIdx.x; g < gpart; g += gridDim.x) {  // at most two rounds, block-uniform
        for (int64_t tile = g; tile < tiles; tile += gpart) {
            const int64_t i0 = tile * (kPartKeys / 2);
            int32_t u[kPartKeys / 2 / kHistThreads], v[kPartKeys / 2 / kHistThreads];
#pragma unroll
            for (int k = 0; k < kPartKeys / 2 / kHistThreads; ++k) {
                const int64_t i = i0 + k * kHistThreads + t;
                u[k] = i < P ? src[i] : 0;
                v[k] = i < P ? dst[i] : 0;
            }
#pragma unroll
            for (int k = 0; k < kPartKeys / 2 / kHistThreads; ++k) {
                if (i0 + k * kHistThreads + t < P && pair_ok(u[k], v[k], n, &bad)) {
                    atomicAdd(&cnt[u[k] >> shift], 1);
                    atomicAdd(&cnt[v[k] >> shift], 1);
                }
            }
        }
        __syncthreads();
        // one wave per part: its windows' sum, less what the round before counted
        for (int p = t >> 6; p < parts; p += kHistThreads / 64) {
            int32_t s = 0;
            for (int i = t & 63; i < per; i += 64) s += cnt[p * per + i];
            s = wave_sum(s);
            if ((t & 63) == 0) {
                partrows[(int64_t)g * parts + p] = s - before[p];
                before[p] = s;
            }
        }
        __syncthreads();
    }
    for (int i = t; i < bins; i += kHistThreads) binrows[(int64_t)blockIdx.x * bins + i] = cnt[i];
    if (bad) info[kBad] = 1;
}

// Of every window: its keys (the sum of its column), its units (one, or the
// tiles of a window above cap), its tiles and its keys if above cap.  Their
// exclusive prefixes are what the passes below use: start, unit0, tile0 and
// concat (bins + 1 entries each).
__global__ void __launch_bounds__(256) k_csr_bins(int bins, int rows, int32_t cap, const int32_t* __restrict__ binrows,
                                                   int32_t* __restrict__ start, int32_t* __restrict__ unit0,
                                                   int32_t* __restrict__ tile0, int32_t* __restrict__ concat) {
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= bins) return;
    int32_t s = 0;
#pragma unroll 8
    for (int r = 0; r < rows; ++r) s += binrows[(int64_t)r * bins + b];
    const int32_t T = s > cap ? tiles_of(s, kTile) : 0;
    start[b] = s;
    unit0[b] = T ? T : (s > 0 ? 1 : 0);
    tile0[b] = T;
    concat[b] = T ? s : 0;
}

// The units that hold the keys in order (a window of at most cap keys, or each
// tile of a larger one) as (start, length, window, segment or -1), the larger
// windows (segs, by their first tile) and the cursors of the second pass.
__global__ void __launch_bounds__(256) k_csr_units(int bins, int32_t cap, const int32_t* __restrict__ start,
                                                    const int32_t* __restrict__ unit0,
                                                    const int32_t* __restrict__ tile0,
                                                    const int32_t* __restrict__ concat, int32_t* __restrict__ cursor,
                                                    int4* __restrict__ units, Seg* __restrict__ segs,
                                                    int32_t* __restrict__ tile_seg, int32_t* __restrict__ info) {
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= bins) return;
    const int32_t s0 = start[b], len = start[b + 1] - s0, u0 = unit0[b], t0 = tile0[b];
    if (cursor) cursor[b] = s0;
    if (len > cap) {
        segs[t0] = Seg{b, s0, len, t0, concat[b], 0};
        for (int i = 0; i < tiles_of(len, kTile); ++i) {
            units[u0 + i] = make_int4(s0 + i * kTile, min(kTile, len - i * kTile), b, t0);
            tile_seg[t0 + i] = t0;
        }
    } else if (len > 0) {
        units[u0] = make_int4(s0, len, b, -1);
    }
    if (b == 0) {
        info[kUnits] = unit0[bins];
        info[kBigTiles] = tile0[bins];
    }
}

// partrows[g][p] becomes the first place of block g's keys of part p: one
// block per part, 512 >= gpart threads.
__global__ void __launch_bounds__(512) k_csr_part_base(int gpart, int parts, int bins_per_part,
                                                        const int32_t* __restrict__ start,
                                                        int32_t* __restrict__ partrows) {
    __shared__ int32_t tmp[9];
    const int g = threadIdx.x, p = blockIdx.x;
    const int32_t c = g < gpart ? partrows[(int64_t)g * parts + p] : 0;
    int32_t total;
    const int32_t pre = block_exclusive_sum<512>(c, tmp, &total);
    if (g < gpart) partrows[(int64_t)g * parts + p] = start[p * bins_per_part] + pre;
}

// One tile's keys to their parts: cnt[d] keys of digit d, each with its rank
// among them (LDS atomics, any order), are put in digit order in LDS and
// written from there, so that the stores of a part are contiguous.
// base[d]: the part's next place for this tile.
template <typename K, typename KO, int ITEMS>
__device__ __forceinline__ void part_tile(const K (&key)[ITEMS], const int (&dg)[ITEMS], const int32_t (&rk)[ITEMS],
                                          int32_t* cnt, int32_t* loc, const int32_t* base, int32_t* tmp, K* stage,
                                          int shift, K keep, KO* __restrict__ out) {
    const int t = threadIdx.x;
    int32_t total;
    const int32_t pre = block_exclusive_sum<kPartThreads>(t < kRadix ? cnt[t] : 0, tmp, &total);
    if (t < kRadix) loc[t] = pre;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
        if (dg[k] >= 0) stage[loc[dg[k]] + rk[k]] = key[k];
    __syncthreads();
    for (int32_t j = t; j < total; j += kPartThreads) {
        const K x = stage[j];
        const int d = (int)(x >> shift) & (kRadix - 1);
        out[base[d] + (j - loc[d])] = (KO)(x & keep);
    }
}

// The pass over the pairs: block g takes the tiles g, g + gpart, .. and keeps
// its parts' cursors in LDS.  shift: the position of the first pass's digit
// (at most 8 bits) in a key; keep: the bits of a key that are written.
template <typename K, typename KO>
__global__ void __launch_bounds__(kPartThreads) k_csr_part1(const int32_t* __restrict__ src,
                                                             const int32_t* __restrict__ dst, int64_t P, int64_t n,
                                                             int nb, int shift, K keep, int parts, int64_t tiles,
                                                             const int32_t* __restrict__ partrows,
                                                             KO* __restrict__ out) {
    constexpr int PAIRS = kPartKeys / 2 / kPartThreads;
    __shared__ __attribute__((aligned(16))) K stage[kPartKeys];
    __shared__ int32_t cnt[kRadix], loc[kRadix], base[kRadix], tmp[kPartThreads / 64 + 1];
    const int t = threadIdx.x;
    if (t < kRadix) base[t] = t < parts ? partrows[(int64_t)blockIdx.x * parts + t] : 0;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        if (t < kRadix) cnt[t] = 0;
        const int64_t i0 = tile * (kPartKeys / 2);
        int32_t u[PAIRS], v[PAIRS];
#pragma unroll
        for (int k = 0; k < PAIRS; ++k) {
            const int64_t i = i0 + k * kPartThreads + t;
            u[k] = i < P ? src[i] : 0;
            v[k] = i < P ? dst[i] : 0;
        }
        __syncthreads();
        K key[2 * PAIRS];
        int dg[2 * PAIRS];
        int32_t rk[2 * PAIRS], bad = 0;
#pragma unroll
        for (int k = 0; k < PAIRS; ++k) {
            const bool ok = pair_ok(u[k], v[k], n, &bad);  // (0, 0) past the end: a loop
            key[2 * k] = ((K)(uint32_t)u[k] << nb) | (K)(uint32_t)v[k];
            key[2 * k + 1] = ((K)(uint32_t)v[k] << nb) | (K)(uint32_t)u[k];
#pragma unroll
            for (int e = 2 * k; e < 2 * k + 2; ++e) {
                dg[e] = ok ? (int)(key[e] >> shift) & (kRadix - 1) : -1;
                rk[e] = ok ? atomicAdd(&cnt[dg[e]], 1) : 0;
            }
        }
        __syncthreads();
        part_tile<K, KO, 2 * PAIRS>(key, dg, rk, cnt, loc, base, tmp, stage, shift, keep, out);
        __syncthreads();
        if (t < kRadix) base[t] += cnt[t];
        __syncthreads();
    }
}

// The second pass: tiles of one part each, places claimed per tile and digit
// from the windows' cursors (a few dozen claims on each of 2^15 counters).
template <typename K, typename KO>
__global__ void __launch_bounds__(kPartThreads) k_csr_part2(const K* __restrict__ in, int parts, int bins_per_part,
                                                             int shift, K keep, const int32_t* __restrict__ start,
                                                             int32_t* __restrict__ cursor, KO* __restrict__ out) {
    constexpr int ITEMS = kPartKeys / kPartThreads;
    __shared__ __attribute__((aligned(16))) K stage[kPartKeys];
    __shared__ int32_t cnt[kRadix], loc[kRadix], base[kRadix], first[kRadix], tmp[kPartThreads / 64 + 1];
    const int t = threadIdx.x;
    // the part of this tile: parts <= 128 threads hold the tile counts' prefix
    int32_t mine = 0, ntiles;
    if (t < parts) {
        const int32_t len = start[(t + 1) * bins_per_part] - start[t * bins_per_part];
        mine = tiles_of(len, kPartKeys);
    }
    const int32_t pre = block_exclusive_sum<kPartThreads>(mine, tmp, &ntiles);
    if ((int32_t)blockIdx.x >= ntiles) return;  // block-uniform
    if (t < parts) first[t] = pre;
    if (t < kRadix) cnt[t] = 0;
    __syncthreads();
    int lo = 0, hi = parts - 1;  // the last part whose tiles start at or before this one
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= (int32_t)blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const int64_t i0 = (int64_t)start[lo * bins_per_part] + (int64_t)((int32_t)blockIdx.x - first[lo]) * kPartKeys;
    const int64_t end = start[(lo + 1) * bins_per_part];
    K key[ITEMS];
    int dg[ITEMS];
    int32_t rk[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t i = i0 + k * kPartThreads + t;
        key[k] = i < end ? in[i] : (K)0;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const bool ok = i0 + k * kPartThreads + t < end;
        dg[k] = ok ? (int)(key[k] >> shift) & (kRadix - 1) : -1;
        rk[k] = ok ? atomicAdd(&cnt[dg[k]], 1) : 0;
    }
    __syncthreads();
    if (t < kRadix) base[t] = cnt[t] ? atomicAdd(&cursor[lo * bins_per_part + t], cnt[t]) : 0;
    part_tile<K, KO, ITEMS>(key, dg, rk, cnt, loc, base, tmp, stage, shift, keep, out);
}

// Orders one wave's LDS accesses (they execute in issue order).
__device__ __forceinline__ void csr_wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Stable ranks of a block's keys by one digit.  Wave w holds the positions
// [w per, (w + 1) per), item i of lane l at w per + 64 i + l; the keys of one
// digit before an item's are counted per wave in hist[w][digit], their peers
// in the same 64 found by one ballot per digit bit.  Afterwards hist[w][d] is
// the place of wave w's first key of digit d among the block's, and rk the
// rank behind it.  Leaves the block synchronised.
template <int T, int I, typename K>
__device__ __forceinline__ void radix_ranks(const K (&key)[I], int32_t (&rk)[I], int32_t count, int32_t per, int shift,
                                            int bits, int32_t* hist, int32_t* tmp) {
    constexpr int NW = T / 64;
    const int t = threadIdx.x, w = t >> 6, lane = __lane_id();
    for (int i = t; i < NW * kRadix; i += T) hist[i] = 0;
    __syncthreads();
    int32_t* mine = hist + w * kRadix;
    const uint64_t below = lanes_below();
#pragma unroll
    for (int i = 0; i < I; ++i) {
        if (64 * i < per) {  // block-uniform
            const bool ok = w * per + 64 * i + lane < count;
            const uint32_t d = (uint32_t)(key[i] >> shift) & ((1u << bits) - 1);
            uint64_t peers = ballot64(ok);
#pragma unroll
            for (int b = 0; b < kDigit; ++b) {  // bits past `bits` are zero in every key
                const int32_t s = (int32_t)(d << (31 - b)) >> 31;  // all ones where bit b is set
                const uint64_t bal = ballot64(ok && s);
                peers &= ~(bal ^ (uint64_t)(int64_t)s);
            }
            const int32_t had = mine[d];
            rk[i] = had + (int32_t)__popcll(peers & below);
            csr_wave_order();
            if (ok && (peers & below) == 0) mine[d] = had + (int32_t)__popcll(peers);
            csr_wave_order();
        }
    }
    __syncthreads();
    int32_t sum = 0;
    if (t < kRadix)
        for (int q = 0; q < NW; ++q) sum += hist[q * kRadix + t];
    int32_t total;
    int32_t run = block_exclusive_sum<T>(sum, tmp, &total);
    if (t < kRadix)
        for (int q = 0; q < NW; ++q) {
            const int32_t c = hist[q * kRadix + t];
            hist[q * kRadix + t] = run;
            run += c;
        }
    __syncthreads();
}

// Windows of at most 1024 I keys, one block each: sorted in LDS by their rest bits,
// made unique, written back to the window's start with their number, and the
// degree of every row that has keys stored.
//
// The keys are counted per group (the top bits of a row's place in the window:
// a row each, up to 256), and a group of c keys is cut by its next bits into
// c / 4 to c / 2 sub-windows, so that a hub's row is cut finer than its
// neighbours'.  Every key then counts the smaller keys of its sub-window: a
// few LDS reads, where radix passes over all 29 bits took four passes of
// ranking by ballots (R-MAT s22: 2.97 ms for the windows, this 1.0).  The
// count is quadratic in a sub-window: past kSubPerPass keys in one for each
// pass that the radix would take, where a row's neighbours are bunched, the
// radix passes are the shorter way.  The count's kernel (a block per window)
// leaves such a window as it is and lists it, and the RADIX kernel's persistent
// blocks take the list.  Complete bipartite 2000 x 20000 and 1000 x 30000, 15
// rest bits, sub-windows of 64 and 128 keys: builds of 4.7 and 3.2 ms with
// 128 allowed whatever the passes, 2.6 and 2.5 with 24 a pass; 2^20 vertices with
// 16 pairs each among the next 40, 25 bits: 1.9 ms with 16 allowed in all, 1.3
// with 16 to 28 a pass.
constexpr int kGroupBits = 8;
constexpr int32_t kSubPerPass = 24;
// counters: half the keys, one more per group, as whole rounds of 1024
constexpr int sub_windows(int items) { return items * 512 + 1024; }

template <int I, bool RADIX, typename K>
__global__ void __launch_bounds__(1024, I == 8 && sizeof(K) == 4 && !RADIX ? 8 : 4)
k_csr_sort(K* __restrict__ keys, const int32_t* __restrict__ start, const int32_t* __restrict__ unit0, int nb, int rest,
           int row_bits, int32_t* __restrict__ list, int32_t* __restrict__ listed, int32_t* __restrict__ ucount,
           int32_t* __restrict__ deg) {
    constexpr int T = 1024, HI = T * I, NW = T / 64, SUB = sub_windows(I);
    static_assert(NW * kRadix <= SUB && HI / 2 + (1 << kGroupBits) <= SUB, "radix counts; sub-windows");
    extern __shared__ __attribute__((aligned(16))) char sort_lds[];
    K* s = reinterpret_cast<K*>(sort_lds);
    int32_t* cnt = reinterpret_cast<int32_t*>(sort_lds + sizeof(K) * HI);  // SUB + 1
    __shared__ int32_t tmp[NW + 1], most[NW], group[1 << kGroupBits];
    const int t = threadIdx.x, w = t >> 6, lane = __lane_id();
    for (int32_t it = blockIdx.x; !RADIX || it < listed[0]; it += gridDim.x) {
        const int bin = RADIX ? list[it] : it;
        const int32_t s0 = start[bin];
        const int32_t count = start[bin + 1] - s0;
        if (count == 0 || count > HI) return;  // block-uniform; the list holds none such
        const int32_t per = (count + T - 1) / T * 64;
        // wave w: positions [w per, (w + 1) per), item i of lane l at w per + 64 i + l
        K key[I];
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const int32_t j = w * per + 64 * i + lane;
            key[i] = 64 * i < per && j < count ? keys[s0 + j] : (K)0;
        }
        int32_t at[I];
        if constexpr (RADIX) {
            for (int shift = 0; shift < rest; shift += kDigit) {
                const int bits = min(kDigit, rest - shift);
                radix_ranks<T, I, K>(key, at, count, per, shift, bits, cnt, tmp);
#pragma unroll
                for (int i = 0; i < I; ++i) {
                    if (64 * i < per && w * per + 64 * i + lane < count) {
                        const uint32_t d = (uint32_t)(key[i] >> shift) & ((1u << bits) - 1);
                        s[cnt[w * kRadix + d] + at[i]] = key[i];
                    }
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < I; ++i)
                    if (64 * i < per) key[i] = s[min(w * per + 64 * i + lane, count - 1)];
                // the next digit's scatter comes after its barriers
            }
        } else {
            for (int i = t; i <= SUB; i += T) cnt[i] = 0;
            if (t < (1 << kGroupBits)) group[t] = 0;
            __syncthreads();
            const int gs = rest - min(row_bits, kGroupBits);  // >= 1: the bits below the group
#pragma unroll
            for (int i = 0; i < I; ++i)
                if (64 * i < per && w * per + 64 * i + lane < count) atomicAdd(&group[(int)(key[i] >> gs)], 1);
            __syncthreads();
            {
                const int32_t c = t < (1 << kGroupBits) ? group[t] : 0;
                const int k = c >= 4 ? min(30 - __builtin_clz((uint32_t)c), gs) : 0;
                int32_t total;
                const int32_t first = block_exclusive_sum<T>(c ? 1 << k : 0, tmp, &total);
                if (t < (1 << kGroupBits)) group[t] = first | (k << 16);  // at most HI / 2 + 256 in all
            }
            __syncthreads();
            auto sub_of = [&](K x) {
                const int32_t g = group[(int)(x >> gs)];
                const int k = g >> 16;
                return (g & 0xFFFF) + (int32_t)((x >> (gs - k)) & (((K)1 << k) - 1));
            };
            // at: arrival rank in the sub-window, then the place in s
#pragma unroll
            for (int i = 0; i < I; ++i)
                if (64 * i < per && w * per + 64 * i + lane < count) at[i] = atomicAdd(&cnt[sub_of(key[i])], 1);
            __syncthreads();
            {
                constexpr int C = SUB / T;  // consecutive counters of a thread
                int32_t c[C], sum = 0, top = 0;
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    c[i] = cnt[t * C + i];
                    sum += c[i];
                    top = c[i] > top ? c[i] : top;
                }
                top = wave_max(top);
                if (lane == 0) most[w] = top;
                int32_t total;
                int32_t run = block_exclusive_sum<T>(sum, tmp, &total);
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    cnt[t * C + i] = run;
                    run += c[i];
                }
                if (t == T - 1) cnt[SUB] = total;
            }
            __syncthreads();
            int32_t top = most[0];
            for (int i = 1; i < NW; ++i) top = max(top, most[i]);
            if (top > kSubPerPass * ((rest + kDigit - 1) / kDigit)) {  // block-uniform
                if (t == 0) list[atomicAdd(listed, 1)] = bin;
                return;
            }
#pragma unroll
            for (int i = 0; i < I; ++i)
                if (64 * i < per && w * per + 64 * i + lane < count) {
                    at[i] += cnt[sub_of(key[i])];
                    s[at[i]] = key[i];
                }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < I; ++i)
                if (64 * i < per && w * per + 64 * i + lane < count) {
                    const int sub = sub_of(key[i]);
                    const int32_t a = cnt[sub], e = cnt[sub + 1];
                    int32_t r = a;  // equal keys keep their order of arrival
                    // a small multigraph's hub window holds long runs of equal keys:
                    // four reads in flight (10,007 vertices, 160,000 R-MAT pairs: 54 ->
                    // 46 us); with 8 items the sub-windows are 3 keys on average
                    constexpr int U = I == 16 ? 4 : 1;
#pragma unroll U
                    for (int32_t j = a; j < e; ++j) {
                        const K x = s[j];
                        r += x < key[i] || (x == key[i] && j < at[i]) ? 1 : 0;
                    }
                    at[i] = r;
                }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < I; ++i)
                if (64 * i < per && w * per + 64 * i + lane < count) s[at[i]] = key[i];
            __syncthreads();
        }
        // the first of each run of equal keys, in order: ranks by wave ballots
        uint32_t first = 0;  // bit i: item i is one
        int32_t mine = 0;    // of this wave
        const uint64_t below = lanes_below();
#pragma unroll
        for (int i = 0; i < I; ++i) {
            if (64 * i < per) {
                const int32_t j = w * per + 64 * i + lane;
                key[i] = s[min(j, count - 1)];
                const bool f = j < count && (j == 0 || s[j - 1] != key[i]);
                if (f) first |= 1u << i;
                mine += (int32_t)__popcll(ballot64(f));
            }
        }
        int32_t total;
        int32_t run = block_exclusive_sum<T>(lane == 0 ? mine : 0, tmp, &total);
        run = __shfl(run, 0, 64);
        __syncthreads();  // all reads of s done
#pragma unroll
        for (int i = 0; i < I; ++i) {
            if (64 * i < per) {
                const uint64_t b = ballot64((first >> i) & 1u);
                if ((first >> i) & 1u) {
                    const int32_t o = run + (int32_t)__popcll(b & below);
                    s[o] = key[i];
                    keys[s0 + o] = key[i];
                }
                run += (int32_t)__popcll(b);
            }
        }
        __syncthreads();
        // the last key of a row stores the row's degree: its place less the row's first
        const int64_t row0 = (int64_t)bin << row_bits;
        for (int32_t j = t; j < total; j += T) {
            const K r = s[j] >> nb;
            if (j + 1 < total && (s[j + 1] >> nb) == r) continue;
            int32_t lo = 0, hi = j;  // the first key of row r
            while (lo < hi) {
                const int32_t mid = (lo + hi) >> 1;
                if ((s[mid] >> nb) < r) lo = mid + 1;
                else hi = mid;
            }
            deg[row0 + (int64_t)r] = j + 1 - lo;
        }
        if (t == 0) ucount[unit0[bin]] = total;
        if (!RADIX) return;
        __syncthreads();  // s is read until here
    }
}

// ---- windows above kWindowCap: stable radix passes over their tiles --------
// Counts are laid out segment, digit, tile, so that one exclusive scan over
// all of them gives every tile's places (plus where the segment starts).

template <typename K>
__global__ void __launch_bounds__(256) k_big_hist(const K* __restrict__ keys, const Seg* __restrict__ segs,
                                                   const int32_t* __restrict__ tile_seg, int shift, int bits,
                                                   int32_t* __restrict__ hist) {
    __shared__ int32_t cnt[kRadix];
    const int t = threadIdx.x;
    const Seg g = segs[tile_seg[blockIdx.x]];
    const int32_t ti = blockIdx.x - g.tile0, T = tiles_of(g.len, kTile);
    cnt[t] = 0;
    __syncthreads();
    // places in the tile, not in the window: those of a window of nearly 2^31 keys leave int32 with the last step
    const int32_t j0 = ti * kTile, count = min(kTile, g.len - j0);
    for (int32_t j = t; j < count; j += 256)
        atomicAdd(&cnt[(uint32_t)(keys[g.start + j0 + j] >> shift) & ((1u << bits) - 1)], 1);
    __syncthreads();
    hist[(int64_t)g.tile0 * kRadix + (int64_t)t * T + ti] = cnt[t];
}

template <typename K>
__global__ void __launch_bounds__(256) k_big_scatter(const K* __restrict__ in, K* __restrict__ out,
                                                      const Seg* __restrict__ segs,
                                                      const int32_t* __restrict__ tile_seg, int shift, int bits,
                                                      const int32_t* __restrict__ offs) {
    constexpr int I = kTile / 256;
    __shared__ __attribute__((aligned(16))) K s[kTile];
    __shared__ int32_t hist[4 * kRadix], at[kRadix], tmp[5];
    const int t = threadIdx.x, w = t >> 6, lane = __lane_id();
    const Seg g = segs[tile_seg[blockIdx.x]];
    const int32_t ti = blockIdx.x - g.tile0, T = tiles_of(g.len, kTile);
    const int32_t j0 = ti * kTile, count = min(kTile, g.len - j0);
    const int32_t per = (count + 255) / 256 * 64;
    K key[I];
    int32_t rk[I];
#pragma unroll
    for (int i = 0; i < I; ++i) {
        const int32_t j = w * per + 64 * i + lane;
        key[i] = 64 * i < per && j < count ? in[g.start + j0 + j] : (K)0;
    }
    radix_ranks<256, I, K>(key, rk, count, per, shift, bits, hist, tmp);
    const uint32_t dmask = (1u << bits) - 1;
    // place of the tile's first key of digit t, less its place inside the tile (hist row 0)
    at[t] = offs[(int64_t)g.tile0 * kRadix + (int64_t)t * T + ti] - g.concat + g.start - hist[t];
#pragma unroll
    for (int i = 0; i < I; ++i)
        if (64 * i < per && w * per + 64 * i + lane < count)
            s[hist[w * kRadix + ((uint32_t)(key[i] >> shift) & dmask)] + rk[i]] = key[i];
    __syncthreads();
    for (int32_t j = t; j < count; j += 256) {
        const K x = s[j];
        out[at[(uint32_t)(x >> shift) & dmask] + j] = x;
    }
}

// Unique keys of every tile, and the degrees.  A hub's row fills many tiles,
// and its keys would meet in one counter: each wave takes a quarter of the
// tile in order and adds a row's keys when the row ends (one atomic per 64
// keys took 0.67 ms on R-MAT s22, this 0.08).
template <typename K>
__global__ void __launch_bounds__(256) k_big_count(const K* __restrict__ keys, const Seg* __restrict__ segs,
                                                    const int32_t* __restrict__ tile_seg,
                                                    const int32_t* __restrict__ unit0, int nb, int row_bits,
                                                    int32_t* __restrict__ ucount, int32_t* __restrict__ deg) {
    __shared__ int32_t tmp[4];
    const int t = threadIdx.x, lane = __lane_id();
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const Seg g = segs[tile_seg[blockIdx.x]];
    const int32_t ti = blockIdx.x - g.tile0;
    const int32_t j0 = ti * kTile, count = min(kTile, g.len - j0);
    const int32_t per = (count + 255) / 256 * 64;
    const int64_t row0 = (int64_t)g.bin << row_bits;
    int32_t mine = 0, cur = -1, held = 0;  // the row being counted (wave-uniform) and its keys so far
    for (int32_t i = w * per; i < min(count, (w + 1) * per); i += 64) {
        const bool in = i + lane < count;
        const int32_t j = in ? j0 + i + lane : 0;
        const K k = in ? keys[g.start + j] : (K)0;
        const bool f = in && (j == 0 || keys[g.start + j - 1] != k);
        const int32_t r = in ? (int32_t)(k >> nb) : -1;
        uint64_t rest = ballot64(f);
        mine += (int32_t)__popcll(rest);
        while (rest) {  // wave-uniform: one pass per row of the 64
            const int32_t row = __builtin_amdgcn_readlane(r, __builtin_ctzll(rest));
            const uint64_t same = rest & ballot64(r == row);
            rest &= ~same;
            if (row != cur) {
                if (held && lane == 0) atomicAdd(&deg[row0 + cur], held);
                cur = row;
                held = 0;
            }
            held += (int32_t)__popcll(same);
        }
    }
    if (held && lane == 0) atomicAdd(&deg[row0 + cur], held);
    if (lane == 0) tmp[w] = mine;
    __syncthreads();
    if (t == 0) ucount[unit0[g.bin] + ti] = tmp[0] + tmp[1] + tmp[2] + tmp[3];
}

// ---- the CSR ----------------------------------------------------------------

// base[u] = unique keys before unit u, and their total (one block)
__global__ void __launch_bounds__(1024) k_csr_unit_scan(const int32_t* __restrict__ ucount, int32_t* __restrict__ base,
                                                         int32_t* __restrict__ info) {
    __shared__ int32_t tmp[17];
    const int32_t units = info[kUnits];
    const int32_t per = (units + 1023) / 1024;
    const int32_t u0 = min((int32_t)threadIdx.x * per, units), u1 = min(u0 + per, units);
    int32_t s = 0;
#pragma unroll 8
    for (int32_t u = u0; u < u1; ++u) s += ucount[u];
    int32_t total;
    s = block_exclusive_sum<1024>(s, tmp, &total);
#pragma unroll 8
    for (int32_t u = u0; u < u1; ++u) {
        const int32_t c = ucount[u];
        base[u] = s;
        s += c;
    }
    if (threadIdx.x == 0) info[kTotal] = total;
}

// degree classes of all vertices and the largest degree
__global__ void __launch_bounds__(256) k_csr_classes(int64_t n, const int32_t* __restrict__ deg,
                                                      uint8_t* __restrict__ cls, int32_t* __restrict__ info) {
    __shared__ int32_t red[4];
    int32_t m = 0;
    for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < n; x += (int64_t)gridDim.x * 256) {
        const int32_t d = deg[x];
        cls[x] = (uint8_t)deg_class(d);
        m = d > m ? d : m;
    }
    m = wave_max(m);
    if (__lane_id() == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 0; i < 4; ++i) m = red[i] > m ? red[i] : m;
        if (m) atomicMax(&info[kMaxDeg], m);
    }
}

// One block per unit: its unique keys as CSR entries.  A window's keys are
// unique already; a tile of a larger one (keys in `big`) still holds runs.
template <typename K>
__global__ void __launch_bounds__(256) k_csr_emit(const int4* __restrict__ units, const Seg* __restrict__ segs,
                                                   const K* __restrict__ keys, const K* __restrict__ big,
                                                   const int32_t* __restrict__ ucount,
                                                   const int32_t* __restrict__ base, int nb, int row_bits,
                                                   const uint8_t* __restrict__ cls, int32_t* __restrict__ col,
                                                   int32_t* __restrict__ src, uint8_t* __restrict__ ncls) {
    __shared__ int32_t part[2][4];
    const int t = threadIdx.x;
    const int4 un = units[blockIdx.x];
    const int64_t o0 = base[blockIdx.x];
    const K vmask = ((K)1 << nb) - 1;
    const int64_t row0 = (int64_t)un.z << row_bits;
    auto put = [&](int64_t o, K k) {
        const int32_t v = (int32_t)(k & vmask);
        __builtin_nontemporal_store(v, col + o);  // the class table keeps the caches
        __builtin_nontemporal_store((int32_t)(row0 + (int64_t)(k >> nb)), src + o);
        __builtin_nontemporal_store(cls[v], ncls + o);
    };
    if (un.w < 0) {
        const int32_t cnt = ucount[blockIdx.x];
#pragma unroll 4
        for (int32_t j = t; j < cnt; j += 256) put(o0 + j, __builtin_nontemporal_load(keys + un.x + j));
        return;
    }
    const bool head = un.x == segs[un.w].start;
    int64_t o = o0;
    for (int32_t jb = 0; jb < un.y; jb += 256) {
        const int32_t j = jb + t;
        const K k = j < un.y ? big[un.x + j] : (K)0;
        const bool f = j < un.y && ((head && j == 0) || big[un.x + j - 1] != k);
        const uint64_t b = ballot64(f);
        int32_t* p = part[(jb >> 8) & 1];
        if (__lane_id() == 0) p[t >> 6] = (int32_t)__popcll(b);
        __syncthreads();
        int32_t pre = 0, tot = 0;
        for (int i = 0; i < 4; ++i) {
            pre += i < (t >> 6) ? p[i] : 0;
            tot += p[i];
        }
        if (f) put(o + pre + (int32_t)__popcll(b & lanes_below()), k);
        o += tot;
    }
}

template <typename Kern>
void raise_lds(Kern kernel, size_t bytes) {
    check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)bytes),
              "LDS size");
}

int64_t max_units(const CsrPlan& c, int64_t N) { return c.bins + N / kTile + 1; }
int64_t max_big_tiles(int64_t N) { return N > kWindowCap ? N / kTile + N / kWindowCap + 1 : 0; }
// info, start, unit0, tile0, concat, cursor, ucount, base and tile_seg in one allocation
int64_t small_ints(const CsrPlan& c, int64_t N) {
    return kInfoN + 4 * (c.bins + 1) + (c.W > kDigit ? c.bins : 0) + 2 * max_units(c, N) + max_big_tiles(N);
}

// K: a whole key, KW: a key inside its window.
template <typename K, typename KW>
int build_csr_t(const CsrPlan& c, int64_t n, int64_t P, const int32_t* src, const int32_t* dst, hipStream_t s,
                tc_graph_s* g) {
    const int64_t N = 2 * P;
    const bool two = c.W > kDigit;
    const int32_t cap = two || sizeof(KW) > 4 ? kWindowCap : 2 * kWindowCap;
    const int row_bits = c.nb - c.W;
    g->n = n;
    g->home = s;
    g->row_ptr = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(n + 1), s);
    g->deg = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(n > 0 ? n : 1), s);
    fill_i32(g->deg, 0, n, s);
    int32_t h[kInfoN] = {0, 0, 0, 0, 0, 0};
    if (N > 0) {
        DevBuf<KW> keys(N, s);
        DevBuf<int4> units(max_units(c, N), s);
        DevBuf<Seg> segs(max_big_tiles(N), s);
        DevBuf<int32_t> small(small_ints(c, N), s);
        int32_t* info = small.get();
        int32_t* start = info + kInfoN;
        int32_t* unit0 = start + c.bins + 1;
        int32_t* tile0 = unit0 + c.bins + 1;
        int32_t* concat = tile0 + c.bins + 1;
        int32_t* cursor = two ? concat + c.bins + 1 : nullptr;
        int32_t* ucount = concat + c.bins + 1 + (two ? c.bins : 0);
        int32_t* base = ucount + max_units(c, N);
        int32_t* tile_seg = base + max_units(c, N);
        fill_i32(info, 0, kInfoN, s);
        DevBuf<uint8_t> cls(n, s);
        {
            DevBuf<int32_t> binrows((size_t)c.ghist * c.bins, s), partrows((size_t)c.gpart * c.parts, s);
            const size_t hlds = sizeof(int32_t) * (size_t)(c.bins + c.parts);
            if (hlds > (64u << 10)) raise_lds(k_csr_hist, hlds);
            TC_LAUNCH("csr_hist", k_csr_hist, dim3(c.ghist), dim3(kHistThreads), hlds, s, src, dst, P, n,
                      c.nb - c.W, (int)c.bins, (int)c.parts, c.tiles, c.gpart, binrows.get(), partrows.get(),
                      info);
            TC_LAUNCH("csr_bins", k_csr_bins, dim3(ceil_div(c.bins, 256)), dim3(256), 0, s, (int)c.bins, c.ghist, cap,
                      (const int32_t*)binrows.get(), start, unit0, tile0, concat);
            int32_t* const four[4] = {start, unit0, tile0, concat};
            scan_exclusive_i32_each(four, 4, c.bins, s);
            TC_LAUNCH("csr_units", k_csr_units, dim3(ceil_div(c.bins, 256)), dim3(256), 0, s, (int)c.bins, cap,
                      (const int32_t*)start, (const int32_t*)unit0, (const int32_t*)tile0, (const int32_t*)concat,
                      cursor, units.get(), segs.get(), tile_seg, info);
            const int bpp = (int)(c.bins / c.parts);
            TC_LAUNCH("csr_part_base", k_csr_part_base, dim3((unsigned)c.parts), dim3(512), 0, s, c.gpart,
                      (int)c.parts, bpp, (const int32_t*)start, partrows.get());
            const K wmask = c.rest >= (int)(8 * sizeof(K)) ? ~(K)0 : (((K)1 << c.rest) - 1);
            const int shift1 = 2 * c.nb - c.b1;
            if (!two) {
                TC_LAUNCH("csr_part", (k_csr_part1<K, KW>), dim3(c.gpart), dim3(kPartThreads), 0, s, src, dst, P, n,
                          c.nb, shift1, wmask, (int)c.parts, c.tiles, (const int32_t*)partrows.get(), keys.get());
            } else {
                DevBuf<K> whole(N, s);
                TC_LAUNCH("csr_part", (k_csr_part1<K, K>), dim3(c.gpart), dim3(kPartThreads), 0, s, src, dst, P, n,
                          c.nb, shift1, ~(K)0, (int)c.parts, c.tiles, (const int32_t*)partrows.get(), whole.get());
                TC_LAUNCH("csr_part", (k_csr_part2<K, KW>), dim3((unsigned)(N / kPartKeys + c.parts)),
                          dim3(kPartThreads), 0, s, (const K*)whole.get(), (int)c.parts, bpp, c.rest, wmask,
                          (const int32_t*)start, cursor, keys.get());
            }
        }
        // windows left to the radix passes go where the larger windows' prefix was
        auto sort = [&](const char* name, auto kernel, int64_t blocks) {
            const size_t lds = sizeof(KW) * (size_t)cap + sizeof(int32_t) * (size_t)(sub_windows(cap / 1024) + 1);
            if (lds > (64u << 10)) raise_lds(kernel, lds);
            TC_LAUNCH(name, kernel, dim3((unsigned)blocks), dim3(1024), lds, s, keys.get(), (const int32_t*)start,
                      (const int32_t*)unit0, c.nb, c.rest, row_bits, concat, info + kListed, ucount, g->deg);
        };
        const int64_t some = std::min<int64_t>(c.bins, num_cus());
        if (cap == kWindowCap) {
            sort("csr_sort", k_csr_sort<8, false, KW>, c.bins);
            sort("csr_sort_radix", k_csr_sort<8, true, KW>, some);
        } else if constexpr (sizeof(KW) == 4) {
            sort("csr_sort", k_csr_sort<16, false, KW>, c.bins);
            sort("csr_sort_radix", k_csr_sort<16, true, KW>, some);
        }
        // row offsets, classes and the units' places; once more if windows above the cap came in between
        auto finish = [&] {
            scan_exclusive_i32(g->deg, g->row_ptr, n, s);
            const unsigned cg = std::max(1u, std::min(ceil_div(n, 256), 2048u));
            TC_LAUNCH("csr_classes", k_csr_classes, dim3(cg), dim3(256), 0, s, n, (const int32_t*)g->deg, cls.get(),
                      info);
            TC_LAUNCH("csr_unit_scan", k_csr_unit_scan, dim3(1), dim3(1024), 0, s, (const int32_t*)ucount,
                      base, info);
            check_hip(hipMemcpyAsync(h, info, sizeof(h), hipMemcpyDeviceToHost, s), "csr sizes");
            check_hip(hipStreamSynchronize(s), "sync");
        };
        finish();
        if (h[kBad]) return 1;
        DevBuf<KW> other;
        KW* big = keys.get();
        if (h[kBigTiles] > 0) {
            const int64_t tiles = h[kBigTiles];
            other.reset(N, s);
            KW* next = other.get();
            DevBuf<int32_t> hist((size_t)kRadix * tiles + 1, s);
            for (int shift = 0; shift < c.rest; shift += kDigit) {
                const int bits = std::min(kDigit, c.rest - shift);
                TC_LAUNCH("csr_big_hist", k_big_hist<KW>, dim3((unsigned)tiles), dim3(256), 0, s, (const KW*)big,
                          (const Seg*)segs.get(), (const int32_t*)tile_seg, shift, bits, hist.get());
                scan_exclusive_i32(hist.get(), hist.get(), kRadix * tiles, s);
                TC_LAUNCH("csr_big_scatter", k_big_scatter<KW>, dim3((unsigned)tiles), dim3(256), 0, s, (const KW*)big,
                          next, (const Seg*)segs.get(), (const int32_t*)tile_seg, shift, bits,
                          (const int32_t*)hist.get());
                std::swap(big, next);
            }
            TC_LAUNCH("csr_big_count", k_big_count<KW>, dim3((unsigned)tiles), dim3(256), 0, s, (const KW*)big,
                      (const Seg*)segs.get(), (const int32_t*)tile_seg, (const int32_t*)unit0, c.nb,
                      row_bits, ucount, g->deg);
            finish();
        }
        const int64_t total = h[kTotal];
        const size_t cap = (size_t)(total > 0 ? total : 1);
        g->m = total / 2;
        g->max_deg = h[kMaxDeg];
        g->col = (int32_t*)dev_alloc(sizeof(int32_t) * cap, s);
        g->src = (int32_t*)dev_alloc(sizeof(int32_t) * cap, s);
        if (total > 0) {
            g->ncls = (uint8_t*)dev_alloc((size_t)total, s);
            TC_LAUNCH("csr_emit", k_csr_emit<KW>, dim3((unsigned)h[kUnits]), dim3(256), 0, s,
                      (const int4*)units.get(), (const Seg*)segs.get(), (const KW*)keys.get(), (const KW*)big,
                      (const int32_t*)ucount, (const int32_t*)base, c.nb, row_bits,
                      (const uint8_t*)cls.get(), g->col, g->src, g->ncls);
        }
    } else {
        g->col = (int32_t*)dev_alloc(sizeof(int32_t), s);
        g->src = (int32_t*)dev_alloc(sizeof(int32_t), s);
        fill_i32(g->row_ptr, 0, n + 1, s);
    }
    check_hip(hipStreamSynchronize(s), "sync");
    return 0;
}

int key_bytes(int bits) { return bits <= 32 ? 4 : 8; }

}  // namespace

int64_t build_csr_bytes(int64_t n, int64_t num_pairs) {
    auto rb = region_bytes;
    const CsrPlan c = csr_plan(n, num_pairs);
    const int64_t N = 2 * num_pairs;
    int64_t b = rb(4 * (n + 1)) + rb(4 * n) + 2 * rb(4 * N) + rb(N) + scan_scratch_bytes(n);  // the CSR (2m <= N)
    if (N == 0) return b;
    const int64_t KW = key_bytes(c.rest), K = key_bytes(2 * c.nb);
    const bool two = c.W > kDigit;
    b += rb(KW * N) + rb(16 * max_units(c, N)) + rb((int64_t)sizeof(Seg) * max_big_tiles(N));
    b += rb(4 * small_ints(c, N)) + rb(n);
    // the partition's scratch, then (in its place) the passes over larger windows
    int64_t part = rb(4 * c.ghist * c.bins) + rb(4 * c.gpart * c.parts) +
                   std::max(two ? rb(K * N) : 0, scan_each_scratch_bytes(4, c.bins));
    int64_t big = 0;
    if (const int64_t t = max_big_tiles(N))
        big = rb(KW * N) + rb(4 * (kRadix * t + 1)) + scan_scratch_bytes(kRadix * t);
    return b + std::max(part, big);
}

int build_csr(int64_t n, int64_t num_pairs, const int32_t* src, const int32_t* dst, hipStream_t s, tc_graph_s* g) {
    PhaseScope ph("csr");
    const CsrPlan c = csr_plan(n, num_pairs);
    if (2 * c.nb <= 32) return build_csr_t<uint32_t, uint32_t>(c, n, num_pairs, src, dst, s, g);
    if (c.rest <= 32) return build_csr_t<uint64_t, uint32_t>(c, n, num_pairs, src, dst, s, g);
    return build_csr_t<uint64_t, uint64_t>(c, n, num_pairs, src, dst, s, g);
}

}  // namespace tc
