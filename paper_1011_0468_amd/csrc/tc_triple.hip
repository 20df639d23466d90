// Triple sampling (section 3.2, "Triple Sampling"; the Simple and Hybrid
// columns of Table 2) on the device.
//
// The candidate set U, in a fixed order: vertices u ascending; a vertex of
// the wedge kind contributes its pairs of neighbour positions (a, b), a < b,
// in colex order, the triple (N(u)[a], u, N(u)[b]); a vertex of the extension
// kind contributes, for each neighbour position a (v = N(u)[a]), each
// neighbour position j of v (w = N(v)[j]), the triple (u, v, w).  Simple:
// every vertex is of the wedge kind; hybrid: the extension kind iff
// deg^2 > m (the degree split of section 3.2).  A triangle appears once per
// wedge-kind and twice per extension-kind vertex, so a closed sample weighs
// 60 / (3 + its extension-kind vertices) and the weights of each triangle's
// appearances sum to 60: |U| * (sum of weights) / (60 s) estimates t.
//
//   1. per vertex, its number of triples: C(d, 2) (thread per vertex), or
//      the sum of its neighbours' degrees with, per list entry, the exclusive
//      prefix of that sum along the list (one block per list);
//   2. their exclusive prefix (int64) with a bucket index;
//   3. the sample numbers partitioned by the top byte of their hash (large
//      calls), so that samples close in U are drawn close in time;
//   4. one thread per sample: index r = high half of h * |U| (h a 64-bit
//      counter hash of the sample number), its vertex by a search of the
//      prefix, the pair by colex unranking or the list entry by binary
//      search over the entry prefix, and the closing edge by binary search in
//      the shorter sorted list.
#include "tc_internal.h"
#include "tc_device.h"
#include "tc_prefix.h"

#include <vector>

namespace tc {

namespace {

// SplitMix64's output function on the host (the device form is mix64)
uint64_t host_mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

__device__ __forceinline__ bool ext_kind(int hybrid, int64_t deg, int64_t m) { return hybrid && deg * deg > m; }

// per vertex of the wedge kind: C(d, 2); the vertices of the extension kind
// are appended to list, in any order (count at *listed), for k_tri_ext
__global__ void __launch_bounds__(256) k_tri_counts(int64_t n, const int32_t* __restrict__ deg, int64_t m, int hybrid,
                                                     int64_t* __restrict__ cnt, int32_t* __restrict__ list,
                                                     int32_t* __restrict__ listed) {
    const int lane = __lane_id();
    const int64_t n64 = (n + 63) / 64 * 64;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n64; x += (int64_t)gridDim.x * blockDim.x) {
        const int64_t d = x < n ? deg[x] : 0;
        const bool ext = ext_kind(hybrid, d, m);
        if (x < n && !ext) cnt[x] = d * (d - 1) / 2;
        const uint64_t b = ballot64(ext);
        if (!b) continue;
        int32_t at = 0;
        if (lane == 0) at = atomicAdd(listed, (int32_t)__popcll(b));
        at = __shfl(at, 0, 64);
        if (ext) list[at + __popcll(b & lanes_below())] = (int32_t)x;
    }
}

// extension-kind lists, one block per list: EP[e] = sum of deg(N(u)[i]) over
// the entries i before e in u's list, and cnt[u] = the whole sum (the vertices
// of a list are distinct: at most 2m, which fits 32 bits as the row offsets
// do).  A list is a serial chain of prefix sums, and the longest holds 10^5
// entries: 8192 of them per round, their gathers all in flight (64 per round, a
// wave per list, took 2.4 ms on R-MAT s22).  A wave takes rows of 64
// consecutive entries, so that a line is read and written by one access: 0.29
// ms, where 8 consecutive entries per thread and 64-bit sums took 0.51.
constexpr int kExtThreads = 1024, kExtItems = 8;
__global__ void __launch_bounds__(kExtThreads) k_tri_ext(const int32_t* __restrict__ list,
                                                          const int32_t* __restrict__ listed,
                                                          const int32_t* __restrict__ rp,
                                                          const int32_t* __restrict__ col,
                                                          const int32_t* __restrict__ deg, int64_t* __restrict__ cnt,
                                                          int32_t* __restrict__ EP) {
    constexpr int NW = kExtThreads / 64;
    __shared__ int32_t tmp[2][NW];
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    const int32_t lists = listed[0];
    int buf = 0;  // a round's sums are read while the next round's are written
    for (int32_t i = blockIdx.x; i < lists; i += gridDim.x) {  // block-uniform
        const int32_t u = list[i];
        const int32_t rs = rp[u], re = rp[u + 1];
        int32_t carry = 0;
        for (int64_t e0 = rs; e0 < re; e0 += kExtThreads * kExtItems) {
            const int64_t e = e0 + (int64_t)w * 64 * kExtItems + lane;
            int32_t v[kExtItems], pre[kExtItems], sum = 0;
#pragma unroll
            for (int k = 0; k < kExtItems; ++k) v[k] = e + 64 * k < re ? col[e + 64 * k] : -1;
#pragma unroll
            for (int k = 0; k < kExtItems; ++k) v[k] = v[k] >= 0 ? deg[v[k]] : 0;
#pragma unroll
            for (int k = 0; k < kExtItems; ++k) {
                const int32_t inc = wave_inclusive_sum(v[k]);
                pre[k] = sum + inc - v[k];
                sum += __builtin_amdgcn_readlane(inc, 63);
            }
            if (lane == 0) tmp[buf][w] = sum;
            __syncthreads();
            int32_t before = 0, total = 0;
            for (int q = 0; q < NW; ++q) {
                before += q < w ? tmp[buf][q] : 0;
                total += tmp[buf][q];
            }
#pragma unroll
            for (int k = 0; k < kExtItems; ++k)
                if (e + 64 * k < re) EP[e + 64 * k] = carry + before + pre[k];
            carry += total;
            buf ^= 1;
        }
        if (threadIdx.x == 0) cnt[u] = carry;
    }
}

// exclusive scan of int64 values: tiles of 2048 per block, then the tile sums
constexpr int kT64 = 256, kI64 = 8, kTile64 = kT64 * kI64;

__global__ void __launch_bounds__(kT64) k_scan64_tile(const int64_t* in, int64_t N, int64_t* out,
                                                       int64_t* __restrict__ bsum) {
    __shared__ int64_t tmp[kT64 / 64 + 1];
    const int64_t base = (int64_t)blockIdx.x * kTile64 + (int64_t)threadIdx.x * kI64;
    int64_t v[kI64];
    int64_t acc = 0;
#pragma unroll
    for (int i = 0; i < kI64; ++i) {
        v[i] = base + i < N ? in[base + i] : 0;
        acc += v[i];
    }
    int64_t total;
    int64_t pre = block_exclusive_sum<kT64>(acc, tmp, &total);
#pragma unroll
    for (int i = 0; i < kI64; ++i) {
        if (base + i < N) out[base + i] = pre;
        pre += v[i];
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// adds each tile's offset (boff[tile], nb > 1) and writes the total to out[N]
__global__ void k_scan64_fin(int64_t* out, int64_t N, const int64_t* __restrict__ boff, int64_t nb) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= N; i += (int64_t)gridDim.x * blockDim.x) {
        if (i == N) out[N] = nb > 1 ? boff[nb] : boff[0];
        else if (nb > 1) out[i] += boff[i / kTile64];
    }
}

}  // namespace

void scan64(const int64_t* in, int64_t* out, int64_t N, hipStream_t s) {
    const int64_t nb = N > 0 ? (N + kTile64 - 1) / kTile64 : 1;
    DevBuf<int64_t> bs(nb + 1, s);
    TC_LAUNCH("tri_scan", k_scan64_tile, dim3((unsigned)nb), dim3(kT64), 0, s, in, N, out, bs.get());
    if (nb > 1) scan64(bs.get(), bs.get(), nb, s);
    const int64_t g = std::min<int64_t>((N + 256) / 256, 65536);
    TC_LAUNCH("tri_scan", k_scan64_fin, dim3((unsigned)g), dim3(256), 0, s, out, N, (const int64_t*)bs.get(), nb);
}

namespace {

// the largest entry e of [lo, hi] with EP[e] <= k (EP[lo] <= k)
__device__ __forceinline__ int32_t last_entry(const int32_t* __restrict__ EP, int32_t lo, int32_t hi, int64_t k) {
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo + 1) >> 1);
        if (EP[mid] <= k) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Of every bucket of the index P that starts in the range of an extension-kind
// vertex u: the entry of u's list that holds the start (the largest e with
// EP[e] at or below it), so that a sample searches between two of them: 36
// entries apart instead of a list of 36000 on R-MAT s22 (2^25 samples:
// 4.00 -> 3.70 ms, and 0.07 for the index).
__global__ void __launch_bounds__(256) k_tri_ext_index(PrefixIndex<int64_t> P, const int32_t* __restrict__ rp,
                                                        const int32_t* __restrict__ EP, int64_t m,
                                                        int32_t* __restrict__ eidx) {
    const uint64_t total = (uint64_t)P.pre[P.n];
    if (total == 0) return;
    const Buckets bs(total, P.k);
    const int64_t B = (int64_t)1 << P.k;
    for (int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x; b < B; b += (int64_t)gridDim.x * 256) {
        const uint64_t r = bs.start((uint64_t)b);
        const int32_t u = P.idx[b];
        const int32_t us = rp[u], du = rp[u + 1] - us;
        if (r >= total || !ext_kind(1, du, m)) continue;
        eidx[b] = last_entry(EP, us, us + du - 1, (int64_t)r - P.pre[u]);
    }
}

// Sum of the closed samples' weights and closed samples, over
// the samples i0 + order[i] (order null: i0 + i), i < s.  Bound by random
// reads: per sample the index, the prefix, the two ends' ids and row starts
// and the steps of the closing search.  Each XCD takes a contiguous eighth, so
// that with the partition its samples' lists and prefixes stay in its L2.
__global__ void __launch_bounds__(256, 8) k_tri_sample(int64_t i0, int64_t s, const int32_t* __restrict__ order,
                                                     uint64_t salt, PrefixIndex<int64_t> P,
                                                     const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                     const int32_t* __restrict__ EP, const int32_t* __restrict__ eidx,
                                                     int64_t m, int hybrid, unsigned long long* __restrict__ acc) {
    const int64_t* CU = P.pre;
    const int64_t size = CU[P.n];
    const float scale = 1.0f / (float)P.n;
    int64_t wsum = 0, closed = 0;
    const int64_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, slots = gridDim.x >> 3;
    const int64_t i8 = s * xcd / 8, c8 = s * (xcd + 1) / 8 - i8;
    const int64_t end = size > 0 ? i8 + c8 * (slot + 1) / slots : 0;
    for (int64_t i = i8 + c8 * slot / slots + threadIdx.x; i < end; i += 256) {
        const int64_t r = (int64_t)__umul64hi(sample_hash(i0 + (order ? order[i] : i), salt), (uint64_t)size);
        const int32_t u = (int32_t)find_item(P, r);
        const int64_t k = r - CU[u];
        const int2 ur = two_at(rp + u);
        const int32_t us = ur.x, du = ur.y - us;
        int32_t x, y, z;
        bool cl;
        if (!ext_kind(hybrid, du, m)) {
            int64_t b = (int64_t)((1.0 + sqrt(1.0 + 8.0 * (double)k)) * 0.5);  // then made exact
            while (b > 1 && b * (b - 1) / 2 > k) --b;
            while ((b + 1) * b / 2 <= k) ++b;
            const int64_t a = k - b * (b - 1) / 2;
            x = col[us + a];
            y = u;
            z = col[us + b];
            cl = adjacent(rp, col, x, z, scale);
        } else {
            int32_t elo = us, ehi = us + du - 1;
            if (eidx) {
                const int64_t b = bucket_of((uint64_t)r, (uint64_t)size, P.k);
                if (b + 1 < (int64_t)1 << P.k) {
                    const int2 i = two_at(P.idx + b), e = two_at(eidx + b);
                    if (i.x == u) elo = e.x;
                    if (i.y == u) ehi = e.y;
                } else if (P.idx[b] == u) {
                    elo = eidx[b];
                }
            }
            elo = last_entry(EP, elo, ehi, k);
            const int32_t v = col[elo];
            x = u;
            y = v;
            z = col[rp[v] + (k - EP[elo])];
            // after the partition u's list is read by the samples around this
            // one and z's by none: 4.3 -> 4.0 ms for 2^25 on R-MAT s22
            cl = z != u && (order ? in_list(col, us, us + du, z, scale) : adjacent(rp, col, u, z, scale));
        }
        if (cl) {
            const auto ext = [&](int32_t w) { return (int)ext_kind(hybrid, rp[w + 1] - rp[w], m); };
            wsum += hybrid ? 60 / (3 + ext(x) + ext(y) + ext(z)) : 20;
            closed += 1;
        }
    }
    add_to_lines(wsum, closed, acc);
}

// Vertices from which, and vertices a sample up to which, the prefix gets an index,
// which costs a pass over the vertices.  Without and with it, uniform graphs: 2^22
// vertices with 10^4 samples 137 and 180 us, with 2^20 472 and 386; 2^23 with 2^20
// 527 and 465; R-MAT s24 with 2^20, simple, 697 and 825.
constexpr int64_t kIndexVertices = (int64_t)1 << 16;
constexpr int64_t kIndexVerticesPerSample = 8;

}  // namespace

void triple_sample(const tc_graph_s* g, int hybrid, int64_t num_samples, uint64_t seed, hipStream_t s,
                   int64_t* size, int64_t* wsum, int64_t* closed) {
    const int64_t n = g->n, m = g->m;
    *size = *wsum = *closed = 0;
    if (n == 0) return;
    // a search of few vertices is short by itself, and its index a launch more
    const int kb = n >= kIndexVertices && num_samples >= n / kIndexVerticesPerSample ? index_bits(n) : 0;
    DevBuf<int64_t> cnt(n + 1, s), CU(n + 1, s);
    DevBuf<int32_t> EP, list, idx, eidx, order, at;  // a call of few samples is also its allocations
    if (hybrid) {
        EP.reset(2 * m, s);
        list.reset(n, s);
    }
    if (kb) idx.reset((size_t)1 << kb, s);
    DevBuf<unsigned long long> acc(kAccLines * kAccStride + 1, s);  // the sums, then the length of list
    fill_i64(reinterpret_cast<int64_t*>(acc.get()), 0, kAccLines * kAccStride + 1, s);
    int32_t* listed = reinterpret_cast<int32_t*>(acc.get() + kAccLines * kAccStride);
    const unsigned vg = (unsigned)std::min<int64_t>((n + 255) / 256, 65536);
    TC_LAUNCH("tri_counts", k_tri_counts, dim3(vg), dim3(256), 0, s, n, (const int32_t*)g->deg, m, hybrid, cnt.get(),
              list.get(), listed);
    if (hybrid)
        TC_LAUNCH("tri_ext", k_tri_ext, dim3((unsigned)std::min<int64_t>(n, (int64_t)num_cus() * 2)),
                  dim3(kExtThreads), 0, s, (const int32_t*)list.get(), (const int32_t*)listed,
                  (const int32_t*)g->row_ptr, (const int32_t*)g->col, (const int32_t*)g->deg, cnt.get(), EP.get());
    scan64(cnt.get(), CU.get(), n, s);
    if (kb) bucket_index("tri_index", n, (const int64_t*)CU.get(), kb, idx.get(), s);
    const PrefixIndex<int64_t> P{CU.get(), kb ? idx.get() : nullptr, n, kb};
    // the lists' index pays for itself from about a sample per bucket
    const bool ext_index = hybrid && kb && num_samples >= (int64_t)1 << kb;
    if (ext_index) {
        eidx.reset((size_t)1 << kb, s);
        TC_LAUNCH("tri_index", k_tri_ext_index, dim3(ceil_div((int64_t)1 << kb, 256)), dim3(256), 0, s, P,
                  (const int32_t*)g->row_ptr, (const int32_t*)EP.get(), m, eidx.get());
    }
    const uint64_t salt = host_mix64(seed ^ 0x54435F545249504CULL);  // "TC_TRIPL"
    const bool part = samples_partitioned(num_samples, m);
    const int64_t chunk = part ? std::min(num_samples, kPartChunk) : num_samples;
    if (part) {
        order.reset(chunk, s);
        at.reset(kParts + 1, s);
    }
    for (int64_t i0 = 0; i0 < num_samples; i0 += chunk) {
        const int64_t c = std::min(chunk, num_samples - i0);
        if (part) partition_samples(i0, c, salt, HashParts{}, at.get(), order.get(), s);
        const unsigned sg = draw_blocks(c);
        TC_LAUNCH("tri_sample", k_tri_sample, dim3(sg), dim3(256), 0, s, i0, c,
                  part ? (const int32_t*)order.get() : (const int32_t*)nullptr, salt, P, (const int32_t*)g->row_ptr,
                  (const int32_t*)g->col, (const int32_t*)EP.get(), ext_index ? (const int32_t*)eidx.get() : nullptr,
                  m, hybrid, acc.get());
    }
    std::vector<int64_t> h(1 + kAccLines * kAccStride);
    check_hip(hipMemcpyAsync(h.data(), CU.get() + n, sizeof(int64_t), hipMemcpyDeviceToHost, s), "size");
    check_hip(hipMemcpyAsync(h.data() + 1, acc.get(), sizeof(int64_t) * kAccLines * kAccStride, hipMemcpyDeviceToHost,
                             s), "acc");
    check_hip(hipStreamSynchronize(s), "sync");
    *size = h[0];
    for (int l = 0; l < kAccLines; ++l) {
        *wsum += h[(size_t)(1 + l * kAccStride)];
        *closed += h[(size_t)(2 + l * kAccStride)];
    }
}

}  // namespace tc
