// Semi-streaming variant (section 5.2): three passes over the edges, with the
// adjacency lists in order.
//
//   pass 1: s1 = ceil(d m^(1/2) ln n) edges drawn uniformly with replacement
//           (the Lemma of section 5.2); their endpoints are the heavy
//           candidates, and those above the degree split (deg^2 > m) form H;
//   pass 2: s draws with replacement from U = L followed by X, where L holds
//           the wedges at the vertices outside H (vertices ascending, pairs of
//           neighbour positions in colex order) and X the pairs (h; e) of a
//           vertex of H and an edge (h ascending, edges in (v, w) order,
//           v < w); a draw asks for its closing edges: one for a wedge, two
//           for a pair whose vertex is not in its edge (none otherwise: never
//           closed);
//   pass 3: a draw is closed iff all its asked-for edges are in the graph.
//           The adjacency lists are in order, so an edge is looked up in one
//           of its ends' lists, and the draws come in the order of U, so that
//           the lists they read lie together: passes 2 and 3 are one kernel.
//
// Every triangle has exactly three closed elements in U, one per vertex, so
// |U| closed / (3 s) estimates t.  Draw i of pass 1 is upper edge
// floor(h m / 2^64), h = mix64(mix64(i) ^ mix64(seed ^ "TC_STRM1")); draw j of
// pass 2 is element floor(h' |U| / 2^64), h' = mix64(mix64(j) ^
// mix64(seed ^ "TC_STRM2")).
#include "tc_internal.h"
#include "tc_device.h"
#include "tc_prefix.h"

#include <algorithm>
#include <cmath>
#include <vector>

namespace tc {

namespace {

uint64_t host_mix(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

__device__ __forceinline__ int64_t hi_mul(uint64_t h, uint64_t size) { return (int64_t)__umul64hi(h, size); }

// Sum of v over the block (256 threads) added to *acc by one atomic.
__device__ __forceinline__ void block_add(int64_t v, unsigned long long* acc) {
    __shared__ int64_t red[4];
    v = wave_sum(v);
    __syncthreads();  // red may still be read by a previous call
    if (__lane_id() == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int64_t t = red[0] + red[1] + red[2] + red[3];
        if (t) atomicAdd(acc, (unsigned long long)t);
    }
}

// up[u] = neighbours of u above u (sorted list: the first position holding an id > u)
__global__ void k_up_deg(int64_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                         int32_t* __restrict__ up) {
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
        int32_t lo = rp[u], hi = rp[u + 1];
        const int32_t end = hi;
        while (lo < hi) {
            const int32_t mid = lo + ((hi - lo) >> 1);
            if (col[mid] <= (int32_t)u) lo = mid + 1;
            else hi = mid;
        }
        up[u] = end - lo;
    }
}

// (u, v) of upper edge r (P: the prefix of the neighbours above each vertex)
__device__ __forceinline__ void upper_edge(const PrefixIndex<int32_t>& P, const int32_t* __restrict__ rp,
                                           const int32_t* __restrict__ col, int64_t r, int32_t& u, int32_t& v) {
    const int64_t x = find_item(P, r);
    u = (int32_t)x;
    v = col[rp[x + 1] - (P.pre[x + 1] - (int32_t)r)];  // its upper entries end the list
}

// pass 1: the endpoints of s1 drawn edges
__global__ void k_stream_draw_edges(int64_t s1, uint64_t salt, int64_t m, const int32_t* __restrict__ rp,
                                    const int32_t* __restrict__ col, PrefixIndex<int32_t> up,
                                    uint8_t* __restrict__ cand) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < s1; i += (int64_t)gridDim.x * blockDim.x) {
        int32_t u, v;
        upper_edge(up, rp, col, hi_mul(mix64(mix64((uint64_t)i) ^ salt), (uint64_t)m), u, v);
        cand[u] = 1;
        cand[v] = 1;
    }
}

// H flags (candidates above the split) and the wedge count of every vertex
// outside H; *found += candidates
__global__ void k_stream_classify(int64_t n, int64_t m, const uint8_t* __restrict__ cand,
                                  const int32_t* __restrict__ deg, int32_t* __restrict__ hf,
                                  int64_t* __restrict__ lc, unsigned long long* __restrict__ found) {
    int64_t nc = 0;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x) {
        const int64_t d = deg[x];
        const bool c = cand[x] != 0;
        const bool h = c && d * d > m;  // the degree split of section 3.2 (c = 1)
        nc += c;
        hf[x] = h;
        lc[x] = h ? 0 : d * (d - 1) / 2;
    }
    block_add(nc, found);
}

__global__ void k_stream_hlist(int64_t n, const int32_t* __restrict__ hf, const int32_t* __restrict__ hpos,
                               int32_t* __restrict__ hlist) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x)
        if (hf[x]) hlist[hpos[x]] = (int32_t)x;
}

// Parts of the draws.  The wedges (elements below L) come first, in the order of
// U; the pairs by the position of their edge, whose lower end's list the first
// lookup reads, in as many of the 256 parts as are left.
struct StreamParts {
    const int64_t* Lp;    // |L|
    const int32_t* Hp;    // |H|
    int64_t m;
    int64_t L;            // from here on set by load()
    double scale, inv_m;  // parts per element, edges per element
    int32_t first;        // the first part of the pairs
    __device__ __forceinline__ void load() {
        L = *Lp;
        const int64_t size = L + (int64_t)*Hp * m;
        scale = size > 0 ? (double)kParts / (double)size : 0.0;
        inv_m = 1.0 / (double)m;
        first = L > 0 ? wedge_part(L - 1) + 1 : 0;
    }
    __device__ __forceinline__ int64_t size() const { return L + (int64_t)*Hp * m; }
    __device__ __forceinline__ int32_t wedge_part(int64_t r) const {
        const int32_t p = (int32_t)((double)r * scale);
        return p < kParts - 1 ? p : kParts - 1;
    }
    __device__ __forceinline__ int32_t operator()(uint64_t hash) const {
        const int64_t r = hi_mul(hash, (uint64_t)size());
        if (r < L) return wedge_part(r);
        const double x = (double)(r - L) * inv_m;
        const int32_t p = first + (int32_t)((x - floor(x)) * (double)(kParts - first));
        return p < kParts - 1 ? p : kParts - 1;
    }
};

// Passes 2 and 3: draws i0 + order[i] (order null: i0 + i), i < s; words 0 and 1
// of the lines of acc += closed draws and closing-edge lookups.  Bound by random
// reads: the element's prefix and list entries and the lists searched.  Each
// XCD takes a contiguous eighth of the partitioned wedges, then one of the
// pairs, so that the lists of the wedges' vertices and of the lower ends of the
// pairs' edges stay in its L2; the second lookup of a pair, which is anywhere in
// the graph, is left out if the first fails.  R-MAT s22, 2^24 draws: 1.62 ms and
// 47 M L2 misses; with the pairs in the order of U, where the heavy vertex's
// list is local and the edge is not, 2.1; as a table of the lookups filled by
// random compare-and-swaps, an edge pass that marks it and a pass that counts,
// 4.0.
__global__ void __launch_bounds__(256, 8) k_stream_draws(int64_t i0, int64_t s, const int32_t* __restrict__ order,
                                                       const int32_t* __restrict__ at, StreamParts parts,
                                                       uint64_t salt, int64_t m, const int32_t* __restrict__ rp,
                                                       const int32_t* __restrict__ col, PrefixIndex<int32_t> up,
                                                       PrefixIndex<int64_t> light, const int32_t* __restrict__ hlist,
                                                       unsigned long long* __restrict__ acc) {
    parts.load();
    const int64_t L = parts.L, size = parts.size();
    const float scale = 1.0f / (float)light.n;
    int64_t closed = 0, queries = 0;
    const int64_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, slots = gridDim.x >> 3;
    const int64_t wedges = order && parts.first > 0 ? at[parts.first - 1] : 0, pairs = s - wedges;
    const int64_t w0 = wedges * xcd / 8, p0 = wedges + pairs * xcd / 8;  // this XCD's of either kind
    const int64_t wc = wedges * (xcd + 1) / 8 - w0, pc = wedges + pairs * (xcd + 1) / 8 - p0;
    const int64_t end = size > 0 ? (wc + pc) * (slot + 1) / slots : 0;
    for (int64_t j = (wc + pc) * slot / slots + threadIdx.x; j < end; j += 256) {
        const int64_t i = j < wc ? w0 + j : p0 + (j - wc);
        const int64_t r = hi_mul(sample_hash(i0 + (order ? order[i] : i), salt), (uint64_t)size);
        if (r < L) {  // wedge k of light vertex u: pair (a, b) of colex order
            const int64_t u = find_item(light, r);
            const int64_t k = r - light.pre[u];
            int64_t b = (int64_t)((1.0 + sqrt(1.0 + 8.0 * (double)k)) * 0.5);  // then made exact
            while (b > 1 && b * (b - 1) / 2 > k) --b;
            while ((b + 1) * b / 2 <= k) ++b;
            const int64_t a = k - b * (b - 1) / 2;
            queries += 1;
            closed += adjacent(rp, col, col[rp[u] + a], col[rp[u] + b], scale);
        } else {  // the pair of heavy vertex h and upper edge (v, w)
            const int64_t qq = r - L;
            const int32_t h = hlist[qq / m];
            int32_t v, w;
            upper_edge(up, rp, col, qq % m, v, w);
            if (h == v || h == w) continue;  // never closed, no lookups
            queries += 2;
            const int2 vr = two_at(rp + v);
            closed += in_list(col, vr.x, vr.y, h, scale) && adjacent(rp, col, w, h, scale);
        }
    }
    add_to_lines(closed, queries, acc);
}

unsigned grid(int64_t N, int64_t cap = 65536) {
    int64_t b = (N + 255) / 256;
    if (b > cap) b = cap;
    return (unsigned)(b > 0 ? b : 1);
}

// kernels that reduce into one counter: a few resident rounds of blocks, so
// that the counter takes about a thousand atomics
constexpr int64_t kReduceBlocks = 1024;

}  // namespace

int64_t stream_draws(int64_t n, int64_t m, double d) {
    if (n < 2 || m < 1) return 0;
    return (int64_t)std::ceil(d * std::sqrt((double)m) * std::log((double)n));
}

void stream_estimate(const tc_graph_s* g, double d, int64_t s, uint64_t seed, hipStream_t st, tc_stream_result* out) {
    const int64_t n = g->n, m = g->m;
    tc_stream_result r{};
    r.m = m;
    r.draws1 = stream_draws(n, m, d);
    if (n < 2 || m < 1) {
        *out = r;
        return;
    }
    PhaseScope ph("stream");
    // the upper entries' prefix: edge r of the stream
    DevBuf<int32_t> upre(n + 1, st);
    TC_LAUNCH("stream_up", k_up_deg, dim3(grid(n)), dim3(256), 0, st, n, (const int32_t*)g->row_ptr,
              (const int32_t*)g->col, upre.get());
    scan_exclusive_i32(upre.get(), upre.get(), n, st);
    // bucket indexes of the two prefixes that draws are searched in
    const int k = index_bits(n);
    const int64_t B = (int64_t)1 << k;
    DevBuf<int32_t> up_idx(B, st), light_idx(B, st);
    bucket_index("stream_index", n, (const int32_t*)upre.get(), k, up_idx.get(), st);
    const PrefixIndex<int32_t> up{upre.get(), up_idx.get(), n, k};
    // pass 1
    DevBuf<uint8_t> cand(n, st);
    fill_u8(cand.get(), 0, n, st);
    const uint64_t salt1 = host_mix(seed ^ 0x54435F5354524D31ULL);  // "TC_STRM1"
    if (r.draws1 > 0)
        TC_LAUNCH("stream_pass1", k_stream_draw_edges, dim3(grid(r.draws1)), dim3(256), 0, st, r.draws1, salt1, m,
                  (const int32_t*)g->row_ptr, (const int32_t*)g->col, up, cand.get());
    DevBuf<int32_t> hf(n + 1, st), hpos(n + 1, st);
    DevBuf<int64_t> lc(n + 1, st), lpre(n + 1, st);
    DevBuf<unsigned long long> acc(kAccLines * kAccStride + 1, st);  // the draws' sums, then the candidates
    fill_i64(reinterpret_cast<int64_t*>(acc.get()), 0, kAccLines * kAccStride + 1, st);
    TC_LAUNCH("stream_classify", k_stream_classify, dim3(grid(n, kReduceBlocks)), dim3(256), 0, st, n, m,
              (const uint8_t*)cand.get(), (const int32_t*)g->deg, hf.get(), lc.get(),
              acc.get() + kAccLines * kAccStride);
    scan_exclusive_i32(hf.get(), hpos.get(), n, st);
    scan64(lc.get(), lpre.get(), n, st);
    DevBuf<int32_t> hlist(n, st);
    TC_LAUNCH("stream_hlist", k_stream_hlist, dim3(grid(n)), dim3(256), 0, st, n, (const int32_t*)hf.get(),
              (const int32_t*)hpos.get(), hlist.get());
    bucket_index("stream_index", n, (const int64_t*)lpre.get(), k, light_idx.get(), st);
    const PrefixIndex<int64_t> light{lpre.get(), light_idx.get(), n, k};
    // passes 2 and 3
    const uint64_t salt2 = host_mix(seed ^ 0x54435F5354524D32ULL);  // "TC_STRM2"
    const bool part = samples_partitioned(s, m);
    const int64_t chunk = part ? std::min(s, kPartChunk) : s;
    DevBuf<int32_t> order(part ? chunk : 0, st), at(part ? kParts + 1 : 0, st);
    const StreamParts parts{lpre.get() + n, hpos.get() + n, m, 0, 0.0, 0.0, 0};
    for (int64_t i0 = 0; i0 < s; i0 += chunk) {
        const int64_t c = std::min(chunk, s - i0);
        if (part) partition_samples(i0, c, salt2, parts, at.get(), order.get(), st);
        const unsigned sg = draw_blocks(c);
        TC_LAUNCH("stream_draws", k_stream_draws, dim3(sg), dim3(256), 0, st, i0, c,
                  part ? (const int32_t*)order.get() : (const int32_t*)nullptr, (const int32_t*)at.get(), parts,
                  salt2, m, (const int32_t*)g->row_ptr, (const int32_t*)g->col, up, light,
                  (const int32_t*)hlist.get(), acc.get());
    }
    std::vector<int64_t> sums(kAccLines * kAccStride + 1);
    int64_t L = 0;
    int32_t H = 0;
    check_hip(hipMemcpyAsync(sums.data(), acc.get(), sizeof(int64_t) * sums.size(), hipMemcpyDeviceToHost, st),
              "stream counts");
    check_hip(hipMemcpyAsync(&H, hpos.get() + n, sizeof(int32_t), hipMemcpyDeviceToHost, st), "heavy count");
    check_hip(hipMemcpyAsync(&L, lpre.get() + n, sizeof(int64_t), hipMemcpyDeviceToHost, st), "light size");
    check_hip(hipStreamSynchronize(st), "sync");
    r.candidates = sums[kAccLines * kAccStride];
    r.heavy = H;
    r.light_size = L;
    r.size = L + (int64_t)H * m;
    for (int l = 0; l < kAccLines; ++l) {
        r.closed += sums[l * kAccStride];
        r.queries += sums[l * kAccStride + 1];
    }
    if (s > 0) {
        volatile double num = (double)r.size * (double)r.closed;
        volatile double den = 3.0 * (double)s;
        r.estimate = num / den;
    }
    *out = r;
}

}  // namespace tc

using namespace tc;

extern "C" tc_status tc_stream_estimate(tc_graph g, double d, int64_t num_samples, uint64_t seed, void* stream,
                                        tc_stream_result* out) {
    try {
        set_last_error("");
        if (!g || !out) fail(TC_ERR_INVALID, "graph or output is NULL");
        if (!std::isfinite(d) || d <= 0.0) fail(TC_ERR_INVALID, "d must be finite and > 0");
        if (num_samples < 0) fail(TC_ERR_INVALID, "num_samples must be >= 0");
        if (num_samples > ((int64_t)1 << 28)) fail(TC_ERR_OVERFLOW, "num_samples exceeds 2^28");
        const int64_t s1 = stream_draws(g->n, g->m, d);
        if (s1 > ((int64_t)1 << 40)) fail(TC_ERR_OVERFLOW, "pass-1 draws exceed 2^40");
        tc_stream_result r;
        stream_estimate(g, d, num_samples, seed, (hipStream_t)stream, &r);
        *out = r;
        profile_collect();
        return TC_OK;
    } catch (const Error& e) {
        set_last_error(e.msg);
        return e.status;
    } catch (const std::exception& e) {
        set_last_error(e.what());
        return TC_ERR_DEVICE;
    } catch (...) {
        set_last_error("unknown error");
        return TC_ERR_DEVICE;
    }
}
