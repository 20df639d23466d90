// Edge sparsification (section 3.1): every undirected edge is kept
// independently with probability p.  The coin is a counter-based hash of the
// edge's (min, max) ids and the seed, so both CSR directions of an edge, and
// any other implementation of the same hash, take the same decision.
//
// Layout: one keep bit per CSR entry, packed 64 to a word (a wave's ballot),
// plus the popcount of each word; an exclusive scan of the popcounts gives the
// compacted position of every kept entry and of every row start.
#include "tc_internal.h"
#include "tc_device.h"

namespace tc {

uint64_t keep_threshold(double p) { return (uint64_t)(p * 9007199254740992.0); }

uint64_t sample_salt(uint64_t seed) {
    uint64_t z = seed ^ 0x54435F53414D504Cull;  // "TC_SAMPL"
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

namespace {

__global__ void __launch_bounds__(256) k_keep_bits(const int32_t* __restrict__ src, const int32_t* __restrict__ col,
                                                    int64_t E2, uint64_t salt, uint64_t thr,
                                                    uint64_t* __restrict__ bits, int32_t* __restrict__ wcnt) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x; e0 < E2; e0 += stride) {
        const int64_t e = e0 + threadIdx.x;
        bool keep = false;
        if (e < E2) keep = edge_kept((uint32_t)src[e], (uint32_t)col[e], salt, thr);
        const uint64_t b = ballot64(keep);
        if (__lane_id() == 0 && e < E2) {
            bits[e >> 6] = b;
            wcnt[e >> 6] = __popcll(b);
        }
    }
}

__device__ __forceinline__ int32_t kept_before(int64_t e, int64_t E2, const uint64_t* bits, const int32_t* wpre) {
    if (e >= E2) return wpre[(E2 + 63) >> 6];
    const uint64_t w = bits[e >> 6];
    const int r = (int)(e & 63);
    const uint64_t below = r == 0 ? 0ull : (w & (~0ull >> (64 - r)));
    return wpre[e >> 6] + __popcll(below);
}

__global__ void k_rows_at(const int32_t* __restrict__ row_ptr, int64_t n, int64_t E2, const uint64_t* __restrict__ bits,
                          const int32_t* __restrict__ wpre, int32_t* __restrict__ rp_out, int32_t* __restrict__ deg_out) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x <= n; x += (int64_t)gridDim.x * blockDim.x) {
        const int32_t a = kept_before(row_ptr[x], E2, bits, wpre);
        if (rp_out) rp_out[x] = a;
        if (deg_out && x < n) deg_out[x] = kept_before(row_ptr[x + 1], E2, bits, wpre) - a;
    }
}

// Each wave takes 4 words of keep bits (256 entries) per step: the words and
// their prefixes first, then the kept entries' loads, then the stores, so the
// latencies of the 4 words overlap.
__global__ void __launch_bounds__(256) k_compact(const int32_t* __restrict__ col, const int32_t* __restrict__ src,
                                                  int64_t E2, const int32_t* __restrict__ E2_dev,
                                                  const uint64_t* __restrict__ bits, const int32_t* __restrict__ wpre,
                                                  int32_t* __restrict__ col_out, int32_t* __restrict__ src_out) {
    const int lane = __lane_id();
    const int64_t valid = E2_dev ? (int64_t)E2_dev[0] : E2;  // entries past it have no bits set
    const int64_t NW = (valid + 63) / 64;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const int64_t wave = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t w0 = wave * 4; w0 < NW; w0 += nwaves * 4) {
        uint64_t bw[4];
        int32_t pre[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool ok = w0 + k < NW;
            bw[k] = ok ? bits[w0 + k] : 0ull;
            pre[k] = ok ? wpre[w0 + k] : 0;
        }
        int32_t cv[4], sv[4];
        bool on[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            on[k] = (bw[k] >> lane) & 1ull;  // set bits lie below valid <= E2
            const int64_t e = (w0 + k) * 64 + lane;
            cv[k] = on[k] ? col[e] : 0;
            sv[k] = (on[k] && src_out) ? src[e] : 0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (on[k]) {
                const int32_t p = pre[k] + __popcll(bw[k] & below);
                col_out[p] = cv[k];
                if (src_out) src_out[p] = sv[k];
            }
        }
    }
}

// Keep bits with the kept entries staged: one wave per range of kStageWords
// words (64 entries each).  The wave writes the range's keep words and their
// popcounts, and packs the range's kept entries, in order, at the start of
// the range's region of the staging arrays (entries [64 w0, 64 w0 + kept)),
// with full-width stores.  Once the word counts are scanned, k_move_staged
// copies each range's packed entries to their place, so no entry of the
// graph is read twice and no store is one lane wide.
constexpr int kStageWords = 8;

__device__ __forceinline__ void wave_lds_order_s() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ void __launch_bounds__(256) k_keep_stage(const int32_t* __restrict__ src, const int32_t* __restrict__ col,
                                                     int64_t E2, uint64_t salt, uint64_t thr,
                                                     uint64_t* __restrict__ bits, int32_t* __restrict__ wcnt,
                                                     int32_t* __restrict__ st_col, int32_t* __restrict__ st_src) {
    constexpr int RW = kStageWords;
    __shared__ int32_t pack[4][2][RW * 64];
    const int lane = __lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t* pc = pack[wv][0];
    int32_t* ps = pack[wv][1];
    const uint64_t below = lanes_below();
    const int64_t NW = (E2 + 63) / 64;
    const int64_t nR = (NW + RW - 1) / RW;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t r = (int64_t)blockIdx.x * 4 + wv; r < nR; r += nwaves) {
        const int64_t w0 = r * RW;
        int32_t uu[RW], vv[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int64_t e = (w0 + i) * 64 + lane;
            const bool in = e < E2;
            uu[i] = in ? src[e] : 0;
            vv[i] = in ? col[e] : 0;
        }
        int32_t cnt = 0;
        uint64_t mine = 0;  // lane i < RW: word w0 + i
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int64_t e = (w0 + i) * 64 + lane;
            const bool keep = e < E2 && edge_kept((uint32_t)uu[i], (uint32_t)vv[i], salt, thr);
            const uint64_t b = ballot64(keep);
            if (lane == i) mine = b;
            if (keep) {
                const int32_t q = cnt + (int32_t)__popcll(b & below);
                pc[q] = vv[i];
                ps[q] = uu[i];
            }
            cnt += (int32_t)__popcll(b);
        }
        if (lane < RW && w0 + lane < NW) {
            bits[w0 + lane] = mine;
            wcnt[w0 + lane] = (int32_t)__popcll(mine);
        }
        wave_lds_order_s();
        for (int32_t q = lane; q < cnt; q += 64) {
            st_col[w0 * 64 + q] = pc[q];
            st_src[w0 * 64 + q] = ps[q];
        }
        wave_lds_order_s();  // read before the next range packs
    }
}

// Each range's staged entries to positions wpre[w0] .. (wpre: exclusive scan
// of the word counts, NW + 1 entries).
__global__ void __launch_bounds__(256) k_move_staged(int64_t E2, const int32_t* __restrict__ wpre,
                                                      const int32_t* __restrict__ st_col,
                                                      const int32_t* __restrict__ st_src, int32_t* __restrict__ col_out,
                                                      int32_t* __restrict__ src_out) {
    constexpr int RW = kStageWords;
    const int lane = __lane_id();
    const int64_t NW = (E2 + 63) / 64;
    const int64_t nR = (NW + RW - 1) / RW;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t r = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); r < nR; r += nwaves) {
        const int64_t w0 = r * RW;
        const int64_t w1 = w0 + RW < NW ? w0 + RW : NW;
        const int32_t a = wpre[w0];
        const int32_t cnt = wpre[w1] - a;
        for (int32_t q = lane; q < cnt; q += 64) {
            col_out[a + q] = st_col[w0 * 64 + q];
            src_out[a + q] = st_src[w0 * 64 + q];
        }
    }
}

// ---------------------------------------------------------------------------
// unions of samples (batched seeds, fused requests)
// ---------------------------------------------------------------------------

// Copy k of the replicated entry space holds g's entries at union positions
// k * 64 NWp + e (e < E2; the rest of its words are never kept), so that no
// word of keep bits straddles two copies.  A block takes kKeepWords words of g,
// a wave kKeepWords / 4 of them, for every copy: the entries are read once and
// the seed-independent first mix of each edge's key is computed once (the coin
// is mix64(mix64(key) ^ salt) >> 11 < thr, section 3.1's coin as the
// single-sample kernels compute it).  Bound by the six 32-bit multiplications
// left per coin: 2.1 G coins (2^25 entries, 64 copies) in 1.32 ms are 9.8 T
// multiplications/s, what a quarter of the lanes' rate gives; with eight of
// them, a scalar load of the salt and a branch per coin it took 1.40 to 1.49.
// 64 copies at a time pass through LDS, where each copy's words lie together,
// so that one store writes a line of the bits.
constexpr int kKeepWords = 16;

__global__ void __launch_bounds__(256) k_keep_rep(const int32_t* __restrict__ src, const int32_t* __restrict__ col,
                                                   int64_t E2, int64_t NWp, int32_t K,
                                                   const uint64_t* __restrict__ salts, uint64_t thr,
                                                   uint64_t* __restrict__ bits, int32_t* __restrict__ wcnt) {
    constexpr int PER = kKeepWords / 4;
    __shared__ uint64_t tile[64][kKeepWords + 1];
    const int lane = __lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t groups = (NWp + kKeepWords - 1) / kKeepWords;
    for (int64_t gr = blockIdx.x; gr < groups; gr += gridDim.x) {  // block-uniform
        uint64_t base[PER];
        uint64_t in[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t e = (gr * kKeepWords + wid * PER + i) * 64 + lane;
            in[i] = ballot64(e < E2);
            base[i] = e < E2 ? mix_fold(edge_mix((uint32_t)src[e], (uint32_t)col[e])) : 0;
        }
        for (int32_t k0 = 0; k0 < K; k0 += 64) {
            const int kc = K - k0 < 64 ? K - k0 : 64;
            const uint64_t mysalt = lane < kc ? mix_fold(salts[k0 + lane]) : 0;
            uint64_t mine[PER] = {};
            for (int k = 0; k < kc; ++k) {
                const uint64_t salt =
                    ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mysalt >> 32), k) << 32) |
                    (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mysalt, k);
                bool below[PER], equal = false;
#pragma unroll
                for (int i = 0; i < PER; ++i) equal |= folded_top(base[i] ^ salt, thr, &below[i]);
                if (__builtin_expect(ballot64(equal) != 0, 0)) {
#pragma unroll
                    for (int i = 0; i < PER; ++i) below[i] = folded_below_exact(base[i] ^ salt, thr);
                }
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const uint64_t b = ballot64(below[i]) & in[i];
                    mine[i] = lane == k ? b : mine[i];
                }
            }
#pragma unroll
            for (int i = 0; i < PER; ++i) tile[lane][wid * PER + i] = mine[i];
            __syncthreads();
            for (int q = threadIdx.x; q < kc * kKeepWords; q += 256) {
                const int k = q / kKeepWords, i = q % kKeepWords;
                const int64_t w = gr * kKeepWords + i;
                if (w < NWp) {
                    const uint64_t b = tile[k][i];
                    bits[(int64_t)(k0 + k) * NWp + w] = b;
                    wcnt[(int64_t)(k0 + k) * NWp + w] = __popcll(b);
                }
            }
            __syncthreads();
        }
    }
}

// Row offsets and degrees of the union of samples in the padded layout: union
// vertex k * npad + x is vertex x of copy k (x >= n: isolated padding).  Per
// word of 64 of them, which lie in one copy: the bits and the number of those
// of degree min_deg and more, and of those of lower degree above 0.  A wave per
// word, where a row's end is the next lane's start (64 seeds of Chung-Lu 2^20 at
// p = 0.05: 0.61 -> 0.49 ms against a thread per vertex and a pass of its own for
// the bits).
__global__ void __launch_bounds__(256) k_rows_rep(const int32_t* __restrict__ row_ptr, int64_t n, int64_t npad,
                                                   int64_t E2, int64_t NWp, int32_t K, int min_deg,
                                                   const uint64_t* __restrict__ bits, const int32_t* __restrict__ wpre,
                                                   int32_t* __restrict__ rp_out, int32_t* __restrict__ deg_out,
                                                   uint64_t* __restrict__ nzb, int32_t* __restrict__ nzc,
                                                   uint64_t* __restrict__ oneb, int32_t* __restrict__ onec) {
    const int lane = __lane_id();
    const uint32_t wpc = (uint32_t)(npad / 64), NV = wpc * (uint32_t)K;  // words per copy, in all
    const int64_t E2U = (int64_t)K * NWp * 64;
    if (blockIdx.x == 0 && threadIdx.x == 0) rp_out[(int64_t)NV * 64] = wpre[K * NWp];
    for (uint32_t w = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); w < NV; w += gridDim.x * 4) {
        const uint32_t k = w / wpc;
        const int64_t x = (int64_t)(w - k * wpc) * 64 + lane;
        const int64_t base = k * NWp * 64;
        const int32_t a = kept_before(base + (x < n ? row_ptr[x] : E2), E2U, bits, wpre);
        int32_t e = __shfl_down(a, 1, 64);
        if (lane == 63) e = kept_before(base + (x < n ? row_ptr[x + 1] : E2), E2U, bits, wpre);
        const int32_t d = e - a;
        const int64_t xu = (int64_t)w * 64 + lane;
        rp_out[xu] = a;
        deg_out[xu] = d;
        const uint64_t b = ballot64(d >= min_deg), o = ballot64(d > 0 && d < min_deg);
        if (lane == 0) {
            nzb[w] = b;
            nzc[w] = __popcll(b);
            oneb[w] = o;
            onec[w] = __popcll(o);
        }
    }
}

// A word of 64 union vertices' table entry (see k_nz_table): their bits, and
// what the count of bits below the word starts from.
struct NzWord {
    uint64_t bits;
    int32_t base;
    __device__ __forceinline__ NzWord(const int4* __restrict__ table, int64_t x) {
        const int4 t = table[x >> 6];
        bits = ((uint64_t)(uint32_t)t.y << 32) | (uint32_t)t.x;
        base = t.z;
    }
    __device__ __forceinline__ bool has(int64_t x) const { return (bits >> (x & 63)) & 1ull; }
    __device__ __forceinline__ int32_t rank(int64_t x) const {
        const int r = (int)(x & 63);
        return base + __popcll(r == 0 ? 0ull : (bits & (~0ull >> (64 - r))));
    }
};

// Orders one wave's LDS accesses (a wave's LDS operations complete in issue
// order; only the compiler must not move accesses across).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Words of g per range of k_compact_rep
constexpr int kRepWords = 8;

// Kept entries of the replicated space, written with the union's final ids
// (nzt's rank of the padded layout's id).  The rows of dropped vertices of
// degree 1 (one entry each, onet) are left out, and the entries that point to
// one get the first unused id of their component (spare[k]), whose degree 0
// ranks below every vertex, as theirs did below the row's.  One wave per range of kRepWords words
// of g: the range's entries are read once and held in registers, and for
// every copy the kept entries of the whole range, which are consecutive in
// that copy's output, are packed in LDS, relabelled by full-width table
// gathers and written with full-width stores (one store per 64 kept entries
// instead of one per word and copy).  The copies' keep words and prefixes
// are loaded 64 at a time (8 copies x 8 words, one per lane) and taken with
// readlane.
__global__ void __launch_bounds__(256) k_compact_rep(const int32_t* __restrict__ col, const int32_t* __restrict__ src,
                                                      int64_t E2, int64_t NWp, int32_t K, int64_t npad,
                                                      const uint64_t* __restrict__ bits,
                                                      const int32_t* __restrict__ wpre, const int4* __restrict__ nzt,
                                                      const int4* __restrict__ onet, const int32_t* __restrict__ spare,
                                                      int32_t* __restrict__ col_out, int32_t* __restrict__ src_out) {
    constexpr int RW = kRepWords, CPL = 64 / RW;  // words per range, copies per load
    __shared__ int32_t pack[4][2][RW * 64];
    const int lane = __lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t* pc = pack[wv][0];
    int32_t* ps = pack[wv][1];
    const uint64_t below = lanes_below();
    const int64_t wave = (int64_t)blockIdx.x * 4 + wv;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    const int64_t nR = (NWp + RW - 1) / RW;
    for (int64_t r = wave; r < nR; r += nwaves) {
        const int64_t w0 = r * RW;
        int32_t vv[RW], uu[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int64_t e = (w0 + i) * 64 + lane;
            const bool in = w0 + i < NWp && e < E2;
            vv[i] = in ? col[e] : 0;
            uu[i] = in ? src[e] : 0;
        }
        for (int32_t k0 = 0; k0 < K; k0 += CPL) {
            const int32_t kl = k0 + lane / RW;
            const int64_t wl = w0 + lane % RW;
            const bool ok = kl < K && wl < NWp;  // words past NWp belong to no copy of this range
            const uint64_t myb = ok ? bits[(int64_t)kl * NWp + wl] : 0ull;
            const int32_t myp = ok ? wpre[(int64_t)kl * NWp + wl] : 0;
#pragma unroll
            for (int j = 0; j < CPL; ++j) {
                const int64_t k = k0 + j;
                if (k >= K) break;
                const int32_t base = __builtin_amdgcn_readlane(myp, j * RW);  // the copy's first kept entry here
                int32_t cnt = 0;
#pragma unroll
                for (int i = 0; i < RW; ++i) {
                    const int src_lane = j * RW + i;
                    const uint64_t bw =
                        ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(myb >> 32), src_lane) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)myb, src_lane);
                    if ((bw >> lane) & 1ull) {  // set bits lie below E2
                        const int32_t q = cnt + (int32_t)__popcll(bw & below);
                        pc[q] = (int32_t)(k * npad + vv[i]);
                        ps[q] = (int32_t)(k * npad + uu[i]);
                    }
                    cnt += (int32_t)__popcll(bw);
                }
                if (cnt == 0) continue;
                wave_lds_order();
                const int32_t none = onet ? spare[k] : 0;
                for (int32_t q = lane; q < cnt; q += 64) {
                    const int32_t v = pc[q], u = ps[q];
                    const NzWord wu(nzt, u), wv2(nzt, v);
                    int32_t at = base + q;
                    if (onet) {
                        if (!wu.has(u)) continue;  // the row of a vertex of degree 1
                        at -= NzWord(onet, u).rank(u);
                    }
                    col_out[at] = wv2.has(v) ? wv2.rank(v) : none;
                    src_out[at] = wu.rank(u);
                }
                wave_lds_order();  // read before the next copy packs
            }
        }
    }
}

// Keep bits of a union graph whose component k is sampled with (thrs[k],
// salts[k]) on its local ids (x - off[k]).
__global__ void __launch_bounds__(256) k_keep_comp(const int32_t* __restrict__ src, const int32_t* __restrict__ col,
                                                    int64_t E2, const int32_t* __restrict__ comp,
                                                    const int32_t* __restrict__ off,
                                                    const uint64_t* __restrict__ salts,
                                                    const uint64_t* __restrict__ thrs, uint64_t* __restrict__ bits,
                                                    int32_t* __restrict__ wcnt) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x; e0 < E2; e0 += stride) {
        const int64_t e = e0 + threadIdx.x;
        bool keep = false;
        if (e < E2) {
            const int32_t u = src[e], v = col[e];
            const int32_t k = comp[u];
            const int32_t o = off[k];
            keep = edge_kept((uint32_t)(u - o), (uint32_t)(v - o), salts[k], thrs[k]);
        }
        const uint64_t b = ballot64(keep);
        if (__lane_id() == 0 && e < E2) {
            bits[e >> 6] = b;
            wcnt[e >> 6] = __popcll(b);
        }
    }
}

// ---- dropping vertices of a union of samples -------------------------------
// A vertex without kept edges takes part in no triangle and in no statistic
// of the count, and one with a single edge neither, as long as it is not heavy:
// it is no source (d+ >= 2) and no source's out-neighbour (whose degrees are no
// smaller), and every other vertex keeps its degree.  An order-preserving
// relabelling keeps the (deg, id) order, so the union keeps only the vertices
// of degree >= min_deg: component k's nz[k] of them take new ids off'[k] ..
// off'[k] + nz[k] - 1 in their old order, and off'[k + 1] = off'[k] + nz[k] + 1
// rounded up to kUnionAlign, so that every component has an unused id.  64
// seeds of Chung-Lu 2^20 at p = 0.05: 9.5 -> 7.4 ms without the vertices of degree 1.

// new component offsets off2[k] (off2[K] = new n) and unused ids spare[k] (one
// thread; K is small); mk[k] = edges of component k in the padded layout
__global__ void k_nz_offsets(int32_t K, int64_t npad, const int32_t* __restrict__ nzpre, const int32_t* __restrict__ rp,
                             int32_t* __restrict__ off2, int32_t* __restrict__ spare, int64_t* __restrict__ mk) {
    if (blockIdx.x != 0) return;
    for (int32_t k = threadIdx.x; k < K; k += blockDim.x)
        mk[k] = ((int64_t)rp[(k + 1) * npad] - (int64_t)rp[k * npad]) / 2;
    if (threadIdx.x != 0) return;
    int64_t o = 0;
    const int64_t wpc = npad / 64;  // words per component
    for (int32_t k = 0; k < K; ++k) {
        off2[k] = (int32_t)o;
        const int64_t nz = (int64_t)nzpre[(k + 1) * wpc] - (int64_t)nzpre[k * wpc];
        spare[k] = (int32_t)(o + nz);
        o += (nz + kUnionAlign) / kUnionAlign * kUnionAlign;
    }
    off2[K] = (int32_t)o;
}

// For the relabelling and placing gathers: nzt[w] = (bits of the kept vertices
// 64 w .. 64 w + 63, new id of the first kept one at or after 64 w), onet[w] =
// (bits of the dropped ones of degree 1, their number before 64 w)
__global__ void k_nz_table(int64_t NV, int64_t npad, const uint64_t* __restrict__ nzb,
                           const int32_t* __restrict__ nzpre, const int32_t* __restrict__ off2,
                           const uint64_t* __restrict__ oneb, const int32_t* __restrict__ onepre,
                           int4* __restrict__ nzt, int4* __restrict__ onet) {
    const int64_t wpc = npad / 64;
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < NV; w += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = w / wpc;
        const uint64_t b = nzb[w], o = oneb[w];
        nzt[w] = make_int4((int32_t)(uint32_t)b, (int32_t)(uint32_t)(b >> 32),
                           (int32_t)(off2[k] + nzpre[w] - nzpre[k * wpc]), 0);
        onet[w] = make_int4((int32_t)(uint32_t)o, (int32_t)(uint32_t)(o >> 32), onepre[w], 0);
    }
}

// row offsets, degrees and components of the kept vertices at their new ids;
// the unused ids after each component's vertices get its end offset.  If the
// entries are odd in number, the last id's pair with itself fills E2.
__global__ void k_nz_place(int64_t nU, int64_t npad, int32_t K, int64_t entries, const int32_t* __restrict__ rp,
                           const int32_t* __restrict__ deg, const int4* __restrict__ nzt,
                           const int4* __restrict__ onet, const int32_t* __restrict__ onepre,
                           const int32_t* __restrict__ spare, const int32_t* __restrict__ off2,
                           int32_t* __restrict__ rp2, int32_t* __restrict__ deg2, int32_t* __restrict__ comp2,
                           int32_t* __restrict__ col, int32_t* __restrict__ src) {
    const int64_t nU2 = off2[K];
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < nU; x += (int64_t)gridDim.x * blockDim.x) {
        const NzWord w(nzt, x);
        if (w.has(x)) {
            const int32_t y = w.rank(x);
            rp2[y] = rp[x] - NzWord(onet, x).rank(x);
            deg2[y] = deg[x];
            comp2[y] = (int32_t)(x / npad);
        }
    }
    for (int64_t k = blockIdx.x * blockDim.x + threadIdx.x; k < K; k += (int64_t)gridDim.x * blockDim.x) {
        const int32_t end = rp[(k + 1) * npad] - onepre[(k + 1) * (npad / 64)];
        for (int64_t y = spare[k]; y < off2[k + 1]; ++y) {
            rp2[y] = end;
            deg2[y] = 0;
            comp2[y] = (int32_t)k;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        rp2[nU2] = (int32_t)entries;
        if (entries & 1) col[entries] = src[entries] = (int32_t)(nU2 - 1);
    }
}

// comp[x] = the k with off[k] <= x < off[k + 1] (largest such k)
__global__ void k_comp_from_off(int64_t n, int32_t K, const int32_t* __restrict__ off, int32_t* __restrict__ comp) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x) {
        int32_t lo = 0, hi = K - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (off[mid] <= x) lo = mid; else hi = mid - 1;
        }
        comp[x] = lo;
    }
}

// comp[x] = x / npad, off[k] = k * npad
__global__ void k_comp_rep(int64_t npad, int32_t K, int32_t* __restrict__ comp, int32_t* __restrict__ off) {
    const int64_t nU = (int64_t)K * npad;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < nU; x += (int64_t)gridDim.x * blockDim.x)
        comp[x] = (int32_t)(x / npad);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t <= K) off[t] = (int32_t)(t * npad);
}

// mk[k] = edges of component k = (rp[off[k+1]] - rp[off[k]]) / 2
__global__ void k_comp_edges(int32_t K, const int32_t* __restrict__ off, const int32_t* __restrict__ rp,
                             int64_t* __restrict__ mk) {
    for (int32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < K; k += gridDim.x * blockDim.x)
        mk[k] = ((int64_t)rp[off[k + 1]] - (int64_t)rp[off[k]]) / 2;
}

unsigned grid_for(int64_t N, int threads) {
    unsigned b = ceil_div(N, threads);
    if (b > 65536) b = 65536;
    return b ? b : 1;
}

}  // namespace

void sample_keep_bits(const tc_graph_s* g, uint64_t salt, uint64_t thr, uint64_t* bits, int32_t* wcnt, hipStream_t s) {
    const int64_t E2 = 2 * g->m;
    if (E2 == 0) return;
    TC_LAUNCH("sample_keep", k_keep_bits, dim3(grid_for(E2, 256)), dim3(256), 0, s, g->src, g->col, E2, salt, thr, bits,
              wcnt);
}

void sample_keep_staged(const tc_graph_s* g, uint64_t salt, uint64_t thr, uint64_t* bits, int32_t* wcnt,
                        int32_t* st_col, int32_t* st_src, hipStream_t s) {
    const int64_t E2 = 2 * g->m;
    if (E2 == 0) return;
    const int64_t nR = ((E2 + 63) / 64 + kStageWords - 1) / kStageWords;
    TC_LAUNCH("sample_keep", k_keep_stage, dim3(grid_for(nR, 4)), dim3(256), 0, s, g->src, g->col, E2, salt, thr,
              bits, wcnt, st_col, st_src);
}

void move_staged(int64_t E2, const int32_t* wpre, const int32_t* st_col, const int32_t* st_src, int32_t* col_out,
                 int32_t* src_out, hipStream_t s) {
    if (E2 == 0) return;
    const int64_t nR = ((E2 + 63) / 64 + kStageWords - 1) / kStageWords;
    TC_LAUNCH("compact", k_move_staged, dim3(grid_for(nR, 4)), dim3(256), 0, s, E2, wpre, st_col, st_src, col_out,
              src_out);
}

void positions_at_rows(const int32_t* row_ptr, int64_t n, int64_t E2, const uint64_t* bits, const int32_t* wpre,
                       int32_t* rp_out, int32_t* deg_out, hipStream_t s) {
    TC_LAUNCH("rows_at", k_rows_at, dim3(grid_for(n + 1, 256)), dim3(256), 0, s, row_ptr, n, E2, bits, wpre, rp_out,
              deg_out);
}

void compact_kept(const int32_t* col, const int32_t* src, int64_t E2, const uint64_t* bits, const int32_t* wpre,
                  int32_t* col_out, int32_t* src_out, hipStream_t s, const int32_t* E2_dev) {
    if (E2 == 0) return;
    TC_LAUNCH("compact", k_compact, dim3(grid_for((E2 + 63) / 64, 16)), dim3(256), 0, s, col, src, E2, E2_dev, bits,
              wpre, col_out, src_out);
}

}  // namespace tc

namespace tc {

static int32_t read_total(const int32_t* p, hipStream_t s) {
    int32_t t = 0;
    check_hip(hipMemcpyAsync(&t, p, sizeof(int32_t), hipMemcpyDeviceToHost, s), "sample total");
    check_hip(hipStreamSynchronize(s), "sync");
    return t;
}

int64_t sample_union_replicas(const tc_graph_s* g, int32_t K, const uint64_t* salts, uint64_t thr, int min_deg,
                              hipStream_t s, tc_graph_s* out, int32_t* comp, int32_t* off, int64_t* mk) {
    const int64_t n = g->n, E2 = 2 * g->m;
    const int64_t npad = (n + kUnionAlign - 1) / kUnionAlign * kUnionAlign;
    const int64_t nU = (int64_t)K * npad;
    const int64_t NWp = (E2 + 63) / 64;
    const int64_t NW = (int64_t)K * NWp;
    if (nU > 0x7fffffffLL || NW * 64 > 0x7fffffffLL) fail(TC_ERR_OVERFLOW, "the union of the samples exceeds int32 ids");
    PhaseScope ph("sample");
    out->home = s;
    out->max_deg = g->max_deg;  // sampled degrees never exceed the graph's
    if (NW == 0 || nU == 0) {  // no entries: every component is empty
        TC_LAUNCH("comp_rep", k_comp_rep, dim3(grid_for(nU > K + 1 ? nU : K + 1, 256)), dim3(256), 0, s, npad, K, comp,
                  off);
        out->n = nU;
        out->row_ptr = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(nU + 1), s);
        out->deg = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(nU > 0 ? nU : 1), s);
        fill_i32(out->row_ptr, 0, nU + 1, s);
        if (nU > 0) fill_i32(out->deg, 0, nU, s);
        out->m = 0;
        out->col = (int32_t*)dev_alloc(sizeof(int32_t), s);
        out->src = (int32_t*)dev_alloc(sizeof(int32_t), s);
        TC_LAUNCH("comp_edges", k_comp_edges, dim3(ceil_div(K, 256)), dim3(256), 0, s, K, (const int32_t*)off,
                  (const int32_t*)out->row_ptr, mk);
        return 0;
    }
    // 1. keep bits of every copy and their scan
    DevBuf<uint64_t> bits(NW, s);
    DevBuf<int32_t> wpre(NW + 1, s);
    TC_LAUNCH("keep_rep", k_keep_rep, dim3(grid_for(ceil_div(NWp, kKeepWords), 1)), dim3(256), 0, s, (const int32_t*)g->src,
              (const int32_t*)g->col, E2, NWp, K, salts, thr, bits.get(), wpre.get());
    scan_exclusive_i32(wpre.get(), wpre.get(), NW, s);
    DevBuf<int32_t> rp(nU + 1, s), deg(nU, s);
    // 2. rows in the padded layout, the vertices that are kept and the components' new offsets
    const int64_t NV = nU / 64;  // nU is a multiple of kUnionAlign
    DevBuf<uint64_t> nzb(NV, s), oneb(NV, s);
    DevBuf<int32_t> nzpre(NV + 1, s), onepre(NV + 1, s), spare(K, s);
    TC_LAUNCH("rows_rep", k_rows_rep, dim3(grid_for(NV, 4)), dim3(256), 0, s, (const int32_t*)g->row_ptr, n, npad, E2,
              NWp, K, min_deg, (const uint64_t*)bits.get(), (const int32_t*)wpre.get(), rp.get(), deg.get(), nzb.get(),
              nzpre.get(), oneb.get(), onepre.get());
    int32_t* const both[2] = {nzpre.get(), onepre.get()};
    scan_exclusive_i32_each(both, 2, NV, s);
    TC_LAUNCH("nz_offsets", k_nz_offsets, dim3(1), dim3(64), 0, s, K, npad, (const int32_t*)nzpre.get(),
              (const int32_t*)rp.get(), off, spare.get(), mk);
    int32_t sizes[3] = {0, 0, 0};  // 2m' of the samples, new vertex count, dropped vertices of degree 1
    check_hip(hipMemcpyAsync(&sizes[0], wpre.get() + NW, sizeof(int32_t), hipMemcpyDeviceToHost, s), "sample total");
    check_hip(hipMemcpyAsync(&sizes[1], off + K, sizeof(int32_t), hipMemcpyDeviceToHost, s), "union vertices");
    check_hip(hipMemcpyAsync(&sizes[2], onepre.get() + NV, sizeof(int32_t), hipMemcpyDeviceToHost, s), "dropped");
    check_hip(hipStreamSynchronize(s), "sync");
    const int64_t entries = (int64_t)sizes[0] - sizes[2], nU2 = sizes[1];
    // 3. the compacted union: rows at the new ids, kept entries relabelled
    out->n = nU2;
    out->m = (entries + 1) / 2;
    const size_t cap = (size_t)(out->m > 0 ? 2 * out->m : 1);
    out->row_ptr = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(nU2 + 1), s);
    out->deg = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(nU2 > 0 ? nU2 : 1), s);
    out->col = (int32_t*)dev_alloc(sizeof(int32_t) * cap, s);
    out->src = (int32_t*)dev_alloc(sizeof(int32_t) * cap, s);
    DevBuf<int4> nzt(NV, s), onet(NV, s);
    TC_LAUNCH("nz_table", k_nz_table, dim3(grid_for(NV, 256)), dim3(256), 0, s, NV, npad, (const uint64_t*)nzb.get(),
              (const int32_t*)nzpre.get(), (const int32_t*)off, (const uint64_t*)oneb.get(),
              (const int32_t*)onepre.get(), nzt.get(), onet.get());
    TC_LAUNCH("nz_place", k_nz_place, dim3(grid_for(nU, 256)), dim3(256), 0, s, nU, npad, K, entries,
              (const int32_t*)rp.get(), (const int32_t*)deg.get(), (const int4*)nzt.get(), (const int4*)onet.get(),
              (const int32_t*)onepre.get(), (const int32_t*)spare.get(), (const int32_t*)off, out->row_ptr, out->deg,
              comp, out->col, out->src);
    TC_LAUNCH("compact_rep", k_compact_rep, dim3(grid_for((NWp + kRepWords - 1) / kRepWords, 4)), dim3(256), 0, s,
              (const int32_t*)g->col, (const int32_t*)g->src, E2, NWp, K, npad, (const uint64_t*)bits.get(),
              (const int32_t*)wpre.get(), (const int4*)nzt.get(), min_deg > 1 ? (const int4*)onet.get() : nullptr,
              (const int32_t*)spare.get(), out->col, out->src);
    return sizes[0] / 2;
}

void comp_from_offsets(int64_t n, int32_t K, const int32_t* off, int32_t* comp, hipStream_t s) {
    if (n > 0 && K > 0)
        TC_LAUNCH("comp_from_off", k_comp_from_off, dim3(grid_for(n, 256)), dim3(256), 0, s, n, K, off, comp);
}

void sample_union_components(const tc_graph_s* gU, int32_t K, const int32_t* comp, const int32_t* off,
                             const uint64_t* salts, const uint64_t* thrs, hipStream_t s, tc_graph_s* out,
                             int64_t* mk) {
    const int64_t n = gU->n, E2 = 2 * gU->m, NW = (E2 + 63) / 64;
    PhaseScope ph("sample");
    out->n = n;
    out->home = s;
    out->max_deg = gU->max_deg;
    out->row_ptr = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(n + 1), s);
    out->deg = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(n > 0 ? n : 1), s);
    int32_t total = 0;
    if (E2 > 0) {
        DevBuf<uint64_t> bits(NW, s);
        DevBuf<int32_t> wpre(NW + 1, s);
        TC_LAUNCH("keep_comp", k_keep_comp, dim3(grid_for(E2, 256)), dim3(256), 0, s, (const int32_t*)gU->src,
                  (const int32_t*)gU->col, E2, comp, off, salts, thrs, bits.get(), wpre.get());
        scan_exclusive_i32(wpre.get(), wpre.get(), NW, s);
        positions_at_rows(gU->row_ptr, n, E2, bits.get(), wpre.get(), out->row_ptr, out->deg, s);
        total = read_total(wpre.get() + NW, s);
        out->m = total / 2;
        out->col = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(total > 0 ? total : 1), s);
        out->src = (int32_t*)dev_alloc(sizeof(int32_t) * (size_t)(total > 0 ? total : 1), s);
        compact_kept(gU->col, gU->src, E2, bits.get(), wpre.get(), out->col, out->src, s);
    } else {
        fill_i32(out->row_ptr, 0, n + 1, s);
        if (n > 0) fill_i32(out->deg, 0, n, s);
        out->m = 0;
        out->col = (int32_t*)dev_alloc(sizeof(int32_t), s);
        out->src = (int32_t*)dev_alloc(sizeof(int32_t), s);
    }
    TC_LAUNCH("comp_edges", k_comp_edges, dim3(ceil_div(K, 256)), dim3(256), 0, s, K, off,
              (const int32_t*)out->row_ptr, mk);
}

}  // namespace tc
