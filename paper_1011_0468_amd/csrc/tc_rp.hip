// Random-projection trace estimator (section 5.1).  The paper projects the
// adjacency columns with a Gaussian matrix R and shows E[Y] = k tr(A^3) for
// Y = sum_l r_l^T A^3 r_l.  Here each r_l is a Rademacher vector x_l (the same
// mean, E[x_i x_j] = delta_ij) so that q_l = x_l^T A^3 x_l = (A x_l)^T A (A x_l)
// is an exact integer.  Vectors are processed 64 at a time: one 64-bit hash
// word per vertex holds the 64 signs of a chunk, and lane b of a wave owns
// vector b of the chunk.
//
//   word[i] = mix64(mix64(c << 32 | i) ^ salt)       (computed where it is used)
//   rp_spmm : Y[i][b] = sum_{j in N(i)} x_b[j] = deg i - 2 #{j in N(i) : bit b of word[j]}
//             (per batch of 64 entries: a 64 x 64 bit transpose, then one masked
//             popcount per lane and run of one row)
//   rp_dot  : q[b]    = sum over CSR entries (i, j) of Y[i][b] * Y[j][b]
//                     = 2 * sum over one entry of each edge (see k_rp_dot)
//
// Both sweeps are edge-parallel: wave w owns CSR entries [w L, (w+1) L), so a
// hub row is split over many waves.  rp_dot is a plain sum over entries.  In
// rp_spmm a row that lies entirely inside one wave's range is stored
// directly; the partial rows at range boundaries are accumulated atomically
// into rows that rp_clear_ends zeroes first (the count is additive over any
// split of the row).
#include "tc_internal.h"
#include "tc_device.h"

#include <algorithm>
#include <vector>

namespace tc {

namespace {

constexpr int kRpRange = 4096;  // CSR entries per wave
constexpr int kRpUnroll = 8;    // entries whose loads are issued together

// The 64 signs of vertex i in chunk c (bit b set: x_{64c+b}[i] = -1).
__device__ __forceinline__ uint64_t sign_word(uint64_t chunk, int32_t i, uint64_t salt) {
    return mix64(mix64((chunk << 32) | (uint64_t)(uint32_t)i) ^ salt);
}

__device__ __forceinline__ void rp_flush(int32_t i, int32_t cnt, int32_t ones, int64_t e0, int64_t e1,
                                         const int32_t* __restrict__ row_ptr, int32_t* __restrict__ Y, int lane) {
    const int32_t val = cnt - 2 * ones;
    if ((int64_t)row_ptr[i] >= e0 && (int64_t)row_ptr[i + 1] <= e1) Y[(int64_t)i * 64 + lane] = val;
    else atomicAdd(&Y[(int64_t)i * 64 + lane], val);
}

// Lane exchange with lane ^ J of a 32-bit value (ds_swizzle inside each half
// of the wave, a permute across the halves).
template <int J>
__device__ __forceinline__ uint32_t rp_xor(uint32_t v) {
    if constexpr (J < 32) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (J << 10) | 0x1F);
    else return (uint32_t)__shfl_xor((int)v, J, 64);
}

// Level J < 32 of the 64 x 64 bit transpose on one 32-bit half (m: the bits
// whose index has bit J clear).  Bit c of lane l moves to bit c ^ J of lane
// l ^ J when bit J of l and bit J of c differ, and stays otherwise.
template <int J>
__device__ __forceinline__ uint32_t transpose_level(uint32_t x, uint32_t m, bool hi_lane) {
    const uint32_t o = rp_xor<J>(x);
    return hi_lane ? ((x & ~m) | ((o >> J) & m)) : ((x & m) | ((o << J) & ~m));
}

// Transposes the 64 x 64 bit matrix whose row l is lane l's word (lo, hi):
// afterwards bit k of lane b's word is bit b of lane k's word.  Each level J
// exchanges the elements whose row and column differ in bit J; the levels
// act on different bits of (row xor column), so together they swap every
// element with its mirror.  Whole wave.
__device__ __forceinline__ void transpose64(uint32_t& lo, uint32_t& hi, int lane) {
    {
        const bool h = (lane & 32) != 0;
        const uint32_t got = rp_xor<32>(h ? lo : hi);  // the half the partner keeps below / above
        if (h) lo = got; else hi = got;
    }
    lo = transpose_level<16>(lo, 0x0000FFFFu, (lane & 16) != 0);
    hi = transpose_level<16>(hi, 0x0000FFFFu, (lane & 16) != 0);
    lo = transpose_level<8>(lo, 0x00FF00FFu, (lane & 8) != 0);
    hi = transpose_level<8>(hi, 0x00FF00FFu, (lane & 8) != 0);
    lo = transpose_level<4>(lo, 0x0F0F0F0Fu, (lane & 4) != 0);
    hi = transpose_level<4>(hi, 0x0F0F0F0Fu, (lane & 4) != 0);
    lo = transpose_level<2>(lo, 0x33333333u, (lane & 2) != 0);
    hi = transpose_level<2>(hi, 0x33333333u, (lane & 2) != 0);
    lo = transpose_level<1>(lo, 0x55555555u, (lane & 1) != 0);
    hi = transpose_level<1>(hi, 0x55555555u, (lane & 1) != 0);
}

// Y = A X over the wave's entry range, 64 entries per batch: lane k loads
// entry k and computes its neighbour's sign word (hashing is cheaper than a
// random 8-byte gather per entry), the 64 words are transposed so that lane b
// holds bit b of every entry's word, and each run of entries of one row adds
// its length to cnt and its masked popcount to ones (lane b: the entries
// whose sign b is negative).  A row is written when the next one starts.
__global__ void __launch_bounds__(256) k_rp_spmm(int64_t E2, const int32_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ src, const int32_t* __restrict__ col,
                                                  uint64_t chunk, uint64_t salt, int32_t* __restrict__ Y) {
    const int lane = __lane_id();
    const int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t e0 = w * kRpRange;
    if (e0 >= E2) return;
    const int64_t e1 = e0 + kRpRange < E2 ? e0 + kRpRange : E2;
    int32_t cur = __builtin_amdgcn_readfirstlane(src[e0]);
    int32_t cnt = 0, ones = 0;
    for (int64_t eb = e0; eb < e1; eb += 64) {
        const int64_t el = eb + lane;
        const bool valid = el < e1;
        const int32_t vi = valid ? src[el] : -1;
        const int32_t vj = valid ? col[el] : 0;
        const uint64_t wv = valid ? sign_word(chunk, vj, salt) : 0ull;
        uint32_t lo = (uint32_t)wv, hi = (uint32_t)(wv >> 32);
        transpose64(lo, hi, lane);
        int32_t prev = __shfl_up(vi, 1, 64);
        if (lane == 0) prev = cur;
        const uint64_t V = ballot64(valid);               // a prefix of the lanes
        const uint64_t S = ballot64(valid && vi != prev);  // entries that start a row
        uint64_t rest = V;
        while (rest) {  // wave-uniform: one pass per run of one row
            const int k0 = __builtin_ctzll(rest);
            if ((S >> k0) & 1ull) {
                rp_flush(cur, cnt, ones, e0, e1, row_ptr, Y, lane);
                cur = __builtin_amdgcn_readlane(vi, k0);
                cnt = 0;
                ones = 0;
            }
            const uint64_t after = S & (~1ull << k0);  // row starts past k0
            const uint64_t run = after ? rest & ((1ull << __builtin_ctzll(after)) - 1ull) : rest;
            cnt += (int32_t)__popcll(run);
            ones += (int32_t)(__builtin_popcount(lo & (uint32_t)run) + __builtin_popcount(hi & (uint32_t)(run >> 32)));
            rest &= ~run;
        }
    }
    rp_flush(cur, cnt, ones, e0, e1, row_ptr, Y, lane);
}

// Clears the rows of Y that k_rp_spmm accumulates atomically: a row split
// between two wave ranges is the last row of one and the first of the next,
// so clearing the first and last row of every range covers them (the other
// rows are stored whole, and rows without entries are never read).
__global__ void __launch_bounds__(256) k_rp_clear_ends(int64_t E2, const int32_t* __restrict__ src,
                                                        int32_t* __restrict__ Y) {
    const int lane = __lane_id();
    const int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t e0 = w * kRpRange;
    if (e0 >= E2) return;
    const int64_t e1 = e0 + kRpRange < E2 ? e0 + kRpRange : E2;
    Y[(int64_t)src[e0] * 64 + lane] = 0;
    Y[(int64_t)src[e1 - 1] * 64 + lane] = 0;
}

// q[b] = sum over CSR entries (i, j) of Y[i][b] Y[j][b] = 2 * the sum over one
// entry of each undirected edge (A is symmetric without loops): the one in the
// row of the end with the smaller (degree class, id) in a graph that stores its
// entries' neighbour classes (CLASSES), with the smaller id otherwise.  Bound by the 256-byte
// gathers of Y[j], one per edge: pointing every edge at its end of larger
// degree sends them to the few rows of the hubs, which the L2s and the
// Infinity Cache hold, where the order of the ids alone sends half of them to
// rows that only memory holds.  R-MAT s22 (64 M edges, 16 GB of rows a
// sweep): 2.40 -> 1.72 ms a sweep with the queue below.  A sample stores no
// classes, and gathering them costs more than the order gains (s22 at p = 0.9: by
// id without and with the queue 2.18 and 1.85 ms, by gathered class 2.44; uniform
// 2^22: 2.76, 2.43 and 3.54).
// The entries that count are queued per wave in LDS, so that the gathers run
// over full batches of 64 without a branch per entry, kRpUnroll in flight.
// Y below 4 GiB is read with buffer loads, whose scalar offset is the row's
// byte offset straight from a lane (WIDE: 64-bit addresses): with the
// addresses in scalar arithmetic the kernel took 16 scalar instructions an
// edge and was bound by them.
constexpr int kRpQueue = 128;

template <bool WIDE>
__device__ __forceinline__ int32_t rp_row(const int32_t* __restrict__ Y, __amdgpu_buffer_rsrc_t rs, int32_t v,
                                          int32_t off, int k, int lane) {
    if constexpr (WIDE) return Y[(int64_t)__builtin_amdgcn_readlane(v, k) * 64 + lane];
    else return __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, __builtin_amdgcn_readlane(off, k), 0);
}

// The products of up to 64 queued entries, entry k on lane k (FULL: all 64).
template <bool WIDE, bool FULL>
__device__ __forceinline__ void rp_batch(const int32_t* __restrict__ Y, __amdgpu_buffer_rsrc_t rs, int32_t vi,
                                         int32_t vj, int cnt, int lane, int32_t& cur, int32_t& ycur, int64_t& acc) {
    int32_t prev = __shfl_up(vi, 1, 64);
    if (lane == 0) prev = cur;
    uint64_t fresh = ballot64((FULL || lane < cnt) && vi != prev);  // entries that start a row
    const int32_t oi = (int32_t)((uint32_t)vi << 8), oj = (int32_t)((uint32_t)vj << 8);
    // not unrolled: the rounds of a batch would all be in flight at once, at 2 or 3 waves per SIMD
#pragma unroll 1
    for (int k0 = 0; k0 < (FULL ? 64 : cnt); k0 += kRpUnroll, fresh >>= kRpUnroll) {
        int32_t yj[kRpUnroll], yi[kRpUnroll];
#pragma unroll
        for (int k = 0; k < kRpUnroll; ++k) {
            yj[k] = FULL || k0 + k < cnt ? rp_row<WIDE>(Y, rs, vj, oj, k0 + k, lane) : 0;
            if ((fresh >> k) & 1ull) yi[k] = rp_row<WIDE>(Y, rs, vi, oi, k0 + k, lane);
        }
#pragma unroll
        for (int k = 0; k < kRpUnroll; ++k) {
            if ((fresh >> k) & 1ull) ycur = yi[k];
            acc += (int64_t)ycur * (int64_t)yj[k];
        }
    }
    cur = __builtin_amdgcn_readlane(vi, FULL ? 63 : cnt - 1);
}

template <bool CLASSES, bool WIDE>
__global__ void __launch_bounds__(256) k_rp_dot(int64_t E2, const int32_t* __restrict__ src,
                                                 const int32_t* __restrict__ col, const uint8_t* __restrict__ cls,
                                                 const uint8_t* __restrict__ ncls, const int32_t* __restrict__ Y,
                                                 uint32_t ybytes, int64_t* __restrict__ q) {
    __shared__ int2 queue[4][kRpQueue];
    __shared__ int64_t red[4][64];
    const int lane = __lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t w = (int64_t)blockIdx.x * 4 + wv;
    const int64_t e0 = w * kRpRange;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(Y), 0, WIDE ? 0 : (int)ybytes, 0x00020000);
    int2* Q = queue[wv];
    int64_t acc = 0;
    if (e0 < E2) {
        const int64_t e1 = e0 + kRpRange < E2 ? e0 + kRpRange : E2;
        int32_t cur = -1, ycur = 0;
        int head = 0, held = 0;  // queued entries: Q[head ..], held < 64 between rounds
        for (int64_t eb = e0; eb < e1; eb += 64) {
            const int64_t el = eb + lane;
            const bool in = el < e1;
            const int32_t vi = in ? src[el] : 0;
            const int32_t vj = in ? col[el] : 0;
            const uint32_t ci = CLASSES && in ? cls[vi] : 0u, cj = CLASSES && in ? ncls[el] : 0u;
            const bool up = in && (ci < cj || (ci == cj && vi < vj));
            const uint64_t U = ballot64(up);
            if (up) Q[(head + held + __popcll(U & lanes_below())) & (kRpQueue - 1)] = make_int2(vi, vj);
            held += __popcll(U);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // a wave's LDS operations run in issue order
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (held >= 64) {
                const int2 e = Q[(head + lane) & (kRpQueue - 1)];
                head = (head + 64) & (kRpQueue - 1);
                held -= 64;
                rp_batch<WIDE, true>(Y, rs, e.x, e.y, 64, lane, cur, ycur, acc);
            }
        }
        if (held > 0) {
            const int2 e = lane < held ? Q[(head + lane) & (kRpQueue - 1)] : make_int2(0, 0);
            rp_batch<WIDE, false>(Y, rs, e.x, e.y, held, lane, cur, ycur, acc);
        }
    }
    red[wv][lane] = acc;
    __syncthreads();
    if (wv == 0) {
        const int64_t s = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
        if (s) atomicAdd((unsigned long long*)&q[lane], (unsigned long long)(2 * s));
    }
}

// An upper bound of the sum over CSR entries (i, j) of deg_i * deg_j: deg_j
// taken as the largest degree of its class (at most 1/8 too large), which is
// stored with the entry instead of gathered.  One partial per block, summed on
// the host.
__global__ void __launch_bounds__(256) k_rp_class_bound(const int32_t* __restrict__ src,
                                                         const int32_t* __restrict__ deg,
                                                         const uint8_t* __restrict__ ncls, int64_t E2,
                                                         double* __restrict__ part) {
    double s = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < E2; e += (int64_t)gridDim.x * blockDim.x)
        s += (double)deg[src[e]] * (double)class_max_degree(ncls[e]);
    s = wave_sum(s);
    __shared__ double red[4];
    if (__lane_id() == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// Half the sum over CSR entries (i, j) of deg_i * deg_j, in double (a bound
// only): the entries with j > i, whose mirrors give the same sum, so only
// they gather deg_j.  One partial per block, summed on the host.
__global__ void __launch_bounds__(256) k_rp_bound(const int32_t* __restrict__ src, const int32_t* __restrict__ col,
                                                   const int32_t* __restrict__ deg, int64_t E2,
                                                   double* __restrict__ part) {
    double s = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < E2; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t i = src[e], j = col[e];
        if (j > i) s += (double)deg[i] * (double)deg[j];
    }
    s = wave_sum(s);
    __shared__ double red[4];
    if (__lane_id() == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

}  // namespace

void rp_trace(const tc_graph_s* g, int32_t k, uint64_t seed, hipStream_t s, int64_t* q_host) {
    PhaseScope ph("rp");
    const int64_t n = g->n, E2 = 2 * g->m;
    for (int32_t l = 0; l < k; ++l) q_host[l] = 0;
    if (n == 0 || E2 == 0) return;
    const uint8_t* ncls = g->ncls;
    DevBuf<uint8_t> cls;
    if (ncls) {
        cls.reset(n, s);
        degree_classes(n, g->deg, cls.get(), s);
    }
    {
        // |q_l| <= sum over entries (i, j) of |Y_il| |Y_jl| <= sum of deg_i deg_j; every q_l and their sum
        // stay exact while k times that is below 2^62 (margin for the double rounding).  A bound from the
        // stored degree classes settles most built graphs (R-MAT s22: 0.65 -> 0.25 ms); where it does not, and
        // in samples (gathered classes: 0.59 -> 0.77 ms on s22 at p = 0.9), the degrees themselves decide.
        constexpr unsigned kClassBlocks = 2048, kBlocks = 1024;
        DevBuf<double> part(std::min(ceil_div(E2, 256), kClassBlocks), s);
        auto total = [&](unsigned blocks) {
            std::vector<double> hpart(blocks);
            check_hip(hipMemcpyAsync(hpart.data(), part.get(), sizeof(double) * blocks, hipMemcpyDeviceToHost, s),
                      "bound");
            check_hip(hipStreamSynchronize(s), "sync");
            double t = 0.0;
            for (double v : hpart) t += v;
            return t * (double)k;
        };
        const double limit = 4.611686018427387904e18;
        bool settled = false;
        if (ncls) {
            const unsigned blocks = std::min(ceil_div(E2, 256), kClassBlocks);
            TC_LAUNCH("rp_bound", k_rp_class_bound, dim3(blocks), dim3(256), 0, s, (const int32_t*)g->src,
                      (const int32_t*)g->deg, ncls, E2, part.get());
            settled = total(blocks) * (1.0 + 1e-9) < limit;
        }
        if (!settled) {
            const unsigned blocks = std::min(ceil_div(E2, 256), kBlocks);
            TC_LAUNCH("rp_bound", k_rp_bound, dim3(blocks), dim3(256), 0, s, (const int32_t*)g->src,
                      (const int32_t*)g->col, (const int32_t*)g->deg, E2, part.get());
            if (2.0 * total(blocks) >= limit)
                fail(TC_ERR_OVERFLOW, "k * sum deg_i deg_j reaches 2^62: q could overflow int64");
        }
    }
    const uint64_t salt = [&] {
        uint64_t z = seed ^ 0x52505F5452414345ull;  // "RP_TRACE"
        z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull; z ^= z >> 27; z *= 0x94D049BB133111EBull; z ^= z >> 31;
        return z;
    }();
    DevBuf<int32_t> Y((size_t)n * 64, s);
    DevBuf<int64_t> qd(64, s);
    const int32_t nchunks = (k + 63) / 64;
    const int64_t waves = (E2 + kRpRange - 1) / kRpRange;
    const unsigned wblocks = (unsigned)((waves + 3) / 4);
    const bool wide = n * 256 >= ((int64_t)1 << 32);  // rows past the reach of a buffer load's offset
    const auto dot = wide ? (ncls ? k_rp_dot<true, true> : k_rp_dot<false, true>)
                          : (ncls ? k_rp_dot<true, false> : k_rp_dot<false, false>);
    for (int32_t c = 0; c < nchunks; ++c) {
        fill_i64(qd.get(), 0, 64, s);
        TC_LAUNCH("rp_clear", k_rp_clear_ends, dim3(wblocks), dim3(256), 0, s, E2, (const int32_t*)g->src, Y.get());
        TC_LAUNCH("rp_spmm", k_rp_spmm, dim3(wblocks), dim3(256), 0, s, E2, (const int32_t*)g->row_ptr,
                  (const int32_t*)g->src, (const int32_t*)g->col, (uint64_t)c, salt, Y.get());
        TC_LAUNCH("rp_dot", dot, dim3(wblocks), dim3(256), 0, s, E2, (const int32_t*)g->src, (const int32_t*)g->col,
                  (const uint8_t*)cls.get(), ncls, (const int32_t*)Y.get(), (uint32_t)(n * 256),
                  qd.get());
        int64_t hq[64];
        check_hip(hipMemcpyAsync(hq, qd.get(), sizeof(hq), hipMemcpyDeviceToHost, s), "q");
        check_hip(hipStreamSynchronize(s), "sync");
        for (int b = 0; b < 64 && c * 64 + b < k; ++b) q_host[c * 64 + b] = hq[b];
    }
}

}  // namespace tc
