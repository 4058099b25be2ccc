// Token scheduling on the device (Sections 4.1-4.2): load tables, replica loads,
// Algorithm 1 as interval overlaps, per-pair destinations and permutation indices.
// Integer only; every result is independent of thread timing (no order-dependent
// atomics), so two runs and two devices give the same bits, which the paper's
// distributed scheduling relies on (Section 4.3).
#include "route.h"

namespace fine {

namespace {

constexpr int kWave = 64;

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }

// ---------------------------------------------------------------------------
// 1. One wave per 64-token word: for every expert the mask of tokens that chose it.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_words(const int32_t* __restrict__ topk_idx, int T, int K, int E, int W,
                                               unsigned long long* __restrict__ bitmap) {
    extern __shared__ unsigned long long s_bm[];   // [4][E]
    const int wave = threadIdx.x / kWave, lane = lane_id();
    const int w = blockIdx.x * 4 + wave;
    unsigned long long* bm = s_bm + (size_t)wave * E;
    for (int e = lane; e < E; e += kWave) bm[e] = 0ull;
    __syncthreads();
    const int t = w * kWave + lane;
    if (w < W && t < T) {
        for (int k = 0; k < K; ++k) {
            int e = topk_idx[(size_t)t * K + k];
            if (e >= 0 && e < E) atomicOr(&bm[e], 1ull << lane);   // OR is order independent
        }
    }
    __syncthreads();
    if (w < W)
        for (int e = lane; e < E; e += kWave) bitmap[(size_t)e * W + w] = bm[e];
}

// ---------------------------------------------------------------------------
// 2. One wave per expert: prefix of popcounts over words, load_e, input_e^g.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_scan(const unsigned long long* __restrict__ bitmap, int T, int G, int W,
                                             int32_t* __restrict__ cum, int32_t* __restrict__ inpre,
                                             int32_t* __restrict__ load, int32_t* __restrict__ input_eg) {
    extern __shared__ int32_t s_cum[];             // [W+1]
    const int e = blockIdx.x, lane = lane_id();
    const unsigned long long* bm = bitmap + (size_t)e * W;
    int carry = 0;
    for (int base = 0; base < W; base += kWave) {
        int w = base + lane;
        int c = (w < W) ? __popcll(bm[w]) : 0;
        int inc = flow::wave_incl_scan_i(c);
        if (w < W) s_cum[w] = carry + inc - c;
        carry += __builtin_amdgcn_readlane(inc, kWave - 1);
    }
    if (lane == 0) s_cum[W] = carry;
    __syncthreads();
    for (int w = lane; w <= W; w += kWave) cum[(size_t)e * (W + 1) + w] = s_cum[w];
    if (lane == 0) load[e] = carry;
    const int Tg = T / G;
    for (int g = lane; g < G; g += kWave) {
        int t0 = g * Tg, t1 = t0 + Tg;
        int b0 = s_cum[t0 >> 6] + __popcll(bm[t0 >> 6] & ((1ull << (t0 & 63)) - 1ull));
        int b1 = (t1 >= T) ? carry : s_cum[t1 >> 6] + __popcll(bm[t1 >> 6] & ((1ull << (t1 & 63)) - 1ull));
        inpre[(size_t)e * G + g] = b0;
        input_eg[(size_t)e * G + g] = b1 - b0;
    }
}

__device__ inline int overlap(int a0, int alen, int b0, int blen) {
    int lo = max(a0, b0), hi = min(a0 + alen, b0 + blen);
    return max(hi - lo, 0);
}

// ---------------------------------------------------------------------------
// 3. One wave per expert: the queues of Algorithm 1 (route.h) from the replica loads.  FULL: every expert on every rank,
//    the replica loads have a closed form (the expert-sorted sequence of pairs in chunks of M) and with them the segment
//    offsets, which are written too.
// ---------------------------------------------------------------------------
template <bool FULL>
__global__ __launch_bounds__(64) void k_tables(const int32_t* __restrict__ load, const int32_t* __restrict__ input_eg,
                                               int E, int G, int P, int locality, int rpn,
                                               int32_t* __restrict__ x_eg, int32_t* __restrict__ max_load, RouteTables t,
                                               int32_t* __restrict__ seg_off, int32_t* __restrict__ rank_off) {
    const int e = blockIdx.x, lane = lane_id();
    int xg = 0;
    if (FULL) {
        int before = 0, all = 0;
        for (int i = lane; i < E; i += kWave) {
            const int v = load[i];
            before += i < e ? v : 0;
            all += v;
        }
        const int off = flow::wave_sum_i(before), total = flow::wave_sum_i(all);
        const int M = (P + G - 1) / G;
        if (lane < G) {
            xg = overlap(off, load[e], lane * M, M);
            x_eg[(size_t)e * G + lane] = xg;
            const int lo = min(lane * M, total), hi = min(lane * M + M, total);      // the rows of this rank
            seg_off[(size_t)lane * (E + 1) + e] = min(max(off, lo), hi);
            if (e == E - 1) {
                seg_off[(size_t)lane * (E + 1) + E] = hi;
                rank_off[lane] = lo;
                if (lane == G - 1) rank_off[G] = hi;
            }
        }
        if (e == 0 && lane == 0) max_load[0] = M;
    } else {
        if (lane < G) xg = x_eg[(size_t)e * G + lane];
    }
    write_route(t, e, G, rpn, locality, lane < G ? input_eg[(size_t)e * G + lane] : 0, xg);
}

// ---------------------------------------------------------------------------
// 4. One block per rank: first row of every (rank, expert) segment (replica loads that came from the host).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_segoff(const int32_t* __restrict__ x_eg, int E, int G,
                                                int32_t* __restrict__ seg_off, int32_t* __restrict__ rank_off) {
    __shared__ int s_part[256];
    __shared__ int s_wave[4];
    const int g = blockIdx.x, tid = threadIdx.x;
    int part = 0;
    for (int i = tid; i < E * g; i += 256) {       // rows of all lower ranks
        int e = i / g, gg = i - e * g;
        part += x_eg[(size_t)e * G + gg];
    }
    s_part[tid] = part;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) s_part[tid] += s_part[tid + s];
        __syncthreads();
    }
    const int base = s_part[0];
    __syncthreads();
    int carry = base;
    for (int e0 = 0; e0 < E; e0 += 256) {
        int e = e0 + tid;
        int v = (e < E) ? x_eg[(size_t)e * G + g] : 0;
        int inc = flow::wave_incl_scan_i(v);
        if (lane_id() == kWave - 1) s_wave[tid / kWave] = inc;
        __syncthreads();
        int wbase = 0;
        for (int w = 0; w < tid / kWave; ++w) wbase += s_wave[w];
        int tot = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
        if (e < E) seg_off[(size_t)g * (E + 1) + e] = carry + wbase + inc - v;
        carry += tot;
        __syncthreads();
    }
    if (tid == 0) {
        seg_off[(size_t)g * (E + 1) + E] = carry;
        rank_off[g] = base;
        if (g == G - 1) rank_off[G] = carry;
    }
}

// ---------------------------------------------------------------------------
// 5. One thread per pair: destination rank and row.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pairs(const int32_t* __restrict__ topk_idx, int T, int K, int E, int G, int W,
                                               int locality, int rpn, const unsigned long long* __restrict__ bitmap,
                                               const int32_t* __restrict__ cum, const int32_t* __restrict__ inpre,
                                               const int32_t* __restrict__ input_eg, const int32_t* __restrict__ x_eg,
                                               RouteTables t, const int32_t* __restrict__ seg_off,
                                               int32_t* __restrict__ pair_dst, int32_t* __restrict__ row_of_pair,
                                               int32_t* __restrict__ pair_of_row) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= T * K) return;
    const int tok = p / K;
    const int e = topk_idx[p];
    // A pair without a destination (an expert index out of range; no schedule exists because an
    // expert with load has no replica) keeps its own place: row p <-> pair p.  pair_dst = -1 marks
    // it, and the movement kernels that run on these indices afterwards stay inside their buffers.
    int dst = -1, row = p;
    if (e >= 0 && e < E) {
        const int g = tok / (T / G), w = tok >> 6;
        const size_t row0 = (size_t)e * G;
        const int r = cum[(size_t)e * (W + 1) + w] + __popcll(bitmap[(size_t)e * W + w] & ((1ull << (tok & 63)) - 1ull)) -
                      inpre[row0 + g];           // rank of this token among (expert e, source g)
        int place = 0;
        dst = route_token(t, input_eg + row0, x_eg + row0, row0, G, rpn, locality, g, r, &place);
        if (dst >= 0) row = seg_off[(size_t)dst * (E + 1) + e] + place;
    }
    pair_dst[p] = dst;
    row_of_pair[p] = row;
    pair_of_row[row] = p;
}

// ---------------------------------------------------------------------------
// Small problems: all of the above by one block with every table in LDS.  Four launches of a few microseconds each
// are most of what scheduling a decoding step or a small micro-batch takes.
//   MODE 0  every expert on every rank: everything
//   MODE 1  load tables only (the replica loads come from k_general_x next, with the segment offsets and the queues)
//   MODE 2  the pairs, after that (the token bitmaps are built again)
// Scans and sums by DPP (flow_wave.h): a wave has several experts to do one after another.
// LDS: bitmap u64 [E][W], then int32 cum [E][W+1], inpre, in [E][G], and in MODE 0 x and two queues [E][G], seg_off [G][E+1],
// load [E], and a byte per pair, its expert (kSmallExperts: none).
// The pairs' experts are loaded once, all loads of a thread before the first use, and read again from LDS (4096 pairs: 0.4 us).
// Taken up to 2048 pairs, 128 experts and 2048 (expert, rank)s.  Against four launches, both replayed from a graph (in a stream
// of single launches each of them takes 1-2 us more): 512 pairs, 8 experts on 4 ranks 4.0 : 9.7 us; 1024 pairs, 128 experts on
// 8 ranks 9.8 : 10.9; 2048 pairs, 128 on 8 11.4 : 11.7, 64 on 16 10.1 : 11.1; but 1280 pairs, 192 on 5 13.5 : 12.0, 2048
// pairs, 256 on 8 18.8 : 12.7.  With every expert on every rank and at most 32 experts up to 4096 pairs, here in a stream of single
// launches: 3000 pairs, 8 on 4 7.1 : 13.5; 4096 pairs, 16 on 4 9.3 : 13.9, 32 on 8 10.9 : 13.4 (graph 11.1 : 10.8); but 64 on
// 8 12.5 : 13.4 (graph 12.7 : 11.1), and 8192 pairs, 8 on 4 15.6 : 14.5.  A restricted placement has the bitmaps built twice
// here: 8192 pairs, 16 on 8 46 : 27.
// ---------------------------------------------------------------------------
constexpr int kSmallThreads = 1024, kSmallPairs = 4096, kSmallExperts = 128, kSmallTables = 2048;
constexpr size_t kSmallLds = 64 * 1024;

__host__ __device__ inline size_t small_lds_bytes(int E, int G, int W, int P) {
    return (size_t)E * W * 8 + ((size_t)E * (W + 1) + 5 * (size_t)E * G + (size_t)G * (E + 1) + E) * 4 + P;
}

template <int MODE>
__global__ __launch_bounds__(kSmallThreads) void k_sched_small(const int32_t* __restrict__ topk_idx, int T, int K, int E, int G,
                                                               int W, int locality, int32_t* __restrict__ load,
                                                               int32_t* __restrict__ input_eg, int32_t* __restrict__ x_eg,
                                                               int32_t* __restrict__ max_load, int32_t* __restrict__ pair_dst,
                                                               int32_t* __restrict__ row_of_pair, int32_t* __restrict__ pair_of_row,
                                                               int32_t* __restrict__ seg_off, int32_t* __restrict__ rank_off,
                                                               RouteTables route) {
    extern __shared__ unsigned long long s_small[];
    unsigned long long* bm = s_small;
    int* cum = reinterpret_cast<int*>(bm + E * W);
    int* inpre = cum + E * (W + 1);
    int* in = inpre + E * G;
    int* x = in + E * G;
    int* seg = x + 3 * E * G;
    int* s_load = seg + G * (E + 1);
    unsigned char* expert = reinterpret_cast<unsigned char*>(s_load + E);
    constexpr int kWaves = kSmallThreads / kWave;
    const int tid = threadIdx.x, wave = tid / kWave, lane = lane_id(), P = T * K;

    // 1. token bitmaps
    for (int i = tid; i < E * W; i += kSmallThreads) bm[i] = 0ull;
    __syncthreads();
    int own[kSmallPairs / kSmallThreads];      // all loads before the first use
#pragma unroll
    for (int u = 0; u < kSmallPairs / kSmallThreads; ++u) own[u] = tid + u * kSmallThreads < P ? topk_idx[tid + u * kSmallThreads] : -1;
#pragma unroll
    for (int u = 0; u < kSmallPairs / kSmallThreads; ++u) {
        const int p = tid + u * kSmallThreads, t = p / K;
        const bool ok = own[u] >= 0 && own[u] < E;
        if (p < P) expert[p] = (unsigned char)(ok ? own[u] : kSmallExperts);
        if (ok) atomicOr(&bm[own[u] * W + (t >> 6)], 1ull << (t & 63));      // OR is order independent
    }
    __syncthreads();
    // 2. prefix of popcounts and load_e: a thread per expert where it has few words, else a wave (W <= 64: a word per lane);
    //    then input_e^g, a thread per (expert, source)
    const int Tg = T / G;
    auto put_load = [&](int e, int total) {
        cum[e * (W + 1) + W] = total;
        if (MODE == 0) s_load[e] = total;
        if (MODE != 2) load[e] = total;
    };
    if (W <= 4) {
        for (int e = tid; e < E; e += kSmallThreads) {
            int total = 0;
            for (int w = 0; w < W; ++w) {
                cum[e * (W + 1) + w] = total;
                total += __popcll(bm[e * W + w]);
            }
            put_load(e, total);
        }
    } else {
        for (int e = wave; e < E; e += kWaves) {
            const int c = lane < W ? __popcll(bm[e * W + lane]) : 0, inc = flow::wave_incl_scan_i(c);
            if (lane < W) cum[e * (W + 1) + lane] = inc - c;
            if (lane == kWave - 1) put_load(e, inc);
        }
    }
    __syncthreads();
    for (int i = tid; i < E * G; i += kSmallThreads) {
        const int e = i / G, t0 = (i - e * G) * Tg;
        auto before = [&](int t) -> int {      // pairs of e among the tokens before t
            const int w = t >> 6;
            return cum[e * (W + 1) + w] + (t & 63 ? __popcll(bm[e * W + w] & ((1ull << (t & 63)) - 1ull)) : 0);
        };
        const int b0 = before(t0), b1 = t0 + Tg >= T ? cum[e * (W + 1) + W] : before(t0 + Tg);
        inpre[i] = b0;
        in[i] = b1 - b0;
        if (MODE != 2) input_eg[i] = b1 - b0;
    }
    if (MODE == 1) return;
    __syncthreads();
    // 3. a wave per expert: replica loads, segment offsets, the queues of Algorithm 1 (see k_tables)
    const RouteTables t = MODE == 0 ? RouteTables{x + E * G, x + 2 * E * G, nullptr, nullptr} : route;
    if (MODE == 0) {
        const int M = (P + G - 1) / G;
        for (int e = wave; e < E; e += kWaves) {
            int part = 0, all = 0;
            for (int i = lane; i < E; i += kWave) {
                const int v = s_load[i];
                part += i < e ? v : 0;
                all += v;
            }
            const int off = flow::wave_sum_i(part), total = flow::wave_sum_i(all), mine = s_load[e];
            int xg = 0;
            if (lane < G) {
                xg = overlap(off, mine, lane * M, M);
                x[e * G + lane] = x_eg[e * G + lane] = xg;
                const int lo = min(lane * M, total), hi = min(lane * M + M, total);      // the rows of this rank
                seg[lane * (E + 1) + e] = seg_off[lane * (E + 1) + e] = min(max(off, lo), hi);
                if (e == E - 1) {
                    seg_off[lane * (E + 1) + E] = hi;
                    rank_off[lane] = lo;
                    if (lane == G - 1) rank_off[G] = hi;
                }
            }
            if (e == 0 && lane == 0) max_load[0] = M;
            write_route(t, e, G, 0, locality, lane < G ? in[e * G + lane] : 0, xg);
        }
        __syncthreads();
    }
    // 4. destination and row of every pair (see k_pairs)
    const int* xs = MODE == 0 ? x : x_eg;
    const int* segs = MODE == 0 ? seg : seg_off;
    for (int p = tid; p < P; p += kSmallThreads) {
        const int tok = p / K, e = expert[p];
        int dst = -1, row = p;
        if (e < E) {
            const int g = tok / Tg, w = tok >> 6;
            const int r = cum[e * (W + 1) + w] + __popcll(bm[e * W + w] & ((1ull << (tok & 63)) - 1ull)) - inpre[e * G + g];
            int place = 0;
            dst = route_token(t, in + e * G, xs + e * G, (size_t)e * G, G, 0, locality, g, r, &place);
            if (dst >= 0) row = segs[dst * (E + 1) + e] + place;
        }
        pair_dst[p] = dst;
        row_of_pair[p] = row;
        pair_of_row[row] = p;
    }
}

}  // namespace

SchedWs sched_ws_layout(const fine_shape& s) {
    SchedWs w;
    w.W = cdiv(s.T, 64);
    size_t o = 0;
    w.bitmap = o; o = align_up(o + (size_t)s.E * w.W * 8, 256);
    w.cum = o;    o = align_up(o + (size_t)s.E * (w.W + 1) * 4, 256);
    w.inpre = o;  o = align_up(o + (size_t)s.E * s.G * 4, 256);
    w.route = o;
    // (the contract's size, from when these were two tables of [E][G][G]; at least what the four of [E][G] take when there
    // are nodes, i.e. more than one rank, and the two without)
    o = align_up(o + (size_t)s.E * s.G * s.G * 4, 256);
    o = align_up(o + (size_t)s.E * s.G * s.G * 4, 256);
    w.total = o;
    return w;
}

int launch_general_x(const fine_shape& s, const uint8_t* place, const int32_t* load, const int32_t* x_prev,
                     int32_t* x_eg, int32_t* max_load, const int32_t* input_eg, const RouteTables& t, int32_t* seg_off, int32_t* rank_off,
                     hipStream_t st);

namespace {

struct SchedArrays {
    unsigned long long* bitmap;
    int32_t *cum, *inpre;
    RouteTables route;
    int W;
};
SchedArrays sched_arrays(const fine_shape& s, char* ws) {
    const SchedWs L = sched_ws_layout(s);
    int32_t* r = reinterpret_cast<int32_t*>(ws + L.route);
    const size_t n = (size_t)s.E * s.G;
    return {reinterpret_cast<unsigned long long*>(ws + L.bitmap), reinterpret_cast<int32_t*>(ws + L.cum),
            reinterpret_cast<int32_t*>(ws + L.inpre), RouteTables{r, r + n, r + 2 * n, r + 3 * n}, L.W};
}

int launch_pairs(const fine_shape& s, const int32_t* topk_idx, int rpn, const int32_t* input_eg, const int32_t* x_eg,
                 const SchedArrays& a, int32_t* pair_dst, int32_t* row_of_pair, int32_t* pair_of_row, const int32_t* seg_off,
                 hipStream_t st) {
    hipLaunchKernelGGL(k_pairs, dim3(cdiv(s.T * s.K, 256)), dim3(256), 0, st,
                       topk_idx, s.T, s.K, s.E, s.G, a.W, (s.flags & FINE_FLAG_LOCALITY) ? 1 : 0, rpn, a.bitmap, a.cum,
                       a.inpre, input_eg, x_eg, a.route, seg_off, pair_dst, row_of_pair, pair_of_row);
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

}  // namespace

// load tables (Table 1) into load / input_eg, token bitmaps and prefix counts into the workspace
int launch_sched_tables(const fine_shape& s, const int32_t* topk_idx, int32_t* load, int32_t* input_eg, char* ws,
                        hipStream_t st) {
    const SchedArrays a = sched_arrays(s, ws);
    hipLaunchKernelGGL(k_words, dim3(cdiv(a.W, 4)), dim3(256), (size_t)4 * s.E * 8, st,
                       topk_idx, s.T, s.K, s.E, a.W, a.bitmap);
    FINE_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_scan, dim3(s.E), dim3(64), (size_t)(a.W + 1) * 4, st,
                       a.bitmap, s.T, s.G, a.W, a.cum, a.inpre, load, input_eg);
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

// Algorithm 1 (with the node pass when ranks_per_node > 1) and the indices, from given replica loads
int launch_sched_routing(const fine_shape& s, const int32_t* topk_idx, int ranks_per_node, const int32_t* load,
                         const int32_t* input_eg, int32_t* x_eg, int32_t* pair_dst, int32_t* row_of_pair,
                         int32_t* pair_of_row, int32_t* seg_off, int32_t* rank_off, char* ws, hipStream_t st) {
    const SchedArrays a = sched_arrays(s, ws);
    const int locality = (s.flags & FINE_FLAG_LOCALITY) ? 1 : 0;
    const int rpn = s.G > 1 ? ranks_per_node : 0;
    hipLaunchKernelGGL(k_tables<false>, dim3(s.E), dim3(64), 0, st, load, input_eg, s.E, s.G, s.T * s.K, locality, rpn, x_eg,
                       (int32_t*)nullptr, a.route, (int32_t*)nullptr, (int32_t*)nullptr);
    FINE_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_segoff, dim3(s.G), dim3(256), 0, st, x_eg, s.E, s.G, seg_off, rank_off);
    FINE_LAUNCH_CHECK();
    return launch_pairs(s, topk_idx, rpn, input_eg, x_eg, a, pair_dst, row_of_pair, pair_of_row, seg_off, st);
}

int launch_sched(const fine_shape& s, const int32_t* topk_idx, const uint8_t* place, const int32_t* x_prev,
                 int32_t* load, int32_t* input_eg, int32_t* x_eg, int32_t* max_load,
                 int32_t* pair_dst, int32_t* row_of_pair, int32_t* pair_of_row,
                 int32_t* seg_off, int32_t* rank_off, char* ws, hipStream_t st) {
    const int W = cdiv(s.T, 64);
    const SchedArrays a = sched_arrays(s, ws);
    const bool small = W <= 64 && (long long)s.T * s.K <= (place == nullptr && s.E <= 32 ? kSmallPairs : kSmallPairs / 2) &&
                       s.E <= kSmallExperts && s.E * s.G <= kSmallTables;
    const size_t small_lds = small ? small_lds_bytes(s.E, s.G, W, s.T * s.K) : kSmallLds + 1;
    if (small_lds <= kSmallLds) {
        auto run = [&](auto k) {
            hipLaunchKernelGGL(k, dim3(1), dim3(kSmallThreads), small_lds, st, topk_idx, s.T, s.K, s.E, s.G, W,
                               (s.flags & FINE_FLAG_LOCALITY) ? 1 : 0, load, input_eg, x_eg, max_load, pair_dst, row_of_pair,
                               pair_of_row, seg_off, rank_off, a.route);
            return check_hip(hipGetLastError());
        };
        if (place == nullptr) return run(k_sched_small<0>);
        FINE_TRY(run(k_sched_small<1>));
        FINE_TRY(launch_general_x(s, place, load, x_prev, x_eg, max_load, input_eg, a.route, seg_off, rank_off, st));
        return run(k_sched_small<2>);
    }
    FINE_TRY(launch_sched_tables(s, topk_idx, load, input_eg, ws, st));
    if (place != nullptr) {
        FINE_TRY(launch_general_x(s, place, load, x_prev, x_eg, max_load, input_eg, a.route, seg_off, rank_off, st));
    } else {
        hipLaunchKernelGGL(k_tables<true>, dim3(s.E), dim3(64), 0, st, load, input_eg, s.E, s.G, s.T * s.K,
                           (s.flags & FINE_FLAG_LOCALITY) ? 1 : 0, 0, x_eg, max_load, a.route, seg_off, rank_off);
        FINE_LAUNCH_CHECK();
    }
    return launch_pairs(s, topk_idx, 0, input_eg, x_eg, a, pair_dst, row_of_pair, pair_of_row, seg_off, st);
}

// ---------------------------------------------------------------------------
// Scratch memory of fine_sched_static: an array in the library's device image, for callers that
// cannot hand over (or allocate) a workspace.  Each GPU holds its own copy of the array at its own
// address, and the array's name is only a host-side handle, never a device address: the address is
// asked for once per device, with that device current, and that pointer is what the kernels get.
// ---------------------------------------------------------------------------
namespace {

static __device__ __align__(256) unsigned char scratch[kSchedStaticBytes];

constexpr int kMaxDevices = 64;
std::atomic<unsigned char*> g_scratch_ptr[kMaxDevices];      // zero-initialised: not asked for yet

}  // namespace

int sched_static_scratch(char** out) {
    int dev = 0;
    FINE_TRY(check_hip(hipGetDevice(&dev)));
    if (dev < 0 || dev >= kMaxDevices) return FINE_UNSUPPORTED;
    unsigned char* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (ptr == nullptr) {
        FINE_TRY(check_hip(hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch))));
        if (ptr == nullptr) return FINE_HIP_ERROR;
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);      // concurrent first calls store the same address
    }
    *out = reinterpret_cast<char*>(ptr);
    return FINE_OK;
}

}  // namespace fine
