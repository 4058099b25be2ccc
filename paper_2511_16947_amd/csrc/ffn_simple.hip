// Work-list construction for the grouped GEMMs, and the plain FMA expert FFN (layers wider than the
// matrix-core kernels' 32-bit offsets reach, and a cross-check in tests).
#include "flow_wave.h"

namespace fine {

namespace {

// One block: the work list of the (rank, expert) segments of ranks [rank_lo, rank_hi), one TileEntry per BM rows, in
// the order of the segments.  Neighbouring non-empty segments of ONE expert (its share on a rank and on the next one: a
// hot expert under the full placement fills whole ranks) form one run of rows and are cut into tiles together, so
// that a call over all ranks reads an expert's weights once and not once per rank, and has one short tile per run
// (64 tokens on 8 experts and 8 ranks: 8 tiles instead of 15).  One rank's segments are all of different experts.
// Thread t takes C consecutive segments; everything it needs of the others are two running maxima (the last non-empty
// segment; the first segment of the last run) and a sum of tile counts: three block scans whatever the number of
// segments.  A segment is named by its place in seg_off.  The ranks' rows of seg_off are read into LDS once (CACHED: where they
// fit) and walked there, with no division per segment: 8192 segments 31 -> 23 us,
// 1024 7.1 -> 5.4.
constexpr int kMapThreads = 1024;
constexpr size_t kMapLds = 60 * 1024;

// zeroes the counters that the GEMM launches of a call use
__device__ inline void clear_counts(int32_t* count) {
    for (int i = threadIdx.x; i < 256; i += blockDim.x) {
        count[kSkCounterOffset + i] = 0;
        count[kSkReadyOffset + i] = 0;
    }
    if (threadIdx.x < kQueues) count[kQueueOffset + threadIdx.x * kQueueStride] = 0;
}

// exclusive scan over the block; op(ident, v) = v
template <typename Op>
__device__ inline int block_excl_scan(int v, int ident, int* s_w, Op op) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto wave_incl = [&](int x) {      // (DPP: lane layout in flow_wave.h)
        x = op(flow::dpp_from<0x111, 0xf>(ident, x), x);
        x = op(flow::dpp_from<0x112, 0xf>(ident, x), x);
        x = op(flow::dpp_from<0x114, 0xf>(ident, x), x);
        x = op(flow::dpp_from<0x118, 0xf>(ident, x), x);
        x = op(flow::dpp_from<0x142, 0xa>(ident, x), x);
        x = op(flow::dpp_from<0x143, 0xc>(ident, x), x);
        return x;
    };
    const int inc = wave_incl(v);
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    // what the waves before this one have: their at most 16 totals, scanned by every wave
    const int tot = wave_incl(lane < (int)(blockDim.x >> 6) ? s_w[lane] : ident);
    const int base = wave == 0 ? ident : __builtin_amdgcn_readlane(tot, __builtin_amdgcn_readfirstlane(max(wave - 1, 0)));
    const int up = __shfl_up(inc, 1, 64);
    __syncthreads();      // s_w may be written again
    return lane == 0 ? base : op(base, up);
}

template <bool CACHED>
__global__ __launch_bounds__(kMapThreads) void k_tile_map(const int32_t* __restrict__ seg_off, int E, int rank_lo,
                                                          int rank_hi, int BM, int sole, TileEntry* __restrict__ tiles,
                                                          int32_t* __restrict__ count, int max_tiles) {
    extern __shared__ int32_t s_seg[];
    __shared__ int s_w[kMapThreads / 64];
    const int tid = threadIdx.x;
    clear_counts(count);
    const int32_t* from = seg_off + (size_t)rank_lo * (E + 1);
    int32_t* s_runs = s_seg + (CACHED ? (rank_hi - rank_lo) * (E + 1) : 0);      // sole: runs of each expert
    if (sole != 0)
        for (int e = tid; e < E; e += blockDim.x) s_runs[e] = 0;      // (added to after a scan's barriers)
    if (CACHED) {
        for (int i = tid; i < (rank_hi - rank_lo) * (E + 1); i += blockDim.x) s_seg[i] = from[i];
        __syncthreads();
    }
    auto first_row = [&](int at) { return CACHED ? s_seg[at] : from[at]; };
    auto end_row = [&](int at) { return CACHED ? s_seg[at + 1] : from[at + 1]; };
    const int nseg = (rank_hi - rank_lo) * E, C = (nseg + (int)blockDim.x - 1) / (int)blockDim.x;
    const int s0 = min(tid * C, nseg), s1 = min(s0 + C, nseg), g0 = s0 / E;
    // f(place, expert) for this thread's non-empty segments
    auto each = [&](auto f) {
        int at = g0 * (E + 1) + (s0 - g0 * E), e = s0 - g0 * E;
        for (int s = s0; s < s1; ++s) {
            if (end_row(at) > first_row(at)) f(at, e);
            ++at;
            if (++e == E) {
                e = 0;
                ++at;
            }
        }
    };
    auto max_op = [](int a, int b) { return max(a, b); };
    // last non-empty segment in front of this thread's
    int last = -1;
    each([&](int at, int) { last = at; });
    const int before = block_excl_scan(last, -1, s_w, max_op), before_e = before < 0 ? -1 : before % (E + 1);
    // goes on the run of the segment at `prev` (expert prev_e): the same expert, and its rows follow
    auto continues = [&](int at, int e, int prev, int prev_e) { return prev >= 0 && prev_e == e && end_row(prev) == first_row(at); };
    int head = -1, prev = before, prev_e = before_e;
    each([&](int at, int e) {
        if (!continues(at, e, prev, prev_e)) {
            head = at;
            if (sole != 0) atomicAdd(&s_runs[e], 1);
        }
        prev = at;
        prev_e = e;
    });
    const int head_at = block_excl_scan(head, -1, s_w, max_op);
    const int head_before = head_at < 0 ? 0 : first_row(head_at);      // (ranks' rows may lie in any order)
    // A run's tiles start at its first row + multiples of BM; each belongs to the segment that its first row lies in.
    // visit(e, r): a tile starts at row r of expert e; closed(e, end, head): its run from row `head` has ended at `end`.
    auto walk = [&](auto visit, auto closed) {
        int h = head_before, p = before, pe = before_e;
        each([&](int at, int e) {
            const int r0 = first_row(at), r1 = end_row(at);
            if (!continues(at, e, p, pe)) {
                if (p >= 0) closed(pe, end_row(p), h);
                h = r0;
            }
            p = at;
            pe = e;
            for (int r = h + (r0 - h + BM - 1) / BM * BM; r < r1; r += BM) visit(e, r);
        });
        if (tid == (int)blockDim.x - 1 && p >= 0) closed(pe, end_row(p), h);
    };
    int nt = 0;
    walk([&](int, int) { ++nt; }, [](int, int, int) {});
    const int at0 = block_excl_scan(nt, 0, s_w, [](int a, int b) { return a + b; });
    int at = at0;
    walk(
        [&](int e, int r) {
            if (at < max_tiles) tiles[at] = TileEntry{e, r, BM, 0};
            ++at;
        },
        [](int, int, int) {});
    __syncthreads();
    at = at0;
    walk([&](int, int) { ++at; },
         [&](int e, int end, int h) {      // its last tile is the last one so far
             if (at - 1 >= max_tiles) return;
             tiles[at - 1].rows = end - (h + (end - 1 - h) / BM * BM);
             int alone = end - h <= BM;
             if (alone != 0 && sole != 0 && s_runs[e] == 1) alone = 2;
             tiles[at - 1].alone = alone;
         });
    if (tid == (int)blockDim.x - 1) *count = min(at, max_tiles);
}

// The same for one rank, whose segments are all of different experts: one thread per expert, one scan (a launch in
// front of every rank's GEMMs, so its latency counts: 2.4-5 us).
__global__ __launch_bounds__(kMapThreads) void k_tile_map_rank(const int32_t* __restrict__ seg_off, int E, int BM,
                                                               TileEntry* __restrict__ tiles, int32_t* __restrict__ count,
                                                               int max_tiles) {
    __shared__ int s_w[kMapThreads / 64];
    const int e = threadIdx.x;
    const int r0 = e < E ? seg_off[e] : 0, n = e < E ? max(seg_off[e + 1] - r0, 0) : 0, nt = (n + BM - 1) / BM;
    clear_counts(count);
    const int at = block_excl_scan(nt, 0, s_w, [](int a, int b) { return a + b; });
    for (int i = 0; i < nt && at + i < max_tiles; ++i)
        tiles[at + i] = TileEntry{e, r0 + i * BM, min(BM, n - i * BM), nt == 1 ? 2 : 0};
    if (e == (int)blockDim.x - 1) *count = min(at + nt, max_tiles);
}

__device__ inline float silu_mul(float a, float b) { return a / (1.f + __expf(-a)) * b; }

// C tile 64x64 per block of 256 threads, each thread a 4x4 micro-tile; K stepped by 16.
//   MODE 0: H = silu(X Wg) * (X Wu)   (X [rows,Kd] lda; Wg,Wu [Kd,N]; H [rows,N]); act optional
//   MODE 1: Y = H Wd                  (plain GEMM)
template <typename T, int MODE>
__global__ __launch_bounds__(256) void k_gemm_simple(const T* __restrict__ A, int lda, const T* __restrict__ B0,
                                                     const T* __restrict__ B1, size_t b_expert_stride, int Kd, int N,
                                                     T* __restrict__ C, int ldc, T* __restrict__ act, int ldact,
                                                     const TileEntry* __restrict__ tiles, const int32_t* __restrict__ count) {
    constexpr int BM = 64, BN = 64, BK = 16;
    __shared__ float sA[BK][BM + 1];
    __shared__ float sB0[BK][BN + 1];
    __shared__ float sB1[MODE == 0 ? BK : 1][BN + 1];
    const int ntile_n = (N + BN - 1) / BN;
    const int total = (*count) * ntile_n;
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    for (int work = blockIdx.x; work < total; work += gridDim.x) {
        const TileEntry te = tiles[work / ntile_n];
        const int n0 = (work % ntile_n) * BN;
        const T* Bg = B0 + (size_t)te.expert * b_expert_stride;
        const T* Bu = (MODE == 0) ? B1 + (size_t)te.expert * b_expert_stride : nullptr;
        float acc0[4][4], acc1[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) { acc0[i][j] = 0.f; acc1[i][j] = 0.f; }
        for (int k0 = 0; k0 < Kd; k0 += BK) {
            __syncthreads();
            for (int idx = tid; idx < BM * BK; idx += 256) {
                const int m = idx / BK, kk = idx % BK;
                const int row = te.row0 + min(m, te.rows - 1);
                sA[kk][m] = (k0 + kk < Kd) ? Elem<T>::load(A + (size_t)row * lda + k0 + kk) : 0.f;
            }
            for (int idx = tid; idx < BN * BK; idx += 256) {
                const int kk = idx / BN, n = idx % BN;
                const bool ok = (k0 + kk < Kd) && (n0 + n < N);
                sB0[kk][n] = ok ? Elem<T>::load(Bg + (size_t)(k0 + kk) * N + n0 + n) : 0.f;
                if (MODE == 0) sB1[kk][n] = ok ? Elem<T>::load(Bu + (size_t)(k0 + kk) * N + n0 + n) : 0.f;
            }
            __syncthreads();
#pragma unroll
            for (int kk = 0; kk < BK; ++kk) {
                float a[4], b0[4], b1[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) a[i] = sA[kk][ty * 4 + i];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    b0[j] = sB0[kk][tx * 4 + j];
                    if (MODE == 0) b1[j] = sB1[kk][tx * 4 + j];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        acc0[i][j] = fmaf(a[i], b0[j], acc0[i][j]);
                        if (MODE == 0) acc1[i][j] = fmaf(a[i], b1[j], acc1[i][j]);
                    }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = ty * 4 + i;
            if (m >= te.rows) continue;
            const size_t row = (size_t)te.row0 + m;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = n0 + tx * 4 + j;
                if (n >= N) continue;
                if (MODE == 0) {
                    float av = acc0[i][j], bv = acc1[i][j];
                    if (act != nullptr) {
                        Elem<T>::store(act + row * ldact + n, av);
                        Elem<T>::store(act + row * ldact + N + n, bv);
                    }
                    Elem<T>::store(C + row * ldc + n, silu_mul(av, bv));
                } else {
                    Elem<T>::store(C + row * ldc + n, acc0[i][j]);
                }
            }
        }
    }
}

}  // namespace

int launch_tile_map(const fine_shape& s, const int32_t* seg_off, int rank_lo, int rank_hi, int BM, bool sole,
                    TileEntry* tiles, int32_t* count, int max_tiles, hipStream_t st) {
    if (rank_hi - rank_lo == 1 && s.E <= kMapThreads)
        hipLaunchKernelGGL(k_tile_map_rank, dim3(1), dim3((unsigned)align_up(s.E, 64)), 0, st,
                           seg_off + (size_t)rank_lo * (s.E + 1), s.E, BM, tiles, count, max_tiles);
    else {
        const int n_ranks = rank_hi - rank_lo;
        const size_t runs = sole ? (size_t)s.E * 4 : 0, lds = (size_t)n_ranks * (s.E + 1) * 4 + runs;
        hipLaunchKernelGGL(lds <= kMapLds ? k_tile_map<true> : k_tile_map<false>, dim3(1),
                           dim3((unsigned)std::min<size_t>(kMapThreads, align_up((size_t)n_ranks * s.E, 64))), lds <= kMapLds ? lds : runs, st,
                           seg_off, s.E, rank_lo, rank_hi, BM, (int)sole, tiles, count, max_tiles);
    }
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

FfnWs ffn_ws_layout(const fine_shape& s) {
    FfnWs w;
    const size_t P = (size_t)s.T * s.K;
    // smallest row tile is 32: at most P/32 full tiles plus one ragged tile per segment
    w.max_tiles = (int)(P / 32 + (size_t)s.E * s.G + 1);
    size_t o = 0;
    w.h = o;     o = align_up(o + P * s.f * elem_size(s.dtype), 256);
    w.tiles = o; o = align_up(o + (size_t)w.max_tiles * sizeof(TileEntry), 256);
    w.count = o; o = align_up(o + kCountBytes, 256);
    w.sk = o;    o = align_up(o + (s.dtype == FINE_BF16 ? kSkBytes : 0), 256);
    w.total = o;
    return w;
}

template <typename T>
static int ffn_simple_t(const fine_shape& s, int rank_lo, int rank_hi, const void* x_perm, const void* wg,
                        const void* wu, const void* wd, const int32_t* seg_off, void* y_perm, void* act_save,
                        char* ws, hipStream_t st) {
    const FfnWs L = ffn_ws_layout(s);
    auto* tiles = reinterpret_cast<TileEntry*>(ws + L.tiles);
    auto* count = reinterpret_cast<int32_t*>(ws + L.count);
    T* h = reinterpret_cast<T*>(ws + L.h);
    if ((s.flags & FINE_FLAG_ACT_SAVE_H) && act_save != nullptr)      // H behind the saved pre-activations
        h = static_cast<T*>(act_save) + (size_t)s.T * s.K * 2 * s.f;
    FINE_TRY(launch_tile_map(s, seg_off, rank_lo, rank_hi, 64, false, tiles, count, L.max_tiles, st));
    const int grid = 2048;
    hipLaunchKernelGGL((k_gemm_simple<T, 0>), dim3(grid), dim3(256), 0, st, (const T*)x_perm, s.d, (const T*)wg,
                       (const T*)wu, (size_t)s.d * s.f, s.d, s.f, h, s.f, (T*)act_save, 2 * s.f, tiles, count);
    FINE_LAUNCH_CHECK();
    hipLaunchKernelGGL((k_gemm_simple<T, 1>), dim3(grid), dim3(256), 0, st, (const T*)h, s.f, (const T*)wd,
                       (const T*)nullptr, (size_t)s.f * s.d, s.f, s.d, (T*)y_perm, s.d, (T*)nullptr, 0, tiles, count);
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

int launch_ffn_simple(const fine_shape& s, int rank_lo, int rank_hi, const void* x_perm,
                      const void* wg, const void* wu, const void* wd, const int32_t* seg_off,
                      void* y_perm, void* act_save, char* ws, hipStream_t st) {
    if (s.dtype == FINE_F32)
        return ffn_simple_t<float>(s, rank_lo, rank_hi, x_perm, wg, wu, wd, seg_off, y_perm, act_save, ws, st);
    return ffn_simple_t<uint16_t>(s, rank_lo, rank_hi, x_perm, wg, wu, wd, seg_off, y_perm, act_save, ws, st);
}

}  // namespace fine
