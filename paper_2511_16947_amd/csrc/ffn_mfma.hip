// Grouped SwiGLU expert FFN on bf16 MFMA over variable-length (rank, expert) segments.
//   GEMM 1: [A | B] = X [Wg | Wu] with the SwiGLU epilogue H = silu(A) * B.  The block's
//           n-tile interleaves 32 gate columns with the matching 32 up columns, so every
//           wave holds both halves of each H element in registers.
//   GEMM 2: Y = H Wd.
// Both run as persistent kernels over a device-built work list (row tile x column
// tile), so that nothing about segment lengths has to reach the host.
#include <cmath>

#include "gemm_w8.h"

namespace fine {

namespace {

using namespace mfma;

// silu(a) * b with the hardware reciprocal (1 ulp), far inside the bf16 rounding of the result
__device__ inline float silu_mul(float a, float b) { return a * b * __builtin_amdgcn_rcpf(1.f + __expf(-a)); }

// EPI 0: GEMM 1 (A = x_perm, B0/B1 = Wg/Wu [E,Kd,N]; C = H [P,N]; act [P,2N] optional)
// EPI 1: GEMM 2 (A = H, B0 = Wd [E,Kd,N]; C = y_perm [P,N])
// 8 waves (see gemm_w8.h); the tiles that do not fill a whole round of the grid are cut along
// k so that every block gets the same number of k-steps (sk_partials, sk_counters below).
//
// Row tiles.  The list cuts a run of rows into tiles of BM = 256 or 128 rows; one of at most 128 rows (a whole short run, or
// the end of a longer one) is computed on 128 rows in either case: half the MFMAs and three quarters of the operand
// traffic, about 0.65 of a 256-row tile's time.  So with BM = 256 every run is cut as its own length wants it: 32768 rows on
// 254 experts of 7168 x 2048 (mean 129 rows, longest 1477), both GEMMs 5440 -> 5370 us against 128-row tiles throughout; 32768
// rows on 115 experts of 2048 x 768 446 -> 432 us.
template <int WAVES_M, int WAVES_N, int WN, int EPI>
__device__ __forceinline__ void ffn_gemm_body(const uint16_t* __restrict__ A, int lda, const uint16_t* __restrict__ B0,
                                              const uint16_t* __restrict__ B1, size_t b_expert_stride, int Kd, int N,
                                              uint16_t* __restrict__ C, int ldc, uint16_t* __restrict__ act,
                                              const TileEntry* __restrict__ tiles, int32_t* __restrict__ count,
                                              float* __restrict__ sk_partials, int may_cut, int tall, int nt_from) {
    constexpr int BN = WAVES_N * WN * 32;
    constexpr int BNC = (EPI == 0) ? BN / 2 : BN;      // output columns per block
    static_assert(WAVES_M == 2 && WAVES_N == 4 && WN == 2, "2 x 4 waves on 256 x 256 or 128 x 256");
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int ntn = (N + BNC - 1) / BNC;
    const int nk = Kd / BK;
    const int ntm = *count;
    const int total = ntm * ntn;

    // acc += (rows of tile te) x (its weight columns from n0 on) over k-tiles [kb, kb + kn)
    auto run_tile = [&](auto& acc, const TileEntry& te, int n0, int kb, int kn) {
        constexpr int WM = sizeof(acc) / sizeof(f32x16) / WN, BM = WAVES_M * WM * 32;
        const uint16_t* Bg = B0 + (size_t)te.expert * b_expert_stride;
        const uint16_t* Bu = (EPI == 0) ? B1 + (size_t)te.expert * b_expert_stride : nullptr;
        auto k_tile = [&](int kt) { return KTile{(ptrdiff_t)(kb + kt) * BK, (ptrdiff_t)(kb + kt) * BK, Kd, 0}; };
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        RowDmaOperand<WM, BM> oa;
        // rows past the tile's last lie beyond the descriptor's size: the DMA writes zeros for them
        // and asks memory for nothing (their results are never stored)
        oa.init(A + (size_t)te.row0 * lda, [&](int r) { return (size_t)r * lda; },
                (uint32_t)((size_t)te.rows * lda * 2), (wave / WAVES_N) * WM * 32);
        const int wn = wave % WAVES_N;
        // fragments of the wave that hold valid rows (the rest of a short last tile is skipped)
        const int nf = min(WM, max(0, (te.rows - (wave / WAVES_N) * WM * 32 + 31) / 32));
        auto k_range = [&](auto ragged, auto nt) {
            DmaOperand<WN, nt.value> ob;
            if constexpr (EPI == 0) {
                // panel 0 = 128 gate columns, panel 1 = the matching up columns; a wave's two
                // fragments are the same 32 columns of both
                ob.init(Bg, Bu, [&](int, int c) { return min(n0 + 8 * c, N - 8); }, (size_t)N,
                        [&](int f) { return 128 * f + 32 * wn; });
            } else {
                ob.init(Bg, Bg, [&](int p, int c) { return min(n0 + 128 * p + 8 * c, N - 8); }, (size_t)N,
                        [&](int f) { return 64 * wn + 32 * f; });
            }
            k_loop8<ragged.value, 4>(kn, smem, acc, oa, ob, k_tile, nf);
        };
        // Weights that nobody reads again (see nt_from) bypass the caches, which leaves those to the activations and to weights
        // that are; a tile of exactly BM rows takes the form without row tests, which has one policy: 32 rows on each of 64 experts of 7168 x 2048, both GEMMs 985 -> 894 us (5.7 -> 6.3
        // TB/s); 8192 rows on them (half of the runs one tile) 1254 -> 1219; 10725 rows on 144 of 3776 x 512 394 -> 361; where most
        // runs have several tiles nothing changes.  (Non-temporal throughout is 7 % slower: then weights are shared.)
        if (te.rows == BM) k_range(std::false_type{}, std::false_type{});
        else if (te.alone >= nt_from) k_range(std::true_type{}, std::true_type{});
        else k_range(std::true_type{}, std::false_type{});
    };

    // LDS-staged epilogue of tile te, 8-byte coalesced stores
    auto epilogue = [&](auto& acc, const TileEntry& te, int n0) {
        constexpr int WM = sizeof(acc) / sizeof(f32x16) / WN, BM = WAVES_M * WM * 32;
        constexpr int WMC = (BM * (BNC * 2 + 8) <= 2 * (BM + BN) * 128) ? WM : WM / 2;
        if constexpr (EPI == 0) {
            if (act != nullptr) {
                store_tile_bf16<WAVES_M, WAVES_N, WM, WN / 2, WMC>(
                    smem, [&](auto mi, auto t, auto rg, auto q) { return acc[mi.value][2 * t.value][4 * rg.value + q.value]; },
                    act, (size_t)(2 * N), te.row0, te.rows, n0, N);
                store_tile_bf16<WAVES_M, WAVES_N, WM, WN / 2, WMC>(
                    smem, [&](auto mi, auto t, auto rg, auto q) { return acc[mi.value][2 * t.value + 1][4 * rg.value + q.value]; },
                    act + N, (size_t)(2 * N), te.row0, te.rows, n0, N);
            }
            store_tile_bf16<WAVES_M, WAVES_N, WM, WN / 2, WMC>(
                smem,
                [&](auto mi, auto t, auto rg, auto q) {
                    return silu_mul(acc[mi.value][2 * t.value][4 * rg.value + q.value],
                                    acc[mi.value][2 * t.value + 1][4 * rg.value + q.value]);
                },
                C, (size_t)ldc, te.row0, te.rows, n0, N);
        } else {
            store_tile_bf16<WAVES_M, WAVES_N, WM, WN, WMC>(
                smem, [&](auto mi, auto t, auto rg, auto q) { return acc[mi.value][t.value][4 * rg.value + q.value]; },
                C, (size_t)ldc, te.row0, te.rows, n0, N);
        }
    };

    // Whole tiles first: as many full rounds of the grid as there are.  The remaining rest < nblk tiles are rest * nk k-steps, cut into nblk parts: part p is
    // steps [p * per, (p+1) * per) of that sequence.  Whoever computes only part of a tile's k
    // range counts itself in when its k-loop is done; all but the last to do so write their
    // accumulators to their part's slot (two per part: a range begins and ends inside at most one
    // tile each) and count themselves ready; the last keeps its accumulators, waits until the others
    // are ready (they are past their k-loops and wait for nothing), adds the parts up in part order -
    // the same sum whoever it is - and runs the epilogue.  Partial sums are traffic at the end of a
    // launch, when every block has them at once: one write and one read per part that is not last.
    // (A rest too small for the cut to pay is cut into few parts instead, see below.)
    __shared__ int s_last, s_next;
    const int nblk = gridDim.x, bid = xcd_contiguous_id();
    // the cut pays when the k-steps it saves (the last round would take nk, the cut takes
    // rest * nk / nblk) outweigh writing, re-reading and adding up partial tiles.  Measured
    // break-even: about 16 steps on the 256-row tile (GEMM 2 of a rank with 128 tiles of 224 steps
    // gains 30 %, half a round of 64-step GEMM 1 tiles a little); on the 128-row tile, whose
    // workloads stream weights from HBM, the cut only pays for long k ranges (32 steps).
    const int whole_rounds = may_cut ? (total / nblk) * nblk : total;
    const int rest_if = total - whole_rounds;
    const bool cut_even = 4 * rest_if >= nblk && (long long)nk * (nblk - rest_if) > (long long)(tall ? 16 : 32) * nblk;
    // A rest of less than a quarter of a round, or one below that break-even, would still cost a whole extra round (24 of
    // 280 tiles of 32 steps: one more tile time with 232 CUs idle).  Spread over the whole grid each of its tiles would have
    // four and more parts, up to 32, for its last block to add up; instead every rest tile is cut into p parts ("few parts"),
    // the more the longer k: a part costs its nk / p steps, and p partial tiles about as much as 5 p steps (4 p on 128 rows; all
    // alone in the launch, and so at the same time, another rest / 12 each).
    // Parts go to the XCDs in equal numbers (`dealt`): in eighths of a round, as tiles do, 16 tiles in four parts would be the work
    // of two XCDs with a fourth of the memory path.  After whole rounds sixteen parts stay on one XCD: with 16 to 24 steps the
    // launch takes 1 us (3 %) longer otherwise.  More than 7/8 of a round are left as they lie (60 tiles in four parts 4-6 % slower dealt).
    // A tile's parts are consecutive units after whole rounds (304 tiles of 128 steps 277 us, 292 with its parts `rest` apart), but
    // `rest` apart where they are all there is (56 tiles of 128 steps 99 consecutive, 81 so; on 128 rows 68 and 60).
    // GEMM 2, us, spread over the grid : four parts, not dealt : now.  A round and 8, 16, 32, 48, 56 tiles of 256 rows: 32 steps
    // 151 : 92 : 86, 118 : 99 : 87, 105 : 104 : 89, 103 : 107 : 92, 102 : 104 : 94; 128 steps 346 : 258 : 250, 290 : 277 : 252, 278 : 280 : 261,
    // 287 : 277 : 274, 297 : 280 : 274; 224 steps 480 : 427 : 408, 431 : 452 : 410, 438 : 456 : 424, 473 : 465 : 448, 492 : 460 : 459; of 128
    // rows, 128 steps 182 : 165 : 156, 165 : 163 : 155, 164 : 165 : 163, 174 : 166 : 170, 178 : 170 : 172.  8, 16, 32, 48, 56 tiles alone: 256 rows, 64
    // steps 103 : 51 : 46, 71 : 59 : 47, 63 : 64 : 51, 66 : 67 : 57, 71 : 66 : 61; 224 steps 112 : 98 : 70, 91 : 119 : 75, 114 : 125 : 102, 140 :
    // 123 : 126, 156 : 127 : 128; 128 rows, 128 steps 59 : 46 : 34, 48 : 45 : 36, 51 : 56 : 40, 62 : 60 : 51, 71 : 63 : 58.
    // A rest of more than half a round (and GEMMs whose tiles share weight panels: the 256-row tile) is cut in
    // GROUPS instead: q consecutive rest tiles (same column, adjacent rows) share q + 1 parts of q nk / (q + 1)
    // steps, q = ceil(rest / (nblk - rest)), so that every tile is made of exactly two parts (one write, one
    // read, the last one keeps its own), no part touches more than two tiles, and the tiles of a group
    // walk their weight panel nearly together.  Parts are a little longer than with the even cut over the
    // whole grid (72 -> 86 of 128 steps for 144 tiles) and some blocks stay idle, but measured on one expert
    // with n whole row tiles at the training shape's GEMM 2 (8 column tiles, 128 k-steps) the even cut took
    // 192-241 us for n = 17 ... 22 where its step count says 110-145.
    int grp = 0;
    if (tall && 2 * rest_if > nblk && rest_if < nblk) {
        const int q = (rest_if + (nblk - rest_if) - 1) / (nblk - rest_if);
        if (nk > 16 * (q + 1)) grp = q;      // what a part saves against a whole tile, nk / (q + 1) steps, must pay for a partial tile
    }
    const bool cut = cut_even && grp == 0;
    int few = 0;
    if (!cut && grp == 0 && rest_if > 0) {
        const int fit = nblk / rest_if, most = min(fit >= 4 ? fit : min(fit, 2), nk / 8);      // (at least 8 steps each)
        const int price = 12 * (tall ? 5 : 4) + (whole_rounds == 0 ? rest_if : 0);             // of a partial tile, in 1 / 12 steps
        int p = min(most, 2);
        while (p < most && price * p * (p + 1) < 12 * nk) ++p;
        few = p > 1 ? p : 0;
    }
    const int full = (cut || few || grp) ? whole_rounds : total;
    const int rest = total - full;
    const int per = (rest * nk + nblk - 1) / nblk;
    const int n_groups = grp ? (rest + grp - 1) / grp : 0;
    const int nparts = cut ? nblk : grp ? rest + n_groups : rest * few;
    // (the units of a round are its 256 places, 32 for each XCD: dealt, the first nparts / 8 of these hold a part)
    const bool dealt = few && 8 * nparts <= 7 * nblk && (full == 0 || nparts > 16);
    const int few_step = full == 0 ? rest : 1;      // between the parts of a tile
    int32_t* counters = count + kSkCounterOffset;      // arrivals per rest tile
    int32_t* ready = count + kSkReadyOffset;           // parts written per rest tile
    // steps [u0, u1) of the sequence of rest tiles (tile t = steps [t nk, (t + 1) nk)) that part `part` computes
    auto part_range = [&](int part, int& u0, int& u1) {
        if (grp) {
            const int g = part / (grp + 1), i = part - g * (grp + 1);
            const int tiles_g = min(grp, rest - g * grp);      // the last group may be shorter
            const int steps_g = tiles_g * nk;
            u0 = g * grp * nk + (int)((long long)i * steps_g / (tiles_g + 1));
            u1 = g * grp * nk + (int)((long long)(i + 1) * steps_g / (tiles_g + 1));
            if (i > tiles_g) u0 = u1 = 0;                      // (no such part: a shorter last group has fewer)
        } else {
            u0 = min(rest * nk, part * per);
            u1 = min(rest * nk, u0 + per);
        }
    };
    // a part's slot for its piece of tile t: 0 if the part begins in t, else 1 (few parts: one piece per part)
    auto slot_of = [&](int part, int t) {
        if (few) return part * 2;
        int u0, u1;
        part_range(part, u0, u1);
        return part * 2 + (u0 / nk == t ? 0 : 1);
    };
    // Partial sums travel as 16-byte buffer stores and loads with the sc0 sc1 cache policy: they
    // are written through and read past the per-XCD L2 one by one, so no cache-wide write-back or
    // invalidate (a fence) is needed, which would cost every block on the XCD its cached operand
    // tiles.  A slot is [WM*WN*4 groups][threads] x 16 bytes; group g of a thread = registers
    // 4 (g & 3) .. + 3 of accumulator tile g >> 2.  Two accumulator tiles' worth of loads (8 x 16
    // bytes per lane) are in flight at a time.
    constexpr int kThreadsBlk = WAVES_M * WAVES_N * 64;
    constexpr int kSlotBytes = kSkSlotBytes;
    static_assert(4 * WN * 4 * kThreadsBlk * 16 == kSlotBytes, "a 256-row tile");
    constexpr int kCoherent = 1 | 16;      // sc0 | sc1
    const __amdgpu_buffer_rsrc_t sk_rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)sk_partials, 0, (int)(2 * 256 * (size_t)kSlotBytes), 0x00020000);

    // Who computes what: the units of a launch are its whole tiles [0, full) and then its parts
    // [full, full + nparts), handed out by UnitQueue (counters zeroed by k_tile_map).
    UnitQueue uq;
    uq.init(count + kQueueOffset + (EPI * 8) * kQueueStride, kQueueStride, full + (dealt ? nblk : nparts), bid, true);
    auto request = [&]() { uq.request(); };

    // k-tiles [kb, kb + kn) of tile `work`; part: the part this piece belongs to (-1: a whole tile);
    // ask: request the next unit after the k-loop
    auto piece_of = [&](auto wm_c, const TileEntry& te, int n0, int work, int kb, int kn, int part, bool ask) {
        constexpr int WM = wm_c.value;
        f32x16 acc[WM][WN];
        zero_acc<WM, WN>(acc);
        run_tile(acc, te, n0, kb, kn);
        if (ask) request();
        bool finish = true;
        if (kn != nk) {
            const int t = work - full;
            // the parts that hold pieces of tile t: first, first + step, ... (n_parts of them)
            const int first = few ? (few_step == 1 ? t * few : t) : grp ? (t / grp) * (grp + 1) + t % grp : (t * nk) / per;
            const int n_parts = few ? few : grp ? 2 : (t * nk + nk - 1) / per - first + 1;
            // Whoever arrives last (everybody else has left its k-loop by then) adds the parts up; the
            // others write theirs to their slots and then count themselves ready.  The tile is
            // part 0 + part 1 + part 2 + ... in that order whoever adds: if the last one holds part 0 or
            // part 1 it keeps it in its accumulators (x + y = y + x to the bit, so the chain may start
            // from either of the two) and reads only the others; if it holds a later part it writes that
            // one too and reads them all.
            if (threadIdx.x == 0)
                s_last = __hip_atomic_fetch_add(&counters[t], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                         n_parts - 1;
            __syncthreads();
            finish = s_last != 0;
            const int step = few ? few_step : 1, my_idx = (part - first) / step;
            const bool keep = finish && my_idx <= 1;
            if (!keep) {
                const int mine = slot_of(part, t);
                static_for<WM * WN>([&](auto m) {
                    static_for<4>([&](auto q) {
                        const f32x16& v = acc[m.value / WN][m.value % WN];
                        const f32x4 val = {v[4 * q.value], v[4 * q.value + 1], v[4 * q.value + 2], v[4 * q.value + 3]};
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, val), sk_rs, threadIdx.x * 16,
                                                               mine * kSlotBytes + (m.value * 4 + q.value) * kThreadsBlk * 16,
                                                               kCoherent);
                    });
                });
                __builtin_amdgcn_s_waitcnt(0x0070);      // vmcnt(0): this thread's partial sums have been written
                __syncthreads();
                if (!finish && threadIdx.x == 0)
                    __hip_atomic_fetch_add(&ready[t], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (finish) {
                // The others are past their k-loops and on their way through the lines above, which wait
                // for nothing but their own stores: this wait ends.  (The bound only keeps a mistake
                // elsewhere from hanging the launch: the sums would then be wrong, not the GPU stuck.)
                if (threadIdx.x == 0) {
                    int polls = 0;
                    while (__hip_atomic_load(&ready[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n_parts - 1 &&
                           ++polls < (1 << 20))
                        __builtin_amdgcn_s_sleep(4);
                    ready[t] = 0;          // both counters are zero again for the next launch
                    counters[t] = 0;
                }
                __syncthreads();
                auto add_part = [&](int i, auto assign) {
                    const int sl = slot_of(first + i * step, t);
                    static_for<WM * WN / 2>([&](auto mp) {
                        u32x4 v[8];
                        static_for<8>([&](auto g) {
                            v[g.value] = __builtin_amdgcn_raw_buffer_load_b128(
                                sk_rs, threadIdx.x * 16, sl * kSlotBytes + (mp.value * 8 + g.value) * kThreadsBlk * 16, kCoherent);
                        });
                        static_for<8>([&](auto g) {
                            constexpr int m = mp.value * 2 + g.value / 4, q = g.value % 4;
                            const f32x4 val = __builtin_bit_cast(f32x4, v[g.value]);
                            f32x16& a = acc[m / WN][m % WN];
                            if constexpr (assign.value) {
                                a[4 * q] = val[0]; a[4 * q + 1] = val[1]; a[4 * q + 2] = val[2]; a[4 * q + 3] = val[3];
                            } else {
                                a[4 * q] += val[0]; a[4 * q + 1] += val[1]; a[4 * q + 2] += val[2]; a[4 * q + 3] += val[3];
                            }
                        });
                        __builtin_amdgcn_sched_barrier(0);      // keeps the loads from piling up in registers
                    });
                };
                if (!keep) add_part(0, std::true_type{});
                for (int i = keep ? 0 : 1; i < n_parts; ++i)
                    if (!(keep && i == my_idx)) add_part(i, std::false_type{});
            }
            __syncthreads();
        }
        if (finish) epilogue(acc, te, n0);
    };
    auto piece = [&](int work, int kb, int kn, int part, bool ask) {
        int tm, tn;
        tile_of_work(work, ntm, ntn, tm, tn);
        const TileEntry te = tiles[tm];
        if (te.rows > 128) piece_of(IntC<4>{}, te, tn * BNC, work, kb, kn, part, ask);
        else piece_of(IntC<2>{}, te, tn * BNC, work, kb, kn, part, ask);
    };

    for (int v = uq.first(bid); v >= 0; v = uq.next(v, &s_next)) {
        if (v < full) {
            piece(v, 0, nk, -1, true);
        } else if (few) {
            int part = v - full;
            if (dealt) {
                const int per_x = nblk / 8, x = part / per_x, at = nparts * x / 8 + part - x * per_x;
                part = at < nparts * (x + 1) / 8 ? at : -1;
            }
            if (part < 0) {
                lds_barrier();      // (no k-loop, whose barriers keep the queue's s_next until every wave has read it)
                request();
            } else {
                const int t = few_step == 1 ? part / few : part % rest, i = few_step == 1 ? part - t * few : part / rest;
                piece(full + t, nk * i / few, nk * (i + 1) / few - nk * i / few, part, true);
            }
        } else {
            const int part = v - full;
            int u, u1;
            part_range(part, u, u1);
            if (u >= u1) {      // (an empty part at the end of the sequence)
                lds_barrier();
                request();
            }
            while (u < u1) {
                const int t = u / nk, kb = u - t * nk, kn = min(nk - kb, u1 - u);
                piece(full + t, kb, kn, part, u + kn >= u1);
                u += kn;
            }
        }
    }
}

// 8 waves: two per SIMD, each with 128 architectural and 128 accumulator registers
template <int EPI>
__global__ __launch_bounds__(512) void k_ffn_gemm_w8(const uint16_t* __restrict__ A, int lda,
                                                     const uint16_t* __restrict__ B0, const uint16_t* __restrict__ B1,
                                                     size_t b_expert_stride, int Kd, int N,
                                                     uint16_t* __restrict__ C, int ldc, uint16_t* __restrict__ act,
                                                     const TileEntry* __restrict__ tiles, int32_t* __restrict__ count,
                                                     float* __restrict__ sk_partials, int may_cut, int tall, int nt_from) {
    ffn_gemm_body<2, 4, 2, EPI>(A, lda, B0, B1, b_expert_stride, Kd, N, C, ldc, act, tiles, count, sk_partials, may_cut, tall, nt_from);
}

// BM: rows of the list's tiles, 256 or 128
int run_ffn(const fine_shape& s, int BM, int rank_lo, int rank_hi, const void* x_perm, const void* wg, const void* wu,
            const void* wd, const int32_t* seg_off, void* h_buf, void* y_perm, void* act_save, TileEntry* tiles,
            int32_t* count, int max_tiles, float* sk_partials, bool gemm1, bool gemm2, bool may_cut, hipStream_t st) {
    auto* h = reinterpret_cast<uint16_t*>(h_buf);
    const int nt = nt_from(s, 2, rank_hi - rank_lo);
    FINE_TRY(launch_tile_map(s, seg_off, rank_lo, rank_hi, BM, nt == 2, tiles, count, max_tiles, st));
    const size_t lds = (size_t)w8_lds_bytes(true, 4);
    static std::atomic<uint64_t> lds_set1{0}, lds_set2{0};
    FINE_TRY(raise_lds_limit((const void*)k_ffn_gemm_w8<0>, (int)lds, lds_set1));
    FINE_TRY(raise_lds_limit((const void*)k_ffn_gemm_w8<1>, (int)lds, lds_set2));
    const int grid = 256;      // one block per CU
    if (gemm1) {
        hipLaunchKernelGGL(k_ffn_gemm_w8<0>, dim3(grid), dim3(512), lds, st, (const uint16_t*)x_perm, s.d, (const uint16_t*)wg,
                           (const uint16_t*)wu, (size_t)s.d * s.f, s.d, s.f, h, s.f, (uint16_t*)act_save, tiles, count,
                           sk_partials, (int)may_cut, (int)(BM == 256), nt);
        FINE_LAUNCH_CHECK();
    }
    if (gemm2) {
        hipLaunchKernelGGL(k_ffn_gemm_w8<1>, dim3(grid), dim3(512), lds, st, (const uint16_t*)h, s.f, (const uint16_t*)wd,
                           (const uint16_t*)nullptr, (size_t)s.f * s.d, s.f, s.d, (uint16_t*)y_perm, s.d,
                           (uint16_t*)nullptr, tiles, count, sk_partials, (int)may_cut, (int)(BM == 256), nt);
        FINE_LAUNCH_CHECK();
    }
    return FINE_OK;
}

// Tile choice.
//   3: tiles of 256 rows x 256 columns on 8 waves, those of at most 128 rows on 128 - the fastest per row where runs are long
//      (the tiles of an incomplete last round are cut along k, so few tiles are no problem), and in launches of many rounds
//      also where most are short;
//   2: tiles of 128 rows: in launches of a few rounds it counts how full the last one is and how long, and a short tile's is
//      shorter (4096 rows on 5-13 experts of 2048 x 768, one rank, GEMM 1 / GEMM 2: 36 / 28 us against 53 / 26);
//   1: 64 rows, k split over the waves of a block (ffn_stream.hip).
// 1 is for two kinds of call.  A few rows per expert (decoding): both kernels stream weights, at 5.7 TB/s against 5.2
// (7 experts of 4096 x 14336, 32 rows: 428 against 483 us; 32 of 2048 x 5632, 128 rows: 239 against 247; but 46 experts
// of 2048 x 1408 with 45 rows on average, the longest 429: 198 against 181).  And launches that leave most of the
// CUs without a tile, each of the others waiting out a chain of k-steps: 10 row tiles of 128 on 1088 x 832, 133 tiles
// in both GEMMs, 28 against 43 us per rank; 204 tiles 37 against 47; 286 tiles 51 against 60; 351 tiles 51 against 48.
int pick_tile(const fine_shape& s, int n_ranks) {
    if (!w8_offsets_fit(s)) return 1;
    const int tile = (s.flags & FINE_FLAG_TILE_MASK) >> FINE_FLAG_TILE_SHIFT;
    if (tile != 0) return tile;
    // expected runs of rows of one expert when every expert is on every rank: the rows of n ranks, P / G each, span
    // about n E / G + 1 experts
    const double rows = (double)s.T * s.K * n_ranks / s.G, runs = (double)s.E * n_ranks / s.G + 1.0;
    if (rows / runs < 24.0) return 1;
    const double tiles = (rows / 128.0 + runs) * (cdiv(s.f, 128) + cdiv(s.d, 256));
    if (tiles < 320.0) return 1;
    // (from three rounds of 256-row tiles on in both GEMMs)
    return rows / runs >= 384.0 || rows / 256.0 * std::min(cdiv(s.f, 128), cdiv(s.d, 256)) >= 768.0 ? 3 : 2;
}

}  // namespace

// any_ranks (the backward pass): the same bits whether a call is for one rank or for all, so the tile may not depend on
// the number of ranks, and no tile is cut along k (which tiles a launch cuts, and where, depends on how many it has).
int launch_ffn_parts(const fine_shape& s, int rank_lo, int rank_hi, const void* x_perm, const void* wg,
                     const void* wu, const void* wd, const int32_t* seg_off, void* h_buf, void* y_perm,
                     void* act_save, TileEntry* tiles, int32_t* count, int max_tiles, float* sk_partials, bool gemm1,
                     bool gemm2, bool any_ranks, hipStream_t st) {
    const int tile = pick_tile(s, any_ranks ? s.G : rank_hi - rank_lo);
    if (tile == 1)
        return launch_ffn_stream(s, rank_lo, rank_hi, x_perm, wg, wu, wd, seg_off, h_buf, y_perm, act_save, tiles, count,
                                 max_tiles, gemm1, gemm2, st);
    return run_ffn(s, tile == 2 ? 128 : 256, rank_lo, rank_hi, x_perm, wg, wu, wd, seg_off, h_buf, y_perm, act_save, tiles,
                   count, max_tiles, sk_partials, gemm1, gemm2, !any_ranks, st);
}

int launch_ffn_mfma(const fine_shape& s, int rank_lo, int rank_hi, const void* x_perm,
                    const void* wg, const void* wu, const void* wd, const int32_t* seg_off,
                    void* y_perm, void* act_save, char* ws, hipStream_t st) {
    const FfnWs L = ffn_ws_layout(s);
    // H: in the workspace, or behind the saved pre-activations when the caller keeps it for the backward pass
    void* h_buf = ws + L.h;
    if ((s.flags & FINE_FLAG_ACT_SAVE_H) && act_save != nullptr)
        h_buf = static_cast<char*>(act_save) + (size_t)s.T * s.K * 2 * s.f * elem_size(s.dtype);
    return launch_ffn_parts(s, rank_lo, rank_hi, x_perm, wg, wu, wd, seg_off, h_buf, y_perm, act_save,
                            reinterpret_cast<TileEntry*>(ws + L.tiles), reinterpret_cast<int32_t*>(ws + L.count),
                            L.max_tiles, reinterpret_cast<float*>(ws + L.sk), !(s.flags & FINE_FLAG_ONLY_GEMM2),
                            !(s.flags & FINE_FLAG_ONLY_GEMM1), false, st);
}

}  // namespace fine

