// Grouped SwiGLU expert FFN for small launches (decoding, small micro-batches): bf16 MFMA with the CONTRACTION split
// over the waves of a block.
//
// With few rows per expert the kernel is a weight stream with MFMAs on the side, and a launch of few tiles is a chain
// of memory latencies on few CUs; what counts is bytes in flight and small tiles.  A block of 4 waves computes up to
// 64 rows x 128 columns (GEMM 1: 64 gate columns and the matching 64 up columns, so that SwiGLU is applied in
// registers); each wave streams its own quarter of k through its own LDS by DMA, so that there is no barrier in the
// k-loop and no wave waits for another's memory; the four partial tiles are added in LDS at the end.  20 KB of LDS
// per wave: two blocks per CU, one streaming while the other adds up and stores.
//
// Weights: a ring of stages of 16 k-rows, two panels of [16 k][64 columns] each (rows of 128 bytes; GEMM 2: panel 1 =
// the next 64 columns).  MFMA fragments are read with the transposing LDS read (lane layout in gemm_w8.h); the two
// 64-byte halves of a k-row are swapped where bit 1 of k is set, so that the four k-rows x 64 bytes that half a wave
// reads lie in distinct banks.  Activations: [rows][64 k], whole cache lines per row (loading them to registers as
// the MFMAs want them, 32 bytes of 32 rows per instruction, fetched every line twice to four times and cost 10-30 %
// of the kernel); a step's fragments are read at its start, which frees the buffer for the next step's.
//
// Measured, both GEMMs of a call, against the register-staged 64 x 256 kernel that this one replaced: 128 rows on 8
// experts of 4096 x 14336: 1020 -> 499 us (5.6 TB/s of weights); 1024 rows on 45 used experts of 2048 x 768: 134 ->
// 88 us; against the 128-row tiles of ffn_mfma.hip: 783 rows on 4 experts of 1088 x 832, per rank: 43 -> 28 us.
#include "gemm_w8.h"

namespace fine {

namespace {

using namespace mfma;

constexpr int kStreamRows = 64, kStreamStage = 4096, kStreamWave = 20 * 1024;

__device__ inline float silu_mul(float a, float b) { return a * b * __builtin_amdgcn_rcpf(1.f + __expf(-a)); }

// A wave's operands of one tile: activations A (rows of `lda` elements, a_bytes valid bytes) and the weight panels
// W0, W1 (element (k = 0, column 0 of the tile); k-rows of N elements).  NF: fragments of 32 rows.  The wave's LDS:
// the ring, then the activations.
// NT: the weights are fetched with the non-temporal policy.
template <int NF, bool NT>
struct StreamOperands {
    static constexpr int R = NF == 1 ? 4 : 3;             // stages of the ring
    static constexpr int kA = R * kStreamStage;
    static_assert(kA + NF * 4096 <= kStreamWave, "LDS of a wave");
    __amdgpu_buffer_rsrc_t ra;
    const uint16_t *w0, *w1;
    char* lds;
    uint32_t a_off[NF * 4], b_off, row8, fr[2], fa[4];
    int step_bytes, N;

    __device__ inline void init(const uint16_t* A, uint32_t a_bytes, int lda, const uint16_t* W0, const uint16_t* W1, int N_, char* lds_) {
        const int lane = threadIdx.x & 63;
        lds = lds_;
        const uint32_t base = (uint32_t)(uintptr_t)FINE_LDS_PTR(lds);
        // activations: a DMA instruction fills 8 rows; rows past the tile's last lie beyond the descriptor: zeros
        ra = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, (int)a_bytes, 0x00020000);
#pragma unroll
        for (int j = 0; j < NF * 4; ++j) {
            const int row = 8 * j + (lane >> 3);
            a_off[j] = (uint32_t)row * lda * 2u + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) fa[p] = base + kA + lds_off(lane & 31, 2 * p + (lane >> 5));
        // weights: a DMA instruction fills 8 k-rows of a panel; the swizzle is applied by choosing the source
        w0 = W0;
        w1 = W1;
        N = N_;
        const int krow = lane >> 3, chunk = (lane & 7) ^ (((krow >> 1) & 1) << 2);
        b_off = ((uint32_t)krow * N + 8 * chunk) * 2u;
        row8 = (uint32_t)N * 16u;                       // bytes of 8 k-rows
        step_bytes = (int)((uint32_t)N * 128u);         // of 64 k-rows: what a descriptor covers
        const int i = lane & 15, g = lane >> 4, cl = 2 * (g & 1) + ((i & 3) >> 1), sw = ((i >> 3) & 1) << 2;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            fr[t] = base + (uint32_t)((8 * (g >> 1) + (i >> 2)) * 128 + (((4 * t + cl) ^ sw) << 4) + (i & 1) * 8);
    }
    // requests the activations of step kt: 4 NF DMA instructions
    __device__ inline void issue_a(int kt) const {
        static_for<NF * 4>([&](auto j) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, FINE_LDS_PTR(lds + kA + j.value * 1024), 16, a_off[j.value], kt * 128, 0, 0);
        });
    }
    // requests stage S of step kt into the ring slot at byte `slot`: four DMA instructions
    template <int S>
    __device__ inline void issue_w(int kt, int slot) const {
        const size_t at = (size_t)kt * 64 * N;
        const __amdgpu_buffer_rsrc_t r0 = __builtin_amdgcn_make_buffer_rsrc((void*)(w0 + at), 0, step_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc((void*)(w1 + at), 0, step_bytes, 0x00020000);
        char* st = lds + slot;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r0, FINE_LDS_PTR(st), 16, b_off, 2 * S * row8, 0, NT ? 2 : 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r0, FINE_LDS_PTR(st + 1024), 16, b_off, (2 * S + 1) * row8, 0, NT ? 2 : 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r1, FINE_LDS_PTR(st + 2048), 16, b_off, 2 * S * row8, 0, NT ? 2 : 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r1, FINE_LDS_PTR(st + 3072), 16, b_off, (2 * S + 1) * row8, 0, NT ? 2 : 0);
    }
    // Fragment reads are blocks of assembly with their own waits: ahead of the builtin forms the compiler waits for
    // every DMA into LDS that is in flight, which would drain the ring at each stage.
    // the four fragments (32 columns each) of the stage at byte `slot`
    __device__ inline void frags_b(bf16x8 (&b)[4], int slot) const {
        v4i16 v[8];
        asm volatile(
            "ds_read_b64_tr_b16 %0, %8\n\t"
            "ds_read_b64_tr_b16 %1, %8 offset:512\n\t"
            "ds_read_b64_tr_b16 %2, %9\n\t"
            "ds_read_b64_tr_b16 %3, %9 offset:512\n\t"
            "ds_read_b64_tr_b16 %4, %8 offset:2048\n\t"
            "ds_read_b64_tr_b16 %5, %8 offset:2560\n\t"
            "ds_read_b64_tr_b16 %6, %9 offset:2048\n\t"
            "ds_read_b64_tr_b16 %7, %9 offset:2560\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
            : "v"(fr[0] + slot), "v"(fr[1] + slot)
            : "memory");
        static_for<4>([&](auto t) {
            b[t.value] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v[2 * t.value], v[2 * t.value + 1], 0, 1, 2, 3, 4, 5, 6, 7));
        });
    }
    // the four 16-k pieces of 32 rows of the activations
    template <int MI>
    __device__ inline void frags_a(u32x4 (&a)[4]) const {
        asm volatile(
            "ds_read_b128 %0, %4 offset:%c8\n\t"
            "ds_read_b128 %1, %5 offset:%c8\n\t"
            "ds_read_b128 %2, %6 offset:%c8\n\t"
            "ds_read_b128 %3, %7 offset:%c8\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
            : "v"(fa[0]), "v"(fa[1]), "v"(fa[2]), "v"(fa[3]), "n"(MI * 4096)
            : "memory");
    }
};

// One 64-k step: four stages.  NEXT: a step follows (its activations are requested).  cur: ring slot of its first
// stage; the slot of a stage is refilled with the stage R after it as soon as its fragments are in registers.
template <int NF, bool NEXT, bool NT>
__device__ __forceinline__ void stream_step(f32x16 (&acc)[NF][4], const StreamOperands<NF, NT>& o, int kt, int& cur) {
    constexpr int R = StreamOperands<NF, NT>::R;
    u32x4 a[NF][4];
    static_for<4>([&](auto s) {
        // Stage s (and at s = 0 the activations, requested before it) has landed when at most the requests made after
        // it are outstanding (vmcnt retires in order): the next R - 1 stages, 4 instructions each, as far as there
        // are any, and the next step's activations if the s = 0 of this step lies in between.
        constexpr int later = NEXT ? R - 1 : (R - 1 < 3 - s.value ? R - 1 : 3 - s.value);
        wait_vm_lgkm<4 * later + (NEXT && s.value >= 1 && s.value < R ? 4 * NF : 0)>();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (s.value == 0) static_for<NF>([&](auto mi) { o.template frags_a<mi.value>(a[mi.value]); });
        const int slot = R == 4 ? s.value * kStreamStage : cur;
        bf16x8 b[4];
        o.frags_b(b, slot);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NEXT && s.value == 0) o.issue_a(kt + 1);
        if constexpr (NEXT || s.value + R < 4) o.template issue_w<(s.value + R) & 3>(kt + (s.value + R) / 4, slot);
        if constexpr (R != 4) cur = cur == (R - 1) * kStreamStage ? 0 : cur + kStreamStage;
        __builtin_amdgcn_sched_barrier(0);
        static_for<NF>([&](auto mi) {
            static_for<4>([&](auto t) {
                acc[mi.value][t.value] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    b[t.value], __builtin_bit_cast(bf16x8, a[mi.value][s.value]), acc[mi.value][t.value], 0, 0, 0);
            });
        });
        __builtin_amdgcn_sched_barrier(0);
    });
}

// acc += the 64-k steps [0, nk)
template <int NF, bool NT>
__device__ __forceinline__ void stream_k(f32x16 (&acc)[NF][4], const StreamOperands<NF, NT>& o, int nk) {
    if (nk <= 0) return;
    o.issue_a(0);
    static_for<StreamOperands<NF, NT>::R>([&](auto s) { o.template issue_w<s.value>(0, s.value * kStreamStage); });
    __builtin_amdgcn_sched_barrier(0);
    int cur = 0;
    for (int kt = 0; kt + 1 < nk; ++kt) stream_step<NF, true, NT>(acc, o, kt, cur);
    stream_step<NF, false, NT>(acc, o, nk - 1, cur);
}

// EPI 0: A = x_perm [P,Kd], B0 / B1 = Wg / Wu [E,Kd,N], C = H [P,N]; act [P,2N] optional
// EPI 1: A = H [P,Kd], B0 = Wd [E,Kd,N], C = y_perm [P,N]
template <int EPI>
__global__ __launch_bounds__(256, 2) void k_ffn_stream(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0,
                                                       const uint16_t* __restrict__ B1, int Kd, int N,
                                                       uint16_t* __restrict__ C, uint16_t* __restrict__ act,
                                                       const TileEntry* __restrict__ tiles,
                                                       const int32_t* __restrict__ count,
                                                       const int32_t* __restrict__ seg, int E) {
    constexpr int BNC = EPI == 0 ? 64 : 128;      // output columns per block
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    RankTiles rank;      // seg != NULL: one rank, whose work list every wave makes for itself
    if (seg != nullptr) rank.init(seg, E, kStreamRows);
    const int ntn = (N + BNC - 1) / BNC, ntm = seg != nullptr ? rank.count : *count, total = ntm * ntn;
    const int nk = Kd / BK, kb = nk * wave / 4, kn = nk * (wave + 1) / 4 - kb;
    // an eighth of the tiles per XCD (blocks are dealt to them in turn), so that a last incomplete round lies on all
    const int xcd = blockIdx.x & 7, end = (int)((long long)total * (xcd + 1) / 8);
    for (int work = (int)((long long)total * xcd / 8) + (blockIdx.x >> 3); work < end; work += gridDim.x >> 3) {
        int tm, tn;
        tile_of_work(work, ntm, ntn, tm, tn);
        const TileEntry te = seg != nullptr ? rank.get(tm, kStreamRows) : tiles[tm];
        const int n0 = tn * BNC;
        const size_t w_at = (size_t)te.expert * Kd * N + (size_t)kb * BK * N + n0;
        const uint16_t* W0 = B0 + w_at;
        // (a last tile of 64 columns reads its panel twice; the second result is not stored)
        const uint16_t* W1 = EPI == 0 ? B1 + w_at : W0 + (n0 + 64 < N ? 64 : 0);
        const uint16_t* Ap = A + (size_t)te.row0 * Kd + (size_t)kb * BK;
        const uint32_t a_bytes = ((uint32_t)te.rows * Kd - kb * BK) * 2u;
        auto tile = [&](auto nf) {
            constexpr int NF = nf.value;
            f32x16 acc[NF][4];
            zero_acc<NF, 4>(acc);
            // Weights of a run of one tile bypass the caches (non-temporal): 8 % more from HBM.  (With
            // several tiles per run it would be the other way round: their weights come from the L2 but once.)
            auto k_range = [&](auto nt) {
                StreamOperands<NF, nt.value> o;
                o.init(Ap, a_bytes, Kd, W0, W1, N, smem + wave * kStreamWave);
                stream_k(acc, o, kn);
            };
            if (te.alone) k_range(std::true_type{});
            else k_range(std::false_type{});
            // Add the four waves' parts, 32 rows at a time: [wave][tile][column group rg][lane] x 16 bytes; wave w
            // takes group w of every tile.  The accumulators hold the transposed tiles (see acc_m, acc_n).
            static_for<NF>([&](auto mi) {
                lds_barrier();      // every wave has read its ring (or the previous rows' parts)
                static_for<4>([&](auto t) {
                    static_for<4>([&](auto rg) {
                        const f32x16& v = acc[mi.value][t.value];
                        *reinterpret_cast<f32x4*>(smem + wave * 16384 + t.value * 4096 + rg.value * 1024 + lane * 16) =
                            f32x4{v[4 * rg.value], v[4 * rg.value + 1], v[4 * rg.value + 2], v[4 * rg.value + 3]};
                    });
                });
                lds_barrier();
                f32x4 sum[4];
                static_for<4>([&](auto t) {
                    const char* p = smem + t.value * 4096 + wave * 1024 + lane * 16;
                    f32x4 s = *reinterpret_cast<const f32x4*>(p);
                    static_for<3>([&](auto w) { s += *reinterpret_cast<const f32x4*>(p + (w.value + 1) * 16384); });
                    sum[t.value] = s;
                });
                const int m = 32 * mi.value + (lane & 31), c = 8 * wave + 4 * (lane >> 5);
                if (m < te.rows) {
                    const size_t row = (size_t)te.row0 + m;
                    auto store = [&](uint16_t* p, f32x4 v) {
                        *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
                    };
                    if constexpr (EPI == 0) {
                        static_for<2>([&](auto t) {
                            const f32x4 x = sum[t.value], y = sum[2 + t.value];
                            const int n = n0 + 32 * t.value + c;
                            if (act != nullptr) {
                                store(act + row * (2 * (size_t)N) + n, x);
                                store(act + row * (2 * (size_t)N) + N + n, y);
                            }
                            store(C + row * N + n, f32x4{silu_mul(x[0], y[0]), silu_mul(x[1], y[1]), silu_mul(x[2], y[2]), silu_mul(x[3], y[3])});
                        });
                    } else {
                        static_for<4>([&](auto t) {
                            const int n = n0 + 32 * t.value + c;
                            if (n < N) store(C + row * N + n, sum[t.value]);
                        });
                    }
                }
            });
            lds_barrier();      // the next tile's DMA overwrites what slower waves may still read
        };
        if (te.rows <= 32) tile(IntC<1>{});
        else tile(IntC<2>{});
    }
}

}  // namespace

int launch_ffn_stream(const fine_shape& s, int rank_lo, int rank_hi, const void* x_perm, const void* wg, const void* wu,
                      const void* wd, const int32_t* seg_off, void* h_buf, void* y_perm, void* act_save, TileEntry* tiles,
                      int32_t* count, int max_tiles, bool gemm1, bool gemm2, hipStream_t st) {
    auto* h = reinterpret_cast<uint16_t*>(h_buf);
    const int32_t* seg = nullptr;
    if (rank_hi - rank_lo == 1 && s.E <= kRankMapExperts) seg = seg_off + (size_t)rank_lo * (s.E + 1);
    else FINE_TRY(launch_tile_map(s, seg_off, rank_lo, rank_hi, kStreamRows, false, tiles, count, max_tiles, st));
    const size_t lds = 4 * kStreamWave;
    static std::atomic<uint64_t> lds_set0{0}, lds_set1{0};
    FINE_TRY(raise_lds_limit((const void*)k_ffn_stream<0>, (int)lds, lds_set0));
    FINE_TRY(raise_lds_limit((const void*)k_ffn_stream<1>, (int)lds, lds_set1));
    const unsigned grid = 512;      // two blocks per CU
    if (gemm1) {
        hipLaunchKernelGGL(k_ffn_stream<0>, dim3(grid), dim3(256), lds, st, (const uint16_t*)x_perm, (const uint16_t*)wg,
                           (const uint16_t*)wu, s.d, s.f, h, (uint16_t*)act_save, tiles, count, seg, s.E);
        FINE_LAUNCH_CHECK();
    }
    if (gemm2) {
        hipLaunchKernelGGL(k_ffn_stream<1>, dim3(grid), dim3(256), lds, st, (const uint16_t*)h, (const uint16_t*)wd,
                           (const uint16_t*)nullptr, s.f, s.d, (uint16_t*)y_perm, (uint16_t*)nullptr, tiles, count, seg, s.E);
        FINE_LAUNCH_CHECK();
    }
    return FINE_OK;
}

}  // namespace fine
