// Grouped SwiGLU expert FFN of fp32 layers on the fp32 matrix cores (v_mfma_f32_32x32x2_f32:
// fp32 products and sums, the rate of the chip's fp32 peak, 157 TFLOP/s).
//
// GEMM 1: a block of 4 waves computes 64 rows x 128 columns (64 gate columns and the matching 64 up columns, so
// that SwiGLU is applied in registers), each wave 32 x 64 = two 32 x 32 accumulator tiles.  GEMM 2: 64 x 64, one
// accumulator tile per wave: its output is narrower (d columns instead of 2 f), so it has fewer tiles to even out
// over the CUs (2048 tokens, d 1024, f 2816, 16 experts: 28 us of 940 less than with 64 x 128).
// An fp32 MFMA takes 64 cycles for 4 K FLOP, sixteen times as long per operand byte as a bf16 one,
// so the kernel is bound by the matrix cores and neither LDS nor memory needs care; what counts is
// that a CU's four SIMDs always have a wave with an MFMA ready.  Hence the small tile: at most 48 KB of LDS
// (two buffers of 32 k-values) and three blocks per CU, whose waves fill one another's barriers,
// prologues and epilogues; and 64-row tiles waste little on short segments.  (Five blocks of the smaller
// tile per CU are 7 % slower than three.)  At the size above GEMM 1 takes 416 us and GEMM 2 235 us (114 and
// 100 TFLOP/s of 157; FMA kernels: 1378 and 805 us); an eighth of it is rows past the ends of segments.
//
// Both operands reach LDS by DMA, 16 bytes per lane when d and f are multiples of 4, else 4 bytes per
// lane (rows of any width: an MFMA step leaves enough issue slots for four times the instructions).
// LDS: A [64 rows][32 k], 16-byte chunks swizzled as in lds_off(); B two panels of [32 k][64 columns] with the
// column halves swapped where bit 2 of k is set.  An MFMA's two k-values are k and k + 4: lane half h
// reads k = 8 j + 4 h + 0 .. 3 of its A row in one 16-byte read and uses one of the four per MFMA; both
// read patterns touch every bank once.
#include "gemm_w8.h"

namespace fine {

namespace {

using namespace mfma;

constexpr int kBM = 64, kBK = 32;
constexpr int kABytes = kBM * kBK * 4, kPanelBytes = kBK * 64 * 4;

__device__ inline float silu_mul_f32(float a, float b) { return a / (1.f + __expf(-a)) * b; }

// one DMA instruction: V floats per lane
template <int V>
__device__ inline void dma_to_lds(const __amdgpu_buffer_rsrc_t& rs, char* lds, uint32_t off, uint32_t soff) {
    if constexpr (V == 4) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, FINE_LDS_PTR(lds), 16, off, soff, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, FINE_LDS_PTR(lds), 4, off, soff, 0, 0);
}

// EPI 0: A = x_perm [P,Kd], B0 / B1 = Wg / Wu [E,Kd,N], C = H [P,N]; act [P,2N] optional
// EPI 1: A = H [P,Kd], B0 = Wd [E,Kd,N], C = y_perm [P,N]
// V: floats per lane and DMA instruction
template <int EPI, int V>
__global__ __launch_bounds__(256, 3) void k_ffn_f32(const float* __restrict__ A, const float* __restrict__ B0,
                                                 const float* __restrict__ B1, int Kd, int N, float* __restrict__ C,
                                                 float* __restrict__ act, const TileEntry* __restrict__ tiles,
                                                 const int32_t* __restrict__ count, const int32_t* __restrict__ seg, int E) {
    constexpr int NP = EPI == 0 ? 2 : 1;                  // 64-column panels of B: gate and up / down
    constexpr int BNC = 64;                               // output columns per block
    constexpr int kBuf = kABytes + NP * kPanelBytes;      // one buffer: A and the panels of B
    __shared__ __attribute__((aligned(16))) char smem[2 * kBuf];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, h = lane >> 5;
    RankTiles rank;      // seg != NULL: one rank, whose work list every wave makes for itself
    if (seg != nullptr) rank.init(seg, E, kBM);
    const int ntn = (N + BNC - 1) / BNC, ntm = seg != nullptr ? rank.count : *count, total = ntm * ntn;
    const int nk = (Kd + kBK - 1) / kBK;

    // DMA side.  A: an instruction covers AROWS rows; lane -> (row, k of its first element) with the chunk
    // swizzle applied on the global side.  B: an instruction covers BROWS k-rows of one panel.
    constexpr int AROWS = 64 * V / kBK, AINST = kBM / AROWS / 4;      // instructions per wave
    constexpr int BROWS = 64 * V / 64, BINST = NP * kBK / BROWS / 4;
    const int a_row = lane / (kBK / V), a_w = (lane % (kBK / V)) * V;
    const int b_k = lane / (64 / V), b_w = (lane % (64 / V)) * V;

    // Every XCD (blocks are dealt to them in turn) gets an eighth of the tiles, consecutive ones, and its blocks take
    // them in turn: the tiles of a last incomplete round then lie on all XCDs, on blocks of different CUs.
    const int xcd = blockIdx.x & 7, end = (int)((long long)total * (xcd + 1) / 8);
    for (int work = (int)((long long)total * xcd / 8) + (blockIdx.x >> 3); work < end; work += gridDim.x >> 3) {
        int tm, tn;
        tile_of_work(work, ntm, ntn, tm, tn);
        const TileEntry te = seg != nullptr ? rank.get(tm, kBM) : tiles[tm];
        const int n0 = tn * BNC;
        const float* Bp[2];
        Bp[0] = B0 + (size_t)te.expert * Kd * N;
        Bp[1] = EPI == 0 ? B1 + (size_t)te.expert * Kd * N : Bp[0];
        const float* Ap = A + (size_t)te.row0 * Kd;

        // byte offsets of this lane's pieces inside the first k-step; later steps move the scalar offset (A) or the
        // descriptor's base (B).  Rows past the tile's last lie beyond A's descriptor and arrive as zeros, k-rows past
        // the matrix's last beyond B's; columns past N are clamped, their results never stored.
        uint32_t a_off[AINST], b_off[BINST];
        int a_k[AINST];
#pragma unroll
        for (int j = 0; j < AINST; ++j) {
            const int row = (wave * AINST + j) * AROWS + a_row;
            a_k[j] = ((((a_w >> 2) ^ (row >> 1)) & 7) << 2) + (a_w & 3);
            a_off[j] = ((uint32_t)row * Kd + a_k[j]) * 4u;
        }
#pragma unroll
        for (int j = 0; j < BINST; ++j) {
            const int inst = wave * BINST + j, p = inst / (kBK / BROWS), k = (inst % (kBK / BROWS)) * BROWS + b_k;
            const int c = b_w ^ (((k >> 2) & 1) << 5);
            b_off[j] = ((uint32_t)k * N + min(n0 + c, N - V)) * 4u;
        }
        const __amdgpu_buffer_rsrc_t ra =
            __builtin_amdgcn_make_buffer_rsrc((void*)Ap, 0, (int)((uint32_t)te.rows * Kd * 4u), 0x00020000);
        auto issue = [&](int kt, int buf) {
            char* base = smem + buf * kBuf;
            const int k0 = kt * kBK;
            const bool tail = k0 + kBK > Kd;      // (block-uniform) k-values past Kd of A: moved out of range
#pragma unroll
            for (int j = 0; j < AINST; ++j)
                dma_to_lds<V>(ra, base + (wave * AINST + j) * AROWS * kBK * 4,
                              tail && k0 + a_k[j] >= Kd ? 0xf0000000u : a_off[j], (uint32_t)k0 * 4u);
            const unsigned long long left = (unsigned long long)(Kd - k0) * N * 4u;
            const int b_size = (int)(uint32_t)(left < 0xfffffff0ull ? left : 0xfffffff0ull);
#pragma unroll
            for (int j = 0; j < BINST; ++j) {
                const int inst = wave * BINST + j, p = inst / (kBK / BROWS), kr0 = (inst % (kBK / BROWS)) * BROWS;
                const __amdgpu_buffer_rsrc_t rb =
                    __builtin_amdgcn_make_buffer_rsrc((void*)(Bp[p] + (size_t)k0 * N), 0, b_size, 0x00020000);
                dma_to_lds<V>(rb, base + kABytes + p * kPanelBytes + kr0 * 256, b_off[j], 0);
            }
        };

        f32x16 acc[NP];
#pragma unroll
        for (int t = 0; t < NP; ++t)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[t][q] = 0.f;
        issue(0, 0);
        for (int kt = 0; kt < nk; ++kt) {
            // this step's operands have landed, and everybody is done with the buffer that is filled next
            wait_vm_lgkm<0>();
            block_barrier();
            if (kt + 1 < nk) issue(kt + 1, (kt + 1) & 1);
            const char* sA = smem + (kt & 1) * kBuf;
            const char* sB = sA + kABytes;
            if (wm * 32 < te.rows)      // (wave-uniform) a wave without valid rows leaves the matrix core to the others
#pragma unroll
            for (int j = 0; j < kBK / 8; ++j) {
                const f32x4 a = *reinterpret_cast<const f32x4*>(sA + lds_off(wm * 32 + r, 2 * j + h));
                float b[NP][4];
#pragma unroll
                for (int t = 0; t < NP; ++t)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        b[t][q] = *reinterpret_cast<const float*>(sB + t * kPanelBytes + (8 * j + 4 * h + q) * 256 + ((32 * wn + r) ^ (h << 5)) * 4);
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int t = 0; t < NP; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[t][q], acc[t], 0, 0, 0);
            }
        }
        // the accumulators hold the output as it lies (lane = column, register = row): a store instruction writes
        // 128 contiguous bytes of each of two rows
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int m = wm * 32 + 8 * (q >> 2) + 4 * h + (q & 3);
            if (m >= te.rows) continue;
            const size_t row = (size_t)te.row0 + m;
            const int n = n0 + 32 * wn + r;
            if (n >= N) continue;
            if constexpr (EPI == 0) {
                if (act != nullptr) {
                    act[row * (2 * (size_t)N) + n] = acc[0][q];
                    act[row * (2 * (size_t)N) + N + n] = acc[1][q];
                }
                C[row * N + n] = silu_mul_f32(acc[0][q], acc[1][q]);
            } else {
                C[row * N + n] = acc[0][q];
            }
        }
        block_barrier();      // the next tile's first DMA overwrites a buffer that slower waves may still read
    }
}

}  // namespace

int launch_ffn_f32(const fine_shape& s, int rank_lo, int rank_hi, const void* x_perm, const void* wg, const void* wu,
                   const void* wd, const int32_t* seg_off, void* y_perm, void* act_save, char* ws, hipStream_t st) {
    const FfnWs L = ffn_ws_layout(s);
    auto* tiles = reinterpret_cast<TileEntry*>(ws + L.tiles);
    auto* count = reinterpret_cast<int32_t*>(ws + L.count);
    auto* h = reinterpret_cast<float*>(ws + L.h);
    if ((s.flags & FINE_FLAG_ACT_SAVE_H) && act_save != nullptr)      // H behind the saved pre-activations
        h = static_cast<float*>(act_save) + (size_t)s.T * s.K * 2 * s.f;
    const int32_t* seg = nullptr;
    if (rank_hi - rank_lo == 1 && s.E <= kRankMapExperts) seg = seg_off + (size_t)rank_lo * (s.E + 1);
    else FINE_TRY(launch_tile_map(s, seg_off, rank_lo, rank_hi, kBM, tiles, count, L.max_tiles, st));
    // three blocks per CU; no more blocks than there can be tiles
    const size_t rows_tiles = (size_t)s.T * s.K / kBM + (size_t)s.E * (rank_hi - rank_lo);
    auto grid = [&](int n) { return (unsigned)std::min<size_t>(768, align_up(rows_tiles * cdiv(n, 64), 8)); };
#define FINE_F32(V)                                                                                              \
    do {                                                                                                         \
        hipLaunchKernelGGL((k_ffn_f32<0, V>), dim3(grid(s.f)), dim3(256), 0, st, (const float*)x_perm, (const float*)wg, \
                           (const float*)wu, s.d, s.f, h, (float*)act_save, tiles, count, seg, s.E);                       \
        FINE_LAUNCH_CHECK();                                                                                     \
        hipLaunchKernelGGL((k_ffn_f32<1, V>), dim3(grid(s.d)), dim3(256), 0, st, (const float*)h, (const float*)wd, \
                           (const float*)nullptr, s.f, s.d, (float*)y_perm, (float*)nullptr, tiles, count, seg, s.E);      \
        FINE_LAUNCH_CHECK();                                                                                     \
    } while (0)
    if (s.d % 4 == 0 && s.f % 4 == 0) FINE_F32(4);
    else FINE_F32(1);
#undef FINE_F32
    return FINE_OK;
}

}  // namespace fine
