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

// Small launches: 32 rows x 32 columns (GEMM 1: 32 gate columns and the matching 32 up columns) per block, the contraction
// split over its four waves, operands from memory straight into registers.  With fewer of the tiles above than CUs a
// launch is a chain of latencies on few CUs: a load, its 2048 cycles of MFMA, the next.  Here a quarter of the chain is
// left, four to eight times as many blocks share the work, and a wave asks for 64 k-values before it waits, for all of them: the second
// chunk's request is behind a branch, after which the compiler's waits for the first count down to none.  The four partial tiles are added in LDS, in the order of k.  That is another order than the one chain of the kernel
// above (its distance from 64-bit sums is half as large), and which one a row gets depends on the call's ranks: a rank's call
// and the call over all ranks differ in last bits where one takes this kernel and the other does not.  (The kernel above with
// its sums in the same four ranges takes 2 % longer, 4 % on short k: 4096 rows of 1024 x 2816 561 -> 573, 8192 of 128 x 256 30 -> 31.)
// Measured, both GEMMs of a rank's call, 64-row tiles against these: 128 rows of 128 x 256 18.0 : 13.0 us; 256 rows of 256 x
// 512 27.5 : 14.2; 512 rows on 2-3 experts of 1024 x 2816 (tiles64, below, 330) 133 : 116, 256 rows (210) 115 : 74, 32 rows
// 105 : 46; 768 rows of 768 x 768 (180) 51 : 46; but 900 rows of 768 x 1024 (239) 57 : 62, 1024 rows of 1024 x 2816 (630) 216 :
// 230, 4096 rows (2400) 665 : 826.  With a few rows per expert the 64-row tiles are mostly empty however many they are:
// 16 rows on each of 32 experts of 1024 x 2816 248 : 213, 8 rows 182 : 156; 32 rows 269 : 296.  Rows that are no multiple of
// 16 bytes need four times the loads: 576 rows of 700 x 777 (149) 57 : 54, 435 rows of 172 x 1515 (173) 56 : 43, but 819 rows of
// 700 x 777 (196) 57 : 76, 439 rows of 1082 x 1926 (189) 101 : 131, 696 rows of 338 x 907 (198) 47 : 59.
constexpr int kSM = 32, kSChunk = 32;

template <int EPI, int V>
__global__ __launch_bounds__(256, 2) void k_ffn_f32_split(const float* __restrict__ A, const float* __restrict__ B0,
                                                          const float* __restrict__ B1, int Kd, int N, float* __restrict__ C,
                                                          float* __restrict__ act, const TileEntry* __restrict__ tiles,
                                                          const int32_t* __restrict__ count, const int32_t* __restrict__ seg, int E) {
    constexpr int NP = EPI == 0 ? 2 : 1;
    __shared__ __attribute__((aligned(16))) float part[4 * NP * 16 * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 31, h = lane >> 5;
    RankTiles rank;
    if (seg != nullptr) rank.init(seg, E, kSM);
    const int ntn = (N + 31) / 32, ntm = seg != nullptr ? rank.count : *count, total = ntm * ntn;
    const int nc = (Kd + kSChunk - 1) / kSChunk, c0 = nc * wave / 4, c1 = nc * (wave + 1) / 4;
    for (int work = blockIdx.x; work < total; work += gridDim.x) {
        const int tm = work / ntn, n0 = (work - tm * ntn) * 32;
        const TileEntry te = seg != nullptr ? rank.get(tm, kSM) : tiles[tm];
        const float* Bp[2];
        Bp[0] = B0 + (size_t)te.expert * Kd * N;
        Bp[1] = EPI == 0 ? B1 + (size_t)te.expert * Kd * N : Bp[0];
        // rows past the tile's last and (by the offset) k-values past Kd lie beyond A's descriptor, k-rows past Kd beyond
        // B's: zeros on both sides; columns past N are clamped, their results never stored
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(A + (size_t)te.row0 * Kd), 0, (int)((uint32_t)te.rows * Kd * 4u), 0x00020000);
        const uint32_t b_off = ((uint32_t)4 * h * N + min(n0 + r, N - 1)) * 4u;
        struct Chunk {
            f32x4 a[4];
            float b[NP][16];
        };
        auto fetch = [&](Chunk& c, int at) {
            const int k0 = at * kSChunk;
            const unsigned long long left = (unsigned long long)(Kd - k0) * N * 4u;
            const int b_size = (int)(uint32_t)(left < 0xfffffff0ull ? left : 0xfffffff0ull);
            static_for<4>([&](auto j) {
                const int k = k0 + 8 * j.value + 4 * h;
                auto off = [&](int i) { return k + i < Kd ? ((uint32_t)r * Kd + k + i) * 4u : 0xf0000000u; };
                if constexpr (V == 4) {
                    c.a[j.value] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, off(0), 0, 0));
                } else {
                    static_for<4>([&](auto i) {
                        c.a[j.value][i.value] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ra, off(i.value), 0, 0));
                    });
                }
            });
            static_for<NP>([&](auto t) {
                const __amdgpu_buffer_rsrc_t rb =
                    __builtin_amdgcn_make_buffer_rsrc((void*)(Bp[t.value] + (size_t)k0 * N), 0, b_size, 0x00020000);
                static_for<16>([&](auto i) {
                    c.b[t.value][i.value] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                        rb, b_off, (8 * (i.value / 4) + i.value % 4) * N * 4, 0));
                });
            });
        };
        f32x16 acc[NP];
        static_for<NP>([&](auto t) { static_for<16>([&](auto q) { acc[t.value][q.value] = 0.f; }); });
        auto multiply = [&](const Chunk& c) {
            static_for<16>([&](auto i) {
                static_for<NP>([&](auto t) {
                    acc[t.value] = __builtin_amdgcn_mfma_f32_32x32x2f32(c.a[i.value / 4][i.value % 4], c.b[t.value][i.value], acc[t.value], 0, 0, 0);
                });
            });
        };
        Chunk x, y;
        if (c0 < c1) fetch(x, c0);
        for (int c = c0; c < c1; c += 2) {      // (wave-uniform)
            if (c + 1 < c1) fetch(y, c + 1);
            multiply(x);
            if (c + 2 < c1) fetch(x, c + 2);
            if (c + 1 < c1) multiply(y);
        }
        static_for<NP>([&](auto t) {
            static_for<16>([&](auto q) { part[((wave * NP + t.value) * 16 + q.value) * 64 + lane] = acc[t.value][q.value]; });
        });
        lds_barrier();
        // wave w adds up and stores the rows 8 w .. 8 w + 7 (registers 4 w .. 4 w + 3: lane = column)
        static_for<4>([&](auto q) {
            float v[NP];
            static_for<NP>([&](auto t) {
                const float* p = part + (t.value * 16 + 4 * wave + q.value) * 64 + lane;
                v[t.value] = ((p[0] + p[NP * 1024]) + p[2 * NP * 1024]) + p[3 * NP * 1024];
            });
            const int m = 8 * wave + 4 * h + q.value, n = n0 + r;
            if (m < te.rows && n < N) {
                const size_t row = (size_t)te.row0 + m;
                if constexpr (EPI == 0) {
                    if (act != nullptr) {
                        act[row * (2 * (size_t)N) + n] = v[0];
                        act[row * (2 * (size_t)N) + N + n] = v[1];
                    }
                    C[row * N + n] = silu_mul_f32(v[0], v[1]);
                } else {
                    C[row * N + n] = v[0];
                }
            }
        });
        lds_barrier();      // the next tile's parts
    }
}

// The same on 32 rows x 16 columns (v_mfma_f32_16x16x4_f32, 32 cycles): launches of so few 32 x 32 tiles that half of the CUs
// have none, where what is left of a launch is one trip to memory and a wave's chain of MFMAs, which this halves.  An MFMA's four
// k-values are k, k + 4, k + 8, k + 12 (lane group g has 4 g + i of sixteen), so that a lane's A values are 16 contiguous bytes.
// Bound by latency: a rank's call of 128 rows of 128 x 256 on 8 experts, both GEMMs, 32 x 32 : 32 x 16 tiles (72 expected of the
// former) 9.8 : 8.9 us; 64 rows of 133 x 257 (42) 13.5 : 11.0; 64 rows of 1024 x 1024 (128) 23.4 : 19.2; 256 rows of 256 x 512 (144) 13.8 :
// 12.9; but 1024 rows of 128 x 256 (240) 11.8 : 12.0, 512 rows of 300 x 301 (240) 19.3 : 23.2, 256 of 512 x 512 (384) 18.6 : 24.1.
template <int EPI, int V>
__global__ __launch_bounds__(256, 2) void k_ffn_f32_split16(const float* __restrict__ A, const float* __restrict__ B0,
                                                            const float* __restrict__ B1, int Kd, int N, float* __restrict__ C,
                                                            float* __restrict__ act, const TileEntry* __restrict__ tiles,
                                                            const int32_t* __restrict__ count, const int32_t* __restrict__ seg, int E) {
    constexpr int NP = EPI == 0 ? 2 : 1;
    __shared__ __attribute__((aligned(16))) float part[4 * NP * 8 * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 15, g = lane >> 4;
    RankTiles rank;
    if (seg != nullptr) rank.init(seg, E, kSM);
    const int ntn = (N + 15) / 16, ntm = seg != nullptr ? rank.count : *count, total = ntm * ntn;
    const int nc = (Kd + kSChunk - 1) / kSChunk, c0 = nc * wave / 4, c1 = nc * (wave + 1) / 4;
    for (int work = blockIdx.x; work < total; work += gridDim.x) {
        const int tm = work / ntn, n0 = (work - tm * ntn) * 16;
        const TileEntry te = seg != nullptr ? rank.get(tm, kSM) : tiles[tm];
        const float* Bp[2];
        Bp[0] = B0 + (size_t)te.expert * Kd * N;
        Bp[1] = EPI == 0 ? B1 + (size_t)te.expert * Kd * N : Bp[0];
        // (ranges as in the kernel above)
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(A + (size_t)te.row0 * Kd), 0, (int)((uint32_t)te.rows * Kd * 4u), 0x00020000);
        const uint32_t b_off = ((uint32_t)4 * g * N + min(n0 + r, N - 1)) * 4u;
        struct Chunk {
            f32x4 a[2][2];      // [16 k][16 rows]
            float b[NP][8];
        };
        auto fetch = [&](Chunk& c, int at) {
            const int k0 = at * kSChunk;
            const unsigned long long left = (unsigned long long)(Kd - k0) * N * 4u;
            const int b_size = (int)(uint32_t)(left < 0xfffffff0ull ? left : 0xfffffff0ull);
            static_for<2>([&](auto j) {
                static_for<2>([&](auto f) {
                    const int k = k0 + 16 * j.value + 4 * g, row = 16 * f.value + r;
                    auto off = [&](int i) { return k + i < Kd ? ((uint32_t)row * Kd + k + i) * 4u : 0xf0000000u; };
                    if constexpr (V == 4) {
                        c.a[j.value][f.value] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, off(0), 0, 0));
                    } else {
                        static_for<4>([&](auto i) {
                            c.a[j.value][f.value][i.value] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ra, off(i.value), 0, 0));
                        });
                    }
                });
            });
            static_for<NP>([&](auto t) {
                const __amdgpu_buffer_rsrc_t rb =
                    __builtin_amdgcn_make_buffer_rsrc((void*)(Bp[t.value] + (size_t)k0 * N), 0, b_size, 0x00020000);
                static_for<8>([&](auto i) {
                    c.b[t.value][i.value] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                        rb, b_off, (16 * (i.value / 4) + i.value % 4) * N * 4, 0));
                });
            });
        };
        f32x4 acc[NP][2];
        static_for<NP>([&](auto t) { static_for<2>([&](auto f) { acc[t.value][f.value] = f32x4{0.f, 0.f, 0.f, 0.f}; }); });
        auto multiply = [&](const Chunk& c) {
            static_for<8>([&](auto i) {
                static_for<NP>([&](auto t) {
                    static_for<2>([&](auto f) {
                        acc[t.value][f.value] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.a[i.value / 4][f.value][i.value % 4], c.b[t.value][i.value],
                                                                                     acc[t.value][f.value], 0, 0, 0);
                    });
                });
            });
        };
        Chunk x, y;
        if (c0 < c1) fetch(x, c0);
        for (int c = c0; c < c1; c += 2) {      // (wave-uniform)
            if (c + 1 < c1) fetch(y, c + 1);
            multiply(x);
            if (c + 2 < c1) fetch(x, c + 2);
            if (c + 1 < c1) multiply(y);
        }
        static_for<NP>([&](auto t) {
            static_for<8>([&](auto q) { part[((wave * NP + t.value) * 8 + q.value) * 64 + lane] = acc[t.value][q.value / 4][q.value % 4]; });
        });
        lds_barrier();
        // wave w adds up and stores registers 2 w and 2 w + 1: rows 16 (w / 2) + 4 g + 2 (w & 1) + 0, 1; lane = column
        static_for<2>([&](auto q) {
            float v[NP];
            static_for<NP>([&](auto t) {
                const float* p = part + (t.value * 8 + 2 * wave + q.value) * 64 + lane;
                v[t.value] = ((p[0] + p[NP * 512]) + p[2 * NP * 512]) + p[3 * NP * 512];
            });
            const int m = 16 * (wave >> 1) + 4 * g + 2 * (wave & 1) + q.value, n = n0 + r;
            if (m < te.rows && n < N) {
                const size_t row = (size_t)te.row0 + m;
                if constexpr (EPI == 0) {
                    if (act != nullptr) {
                        act[row * (2 * (size_t)N) + n] = v[0];
                        act[row * (2 * (size_t)N) + N + n] = v[1];
                    }
                    C[row * N + n] = silu_mul_f32(v[0], v[1]);
                } else {
                    C[row * N + n] = v[0];
                }
            }
        });
        lds_barrier();      // the next tile's parts
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
    const int n_ranks = rank_hi - rank_lo;
    const bool wide = s.d % 4 == 0 && s.f % 4 == 0;      // 16-byte pieces of a row are aligned
    // expected tiles of 64 rows (see pick_tile in ffn_mfma.hip)
    const double rows = (double)s.T * s.K * n_ranks / s.G, runs = std::min((double)s.E * n_ranks / s.G + 1.0, (double)s.E);
    const double tiles64 = (rows / kBM + runs) * (cdiv(s.f, 64) + cdiv(s.d, 64)) / 2;
    const bool split = tiles64 < (wide ? 220.0 : 175.0) || rows <= 16.0 * runs;
    const double tiles32 = (rows / kSM + runs) * (cdiv(s.f, 32) + cdiv(s.d, 32)) / 2;
    const bool narrow = split && tiles32 < 160.0;
    const int bm = split ? kSM : kBM, bn = narrow ? 16 : split ? 32 : 64;
    const int32_t* seg = nullptr;
    if (n_ranks == 1 && s.E <= kRankMapExperts) seg = seg_off + (size_t)rank_lo * (s.E + 1);
    else FINE_TRY(launch_tile_map(s, seg_off, rank_lo, rank_hi, bm, false, tiles, count, L.max_tiles, st));
    // three blocks per CU, four of the split kernel (whose registers let two to four in); no more than there can be tiles
    const size_t rows_tiles = (size_t)s.T * s.K / bm + (size_t)s.E * n_ranks;
    auto grid = [&](int n) { return (unsigned)std::min<size_t>(split ? 1024 : 768, align_up(rows_tiles * cdiv(n, bn), 8)); };
    auto run = [&](auto k1, auto k2) {
        hipLaunchKernelGGL(k1, dim3(grid(s.f)), dim3(256), 0, st, (const float*)x_perm, (const float*)wg, (const float*)wu, s.d, s.f,
                           h, (float*)act_save, tiles, count, seg, s.E);
        FINE_LAUNCH_CHECK();
        hipLaunchKernelGGL(k2, dim3(grid(s.d)), dim3(256), 0, st, (const float*)h, (const float*)wd, (const float*)nullptr, s.f, s.d,
                           (float*)y_perm, (float*)nullptr, tiles, count, seg, s.E);
        FINE_LAUNCH_CHECK();
        return (int)FINE_OK;
    };
    if (narrow) return wide ? run(k_ffn_f32_split16<0, 4>, k_ffn_f32_split16<1, 4>) : run(k_ffn_f32_split16<0, 1>, k_ffn_f32_split16<1, 1>);
    if (split) return wide ? run(k_ffn_f32_split<0, 4>, k_ffn_f32_split<1, 4>) : run(k_ffn_f32_split<0, 1>, k_ffn_f32_split<1, 1>);
    return wide ? run(k_ffn_f32<0, 4>, k_ffn_f32<1, 4>) : run(k_ffn_f32<0, 1>, k_ffn_f32<1, 1>);
}

}  // namespace fine
