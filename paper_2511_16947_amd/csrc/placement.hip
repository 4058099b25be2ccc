// Expert placement from known expert loads (Section 5.3), scored by the maximum density
// over induced subgraphs (Section 5.1, Eq. 3).
//
//   k_replica_counts   step 1: every expert one replica, each further replica to the expert with
//                      the largest load per replica (exact, ties to the lower expert index).  One
//                      wavefront; the argmax of a round is a maximum of 64-bit keys over the lanes.
//   k_score            step 2, four candidates per block: one wave draws their placements (or the block reads
//                      given ones), then each wave evaluates Eq. 3 over all 2^G - 1 rank subsets of one
//                      candidate (few candidates: the block's waves share one candidate's subsets).
//   k_score_flow       the same for more than 16 ranks, where the subsets cannot be enumerated: one
//                      wavefront per candidate finds the same m with exact integer flows.
//   k_pick             the candidate with the smallest m (ties: lowest index); draws it again and
//                      writes it out as a mask [E][G].
//
// Eq. 3 over all subsets.  w(S) = sum of load_e over experts whose replica set lies inside S is
// the subset-sum (zeta) transform of f[mask] = sum of load_e with replica set == mask: for
// each rank bit b in turn, every S containing b adds the value of S without b.  One wavefront holds
// the table of the low 11 ranks in registers (32 entries per lane); the remaining high ranks are
// enumerated: for a pattern h of high ranks, the experts whose high part lies inside h are scattered
// by their low part, transformed over the low bits, and every entry L gives the candidate
// w / (popcount(L) + popcount(h)).  (With fewer than 11 ranks the missing ones hold no replicas: a
// set with them has the sum of the set without them and more members, so it never wins.)  Fractions
// are compared exactly (64-bit cross-multiplication); the result is reduced by the gcd.
//
// Drawing a candidate: experts in order of decreasing replica count (ties: lower index); an
// expert's c replicas go to the c ranks with the most free slots, ties by the larger random
// key, then the lower rank.  A lane is a rank: its position in that order is the number of ranks with a
// larger composite key.  Up to 16 ranks a wave draws four candidates at once, one per row of 16 lanes, and
// the comparisons are 15 rotations of the row (DPP); beyond, one cross-lane read per rank.  The keys come
// from a counter-based generator: two rounds of the MurmurHash3 32-bit finaliser over
// (seed, candidate) and (expert, rank).
#include <type_traits>

#include "flow_wave.h"

namespace fine {

namespace {

typedef unsigned long long u64;
typedef long long i64;

constexpr int kScoreThreads = 256;
constexpr int kLow = 11, kTable = 1 << kLow;           // ranks and entries of a wave's table
constexpr int kCandPerBlock = kScoreThreads / 64;      // one per wave
constexpr int kMaxE = 1024;
constexpr int kMaxEnumG = 16;        // Eq. 3 by enumeration of 2^G subsets up to here, by flows beyond

__device__ inline uint32_t mix32(uint32_t h) {
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}
__device__ inline uint32_t rank_key(uint32_t seed, uint32_t cand, uint32_t e, uint32_t g) {
    const uint32_t h = mix32(seed + 0x9E3779B9u * (cand + 1u));
    return mix32(h ^ ((e * 64u + g + 1u) * 0x9E3779B1u));
}

// a.num / a.den > b.num / b.den, exactly (0 <= num < 2^31: a sum of loads; 0 < den <= 64)
struct Frac {
    int num;
    int den;
};
__device__ inline bool frac_gt(Frac a, Frac b) { return (i64)a.num * b.den > (i64)b.num * a.den; }

// ---------------------------------------------------------------------------
// step 1
// ---------------------------------------------------------------------------
// largest of the lanes' keys, in every lane (six DPP steps: lane layout in flow_wave.h)
__device__ inline u64 wave_max_u64(u64 v) {
    auto step = [&](auto from) {
        const u64 o = ((u64)(uint32_t)from((int)(v >> 32)) << 32) | (uint32_t)from((int)v);
        if (o > v) v = o;
    };
    step([](int x) { return flow::dpp_from<0x111, 0xf>(0, x); });
    step([](int x) { return flow::dpp_from<0x112, 0xf>(0, x); });
    step([](int x) { return flow::dpp_from<0x114, 0xf>(0, x); });
    step([](int x) { return flow::dpp_from<0x118, 0xf>(0, x); });
    step([](int x) { return flow::dpp_from<0x142, 0xa>(0, x); });
    step([](int x) { return flow::dpp_from<0x143, 0xc>(0, x); });
    return flow::readlane_u64(v, 63);
}

// Load per replica as an integer that orders exactly like the fraction: two different l / c with c <= 64 are at
// least 1 / 64^2 apart, so floor(2^13 l / c) differs the same way, and equal fractions give equal values.  Below it
// the expert's index, lower = larger.  A round costs one wave maximum and one division (16 rounds on 64
// experts: 18 -> 7 us against fractions compared by cross-multiplication in a butterfly of shuffles).  The division is a
// double's: numerator and quotient have 44 bits at most, so the quotient rounds by at most 2^-9, and one that is no whole
// number is at least 1 / 64 below the next (a division of 64-bit integers is a hundred instructions: 7.7 -> 7.2 us).
__device__ inline u64 count_key(int load, int c, int e) {
    const u64 per = (u64)((double)((u64)(uint32_t)load << 13) / (double)c);
    return per << 10 | (u64)(kMaxE - 1 - e) | 1ull << 60;
}

__global__ __launch_bounds__(64) void k_replica_counts(const int32_t* __restrict__ load, int E, int G, int slots,
                                                       int32_t* __restrict__ counts) {
    __shared__ int s_load[kMaxE], s_cnt[kMaxE];
    __shared__ u64 s_key[kMaxE];             // 0: on all G ranks
    const int lane = threadIdx.x;
    u64 mine = 0ull;                         // best of the experts lane, lane + 64, ...
    for (int e = lane; e < E; e += 64) {
        s_load[e] = max(load[e], 0);
        s_cnt[e] = 1;
        s_key[e] = G > 1 ? count_key(s_load[e], 1, e) : 0ull;
        mine = s_key[e] > mine ? s_key[e] : mine;
    }
    const long long rounds = (long long)G * slots - E;
    for (long long r = 0; r < rounds; ++r) {
        const u64 best = wave_max_u64(mine);
        if (best == 0ull) break;             // every expert is on all G ranks
        const int e = kMaxE - 1 - (int)(best & (kMaxE - 1));
        if (lane == (e & 63)) {              // (only this lane touches its experts' entries)
            const int c = ++s_cnt[e];
            s_key[e] = c < G ? count_key(s_load[e], c, e) : 0ull;
            mine = 0ull;
            for (int i = lane; i < E; i += 64) mine = s_key[i] > mine ? s_key[i] : mine;
        }
    }
    for (int e = lane; e < E; e += 64) counts[e] = s_cnt[e];
}

// ---------------------------------------------------------------------------
// drawing a candidate (one wave; lanes >= G idle along)
// ---------------------------------------------------------------------------
// s_order [E]: experts in drawing order, expert | replica count << 16; s_mask [E] out: replica set of each
// expert as a rank mask
__device__ inline void draw_candidate(const int* s_order, u64* s_mask, int E, int G, int slots,
                                      uint32_t seed, uint32_t cand) {
    const int g = threadIdx.x & 63;       // lane = rank
    int free_slots = slots;
    for (int i = 0; i < E; ++i) {
        const int e = s_order[i] & 0xffff, c = s_order[i] >> 16;
        // larger is better: free slots, then key, then lower rank; distinct over the ranks
        const u64 comp = g < G ? ((u64)(uint32_t)(free_slots + (1 << 20)) << 40) |
                                     ((u64)rank_key(seed, cand, (uint32_t)e, (uint32_t)g) << 8) | (u64)(255 - g)
                               : 0ull;
        int ahead = 0;
        // lane j's value through a scalar register; lanes from G on hold 0, which is ahead of nobody
#pragma unroll
        for (int j = 0; j < 64; ++j) {
            const u64 other = ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(comp >> 32), j) << 32) |
                              (uint32_t)__builtin_amdgcn_readlane((int)comp, j);
            ahead += other > comp;
        }
        const bool chosen = g < G && ahead < c;
        free_slots -= chosen;
        const u64 m = __ballot(chosen);
        if (g == 0) s_mask[e] = m;
    }
}

// Up to 16 ranks: four candidates at once, row r of 16 lanes draws candidate cand0 + r into s_mask[r * E ...].
// A chain of E dependent steps, so a step is kept short: ranks are compared by 32 bits, 10 bits of slots not yet
// used (a rank takes at most one replica per expert, so fewer than 1024 are used before a step) and the upper 22 of the
// key.  Ranks that are equal in these are all chosen or all left, unless the last place falls between them: then a
// row has chosen too many, and the step is done again with all bits.  An expert with one replica, as most have, goes to
// its row's largest value: four rotations instead of fifteen.  (4096 candidates of 64 experts, 16 of them with several
// replicas: 111 -> 98 us; k_pick, one draw and the argmin of 4096 scores, 23 -> 20.)
template <int R, typename F>
__device__ inline void rotations(F& f) {
    if constexpr (R < 16) {
        f(std::integral_constant<int, R>{});
        rotations<R + 1>(f);
    }
}
//
// s_key, unless NULL: the ranks' keys in drawing order, [E][stride] (stride 64: a lane's own; 16: one candidate for every
// row), made by all waves of the block beforehand (draw_keys): two multiplications and a dozen instructions less per step.
__device__ inline uint32_t candidate_hash(uint32_t seed, uint32_t cand) { return mix32(seed + 0x9E3779B9u * (cand + 1u)); }
__device__ inline uint32_t key_of(uint32_t h, int e, int g) { return mix32(h ^ (((uint32_t)e * 64u + (uint32_t)g + 1u) * 0x9E3779B1u)); }

__device__ inline void draw_keys(const int* s_order, uint32_t* s_key, int stride, int E, uint32_t seed, uint32_t cand0) {
    for (int i = threadIdx.x; i < E * stride; i += blockDim.x) {
        const int l = i & (stride - 1);
        s_key[i] = key_of(candidate_hash(seed, cand0 + (uint32_t)(l >> 4)), s_order[i / stride] & 0xffff, l & 15);
    }
    __syncthreads();
}

__device__ inline void draw_rows(const int* s_order, const uint32_t* s_key, int stride, uint32_t* s_mask, int E, int G, uint32_t seed,
                                 uint32_t cand0) {
    const int lane = threadIdx.x & 63, g = lane & 15, row = lane >> 4;
    const uint32_t h = candidate_hash(seed, stride == 16 ? cand0 : cand0 + (uint32_t)row);
    uint32_t unused = 1023u;
    auto key_at = [&](int i, int e) { return s_key != nullptr ? s_key[i * stride + (lane & (stride - 1))] : key_of(h, e, g); };
    int cur = s_order[0], next = s_order[min(1, E - 1)];
    uint32_t next_key = key_at(0, cur & 0xffff);
    uint32_t* const mine = s_mask + row * E;
    // with all bits: slots, key, then lower rank, distinct over the ranks
    auto choose_exactly = [&](uint32_t key, int c) {
        const u64 all = g < G ? (u64)unused << 40 | (u64)key << 8 | (u64)(255 - g) : 0ull;
        int ahead = 0;
        auto count_all = [&](auto r) {
            const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(all >> 32), 0x120 + r.value, 0xf, 0xf, false);
            const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)all, 0x120 + r.value, 0xf, 0xf, false);
            ahead += ((u64)hi << 32 | lo) > all;
        };
        rotations<1>(count_all);
        return g < G && ahead < c;
    };
    int i = 0;
    auto step = [&](int& e, int& c, uint32_t& key) {      // on to expert i, and the next one's loads on their way
        e = __builtin_amdgcn_readfirstlane(cur & 0xffff);
        c = __builtin_amdgcn_readfirstlane(cur >> 16);
        key = next_key;
        cur = next;
        next_key = key_at(min(i + 1, E - 1), cur & 0xffff);
        next = s_order[min(i + 2, E - 1)];
    };
    int e, c;
    uint32_t key;
    for (; i < E; ++i) {                                  // several replicas: counts never grow along the order
        if (__builtin_amdgcn_readfirstlane(cur >> 16) <= 1) break;
        step(e, c, key);
        // larger is better; lanes beyond the ranks hold 0, which is ahead of nobody
        const uint32_t comp = g < G ? unused << 22 | key >> 10 : 0u;
        int ahead = 0;
        auto count = [&](auto r) {
            ahead += (uint32_t)__builtin_amdgcn_mov_dpp((int)comp, 0x120 + r.value, 0xf, 0xf, false) > comp;      // row_ror
        };
        rotations<1>(count);
        bool chosen = g < G && ahead < c;
        u64 m = __ballot(chosen);
        if (__ballot(__popc((uint32_t)(m >> (16 * row)) & 0xffffu) != min(c, G)) != 0ull) {
            chosen = choose_exactly(key, c);
            m = __ballot(chosen);
        }
        unused -= chosen;
        if (g == 0) mine[e] = (uint32_t)(m >> (16 * row)) & 0xffffu;
    }
    for (; i < E; ++i) {
        step(e, c, key);
        const uint32_t comp = g < G ? unused << 22 | key >> 10 : 0u;
        uint32_t top = comp;
        auto larger = [&](auto r) { top = max(top, (uint32_t)__builtin_amdgcn_mov_dpp((int)top, 0x120 + r.value, 0xf, 0xf, false)); };
        larger(std::integral_constant<int, 8>{});
        larger(std::integral_constant<int, 4>{});
        larger(std::integral_constant<int, 2>{});
        larger(std::integral_constant<int, 1>{});
        bool chosen = comp == top;                        // (never 0: at most E < 1024 slots are used up)
        if (__popcll(__ballot(chosen)) != 4) chosen = choose_exactly(key, 1);
        if (c < 1) chosen = false;
        if (c < 1 && g == 0) mine[e] = 0u;
        if (chosen) mine[e] = 1u << g;
        unused -= chosen;
    }
}

// position of every expert in the drawing order: decreasing count, then increasing index
__device__ inline void drawing_order(const int32_t* __restrict__ counts, int* s_cnt, int* s_order, int E) {
    for (int e = threadIdx.x; e < E; e += blockDim.x) s_cnt[e] = counts[e];
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        const int c = s_cnt[e];
        int pos = 0;
        for (int o = 0; o < E; ++o) {
            const int oc = s_cnt[o];
            pos += (oc > c) || (oc == c && o < e);
        }
        s_order[pos] = e | min(max(c, 0), 64) << 16;      // (at most 64 ranks)
    }
    __syncthreads();
}

// Where entry `idx` lies: bits 6..9 are folded into bits 2..5, so that the entries that experts add to fall into
// different banks (most replica sets have few ranks, and the low bits alone would name few banks).
__device__ inline int table_slot(int idx) { return idx ^ (((idx >> 6) & 15) << 2); }

__device__ inline void clear_table(int* s_f) {
#pragma unroll
    for (int q = 0; q < 8; ++q) *reinterpret_cast<int4*>(s_f + q * 256 + (threadIdx.x & 63) * 4) = make_int4(0, 0, 0, 0);
}

// What an expert's additions need, from its replica set m (a lane has the experts e = lane modulo 64): bits 0..10 the
// entry of its first addition; 11..15 the high ranks; bit 16 + i: whether there is an addition i (0 .. 3), to the entry with
// bits 2 and 3 XORed with i.  The two low bits t of the entry number >> 2 run through all values, starting with the
// lane's own (experts with the same few replicas would otherwise all add to one entry at a time), and those that
// contain the expert's part in these bits count.  Experts without load add nothing.
__device__ inline uint32_t additions(uint32_t m, int load, int e) {
    constexpr uint32_t kSuper = 3u;
    const uint32_t first = (uint32_t)e & kSuper, sub = (m >> 2) & kSuper;
    uint32_t out = (uint32_t)table_slot((int)((m & (uint32_t)(kTable - 1) & ~(kSuper << 2)) | first << 2)) | (m >> kLow) << kLow;
    for (uint32_t i = 0; i <= kSuper; ++i)
        if (load > 0 && ((first ^ i) & sub) == sub) out |= 1u << (16 + i);
    return out;
}

// Eq. 3 of one candidate by one wavefront (see the top of the file); lane-local maxima over the patterns that are
// number `part` modulo `parts` of their size.  s_f [kTable]: the wave's own.
//
// Index bits of the table: register bits = bits 0, 1, 8, 9, 10; lane bits 0..5 = bits 2..7.  Register bits are added
// along in registers; lane bits 5 and 4 change places with a register bit (permlane32_swap, permlane16_swap) and
// are added along there; lane bits 2 and 3 by row shifts that write the lanes with the bit set; lane bits 0 and 1
// when the experts are scattered (an expert goes to all supersets of its part in these bits; doing bits 2 and 3 the
// same way, 16 additions instead of 4 and 64 row shifts, measured the same).  No barriers and about 20 LDS accesses
// per 2048 entries: 4096 candidates on 16 ranks and 64 experts take 70 us without drawing them (the table of 13
// ranks in the LDS of a block, three rounds with barriers: 226 us with drawing), bound by the ALUs.  Patterns of
// one size together: their maxima per subset size are kept in six registers and compared as fractions once per size.
// s_f must be all zero and is left so.
__device__ inline Frac max_density(int* s_f, const uint32_t* s_at, const int* s_load, int E, int G, int part, int parts) {
    const int lane = threadIdx.x & 63;
    const int high_bits = max(G - kLow, 0);
    Frac best{0, 1};
    for (int ph = 0; ph <= high_bits; ++ph) {
        int mx[6] = {0, 0, 0, 0, 0, 0};
        int seen = 0;
        for (int h = 0; h < (1 << high_bits); ++h) {
            if (__popc(h) != ph) continue;
            if (seen++ % parts != part) continue;
            for (int e = lane; e < E; e += 64) {
                const uint32_t at = s_at[e];
                if (((at >> kLow) & ~(uint32_t)h & 31u) != 0u) continue;
                const int w = s_load[e];
#pragma unroll
                for (uint32_t i = 0; i < 4; ++i)
                    if (at >> (16 + i) & 1u) atomicAdd(&s_f[(at & (uint32_t)(kTable - 1)) ^ (i << 2)], w);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            int v[32];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int4 w = *reinterpret_cast<const int4*>(s_f + table_slot(q * 256 + lane * 4));
                v[4 * q] = w.x; v[4 * q + 1] = w.y; v[4 * q + 2] = w.z; v[4 * q + 3] = w.w;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (E <= 256) {      // few experts touch few entries
                for (int e = lane; e < E; e += 64) {
                    const uint32_t at = s_at[e] & (uint32_t)(kTable - 1);
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) s_f[at ^ (i << 2)] = 0;
                }
            } else {
                clear_table(s_f);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int b = 0; b < 5; ++b)
#pragma unroll
                for (int j = 0; j < 32; ++j)
                    if (j & (1 << b)) v[j] += v[j ^ (1 << b)];
#pragma unroll
            for (int j = 0; j < 32; j += 2) {      // lane bit 5 <-> register bit 0
                const auto sw = __builtin_amdgcn_permlane32_swap((unsigned)v[j], (unsigned)v[j + 1], false, false);
                v[j] = (int)sw[0];
                v[j + 1] = (int)(sw[0] + sw[1]);
            }
#pragma unroll
            for (int j = 0; j < 32; j += 2) {      // lane bit 4 <-> register bit 0
                const auto sw = __builtin_amdgcn_permlane16_swap((unsigned)v[j], (unsigned)v[j + 1], false, false);
                v[j] = (int)sw[0];
                v[j + 1] = (int)(sw[0] + sw[1]);
            }
#pragma unroll
            for (int j = 0; j < 32; ++j) {
                v[j] += __builtin_amdgcn_update_dpp(0, v[j], 0x114, 0xf, 0xa, false);      // lanes with bit 2: from lane - 4
                v[j] += __builtin_amdgcn_update_dpp(0, v[j], 0x118, 0xf, 0xc, false);      // lanes with bit 3: from lane - 8
            }
#pragma unroll
            for (int j = 0; j < 32; ++j) mx[__builtin_popcount(j)] = max(mx[__builtin_popcount(j)], v[j]);
        }
        // whichever index bits lanes and registers hold by now, a subset's size is the number of bits set in both
        const int den0 = __popc((uint32_t)lane) + ph;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const Frac c{mx[k], max(den0 + k, 1)};       // size 0 is the empty set, whose sum is 0
            if (frac_gt(c, best)) best = c;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const Frac o{__shfl_xor(best.num, off, 64), __shfl_xor(best.den, off, 64)};
        if (frac_gt(o, best)) best = o;
    }
    return best;
}

// Few candidates: a block's waves share the patterns of one candidate.  (1024 candidates give every SIMD a wave.)
inline bool share_candidate(int n, int G) { return G > kLow && n < 1024; }

// ---------------------------------------------------------------------------
// step 2: a block scores kCandPerBlock candidates, one per wave, or (SHARE) one
// ---------------------------------------------------------------------------
// DRAW: candidate c is drawn from (counts, slots, seed, c); else it is place[c].
template <bool DRAW, bool SHARE>
__global__ __launch_bounds__(kScoreThreads) void k_score(const int32_t* __restrict__ load, const int32_t* __restrict__ counts,
                                                         const uint8_t* __restrict__ place, int n, int E, int G, int slots,
                                                         uint32_t seed, int64_t* __restrict__ m_num,
                                                         int32_t* __restrict__ m_den) {
    constexpr int kWaves = kScoreThreads / 64, kCand = SHARE ? 1 : kCandPerBlock;
    extern __shared__ __attribute__((aligned(16))) int s_dyn[];
    int* s_f = s_dyn;                                                  // [kWaves][kTable]
    uint32_t* s_mask = (uint32_t*)(s_f + kWaves * kTable);             // [kCandPerBlock][E]
    int* s_load = (int*)(s_mask + kCandPerBlock * E);                  // [E]
    int* s_order = s_load + E;                                         // [E]
    int* s_cnt = s_order + E;                                          // [E]
    __shared__ Frac s_best[kWaves];
    const int tid = threadIdx.x, wave = tid >> 6;
    const int cand0 = blockIdx.x * kCand;
    const int ncand = min(kCand, n - cand0);

    for (int e = tid; e < E; e += kScoreThreads) s_load[e] = max(load[e], 0);
    if constexpr (DRAW) {
        drawing_order(counts, s_cnt, s_order, E);
        // one wave draws (rows past the last candidate draw unused ones); not the same SIMD's in every block of a CU
        uint32_t* s_key = E <= kWaves * kTable / 64 ? (uint32_t*)s_f : nullptr;      // (the tables are cleared later)
        if (s_key != nullptr) draw_keys(s_order, s_key, 64, E, seed, (uint32_t)cand0);
        if (wave == (int)((blockIdx.x ^ (blockIdx.x >> 8)) & (kWaves - 1)))
            draw_rows(s_order, s_key, 64, s_mask, E, G, seed, (uint32_t)cand0);
    } else {
        const uint8_t* pl = place + (size_t)cand0 * E * G;
        for (int i = tid; i < ncand * E; i += kScoreThreads) {
            uint32_t m = 0;
            for (int g = 0; g < G; ++g) m |= (pl[(size_t)i * G + g] != 0 ? 1u : 0u) << g;
            s_mask[i] = m;
        }
    }
    __syncthreads();
    const int mine = SHARE ? 0 : wave;
    Frac best{0, 1};
    bool bad = false;
    if (mine < ncand) {
        uint32_t* masks = s_mask + mine * E;
        if (!SHARE || wave == 0)
            for (int e = tid & 63; e < E; e += 64) {
                const uint32_t m = masks[e];
                bad |= m == 0 && s_load[e] > 0;                                            // load, but no replica
                masks[e] = additions(m, s_load[e], e);
            }
        bad = __ballot(bad) != 0ull;
        if (SHARE) __syncthreads();
        clear_table(s_f + wave * kTable);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        best = max_density(s_f + wave * kTable, masks, s_load, E, G, SHARE ? wave : 0, SHARE ? kWaves : 1);
    }
    if constexpr (SHARE) {
        if ((tid & 63) == 0) s_best[wave] = best;
        __syncthreads();
        for (int w = 0; w < kWaves; ++w)
            if (frac_gt(s_best[w], best)) best = s_best[w];
    }
    if ((tid & 63) == 0 && mine < ncand && (!SHARE || wave == 0)) {
        int a = best.num, b = best.den;
        while (b != 0) {
            const int t = a % b;
            a = b;
            b = t;
        }
        m_num[cand0 + mine] = bad ? -1 : best.num / a;      // gcd(0, den) = den: zero comes out as 0 / 1
        m_den[cand0 + mine] = bad ? 0 : best.den / a;
    }
}

// ---------------------------------------------------------------------------
// step 2 for more than 16 ranks: 2^G subsets cannot be enumerated.  One wavefront per candidate
// finds the same m with exact integer flows (flow::exact_density) and writes it as a reduced
// fraction.  Loads summing to 2^31 / G or more do not fit the scaled flow: then M* = ceil(m) is
// written as M* / 1.
// ---------------------------------------------------------------------------
template <bool DRAW, typename M, int MAXW>
__global__ __launch_bounds__(64) void k_score_flow(const int32_t* __restrict__ load, const int32_t* __restrict__ counts,
                                                   const uint8_t* __restrict__ place, int E, int G, int slots,
                                                   uint32_t seed, int xs, int64_t* __restrict__ m_num, int32_t* __restrict__ m_den) {
    extern __shared__ __attribute__((aligned(16))) char s_flow[];
    auto c = flow::make_problem(s_flow, E, G, xs);
    int* s_order = reinterpret_cast<int*>(s_flow + flow::ctx_bytes(E, G, xs));      // [E]
    int* s_cnt = s_order + E;                                                   // [E]
    const int l = threadIdx.x;
    const uint32_t cand = blockIdx.x;
    if constexpr (DRAW) {
        drawing_order(counts, s_cnt, s_order, E);
        draw_candidate(s_order, c.pm, E, G, slots, seed, cand);
    } else {
        const uint8_t* pl = place + (size_t)cand * E * G;
        for (int e = l; e < E; e += 64) {
            flow::u64 m = 0ull;
            for (int g = 0; g < G; ++g) m |= (flow::u64)(pl[(size_t)e * G + g] != 0) << g;
            c.pm[e] = m;
        }
    }
    __syncthreads();
    const bool bad = flow::compact(c, load);
    long long Pl = 0;
    for (int e = l; e < E; e += 64) Pl += max(load[e], 0);
    Pl += __shfl_xor(Pl, 32, 64); Pl += __shfl_xor(Pl, 16, 64); Pl += __shfl_xor(Pl, 8, 64);
    Pl += __shfl_xor(Pl, 4, 64); Pl += __shfl_xor(Pl, 2, 64); Pl += __shfl_xor(Pl, 1, 64);
    int num = -1, den = 0;
    if (!bad) flow::with_words<MAXW>(c.n, [&](auto words) {
        flow::Flow<M, words.value> f(c);
        if (Pl * G < 0x7fffffffll) {
            flow::exact_density(f, load, (int)Pl, &num, &den);
            int a = num, b = den;                     // reduce by the greatest common divisor
            while (b != 0) { const int t = a % b; a = b; b = t; }
            if (a > 1) { num /= a; den /= a; }
            if (num == 0) den = 1;
        } else {
            flow::start_on_first_replicas(f, load);
            num = flow::optimum_value(f, (int)min(Pl, 0x7fffffffll));
            den = 1;
        }
    });
    if (l == 0) {
        m_num[cand] = num;
        m_den[cand] = den;
    }
}

// ---------------------------------------------------------------------------
// the best candidate
// ---------------------------------------------------------------------------
constexpr int kPickThreads = 1024, kPickKeys = 256;      // experts whose keys are made beforehand

__global__ __launch_bounds__(kPickThreads) void k_pick(const int64_t* __restrict__ m_num, const int32_t* __restrict__ m_den, int n,
                                              const int32_t* __restrict__ counts, int E, int G, int slots, uint32_t seed,
                                              int32_t* __restrict__ best_out, uint8_t* __restrict__ place) {
    extern __shared__ __attribute__((aligned(16))) int s_dyn[];
    u64* s_mask = (u64*)s_dyn;               // [E]
    int* s_order = (int*)(s_mask + E);       // [E]
    int* s_cnt = s_order + E;                // [E]
    __shared__ int s_idx[kPickThreads / 64], s_num[kPickThreads / 64], s_den[kPickThreads / 64];
    const int tid = threadIdx.x;
    // smallest m, then lowest index; candidates flagged infeasible (den == 0) never win
    int bi = -1, bn = 0, bd = 1;
    for (int c0 = tid; c0 < n; c0 += 4 * kPickThreads) {
        int cn[4], cd[4];                                     // four loads in flight (past the end: the last again)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = min(c0 + j * kPickThreads, n - 1);
            cn[j] = (int)m_num[c];
            cd[j] = m_den[c];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = c0 + j * kPickThreads;
            if (c >= n || cd[j] <= 0) continue;
            if (bi < 0 || (i64)cn[j] * bd < (i64)bn * cd[j]) {      // ascending c: strict '<' keeps the lower index
                bi = c; bn = cn[j]; bd = cd[j];
            }
        }
    }
    // (better: smaller m, then lower index; any candidate is better than none)
    auto take = [&](int i, int num, int den) {
        const i64 l = (i64)num * bd, r = (i64)bn * den;
        if (i >= 0 && (bi < 0 || l < r || (l == r && i < bi))) {
            bi = i; bn = num; bd = den;
        }
    };
#pragma unroll 1      // (code that runs once costs its fetch)
    for (int off = 32; off > 0; off >>= 1) take(__shfl_xor(bi, off, 64), __shfl_xor(bn, off, 64), __shfl_xor(bd, off, 64));
    if ((tid & 63) == 0) {
        s_idx[tid >> 6] = bi; s_num[tid >> 6] = bn; s_den[tid >> 6] = bd;
    }
    __syncthreads();
    bi = s_idx[tid & 15]; bn = s_num[tid & 15]; bd = s_den[tid & 15];
    static_assert(kPickThreads / 64 == 16, "one entry per wave");
#pragma unroll 1
    for (int off = 8; off > 0; off >>= 1) take(__shfl_xor(bi, off, 64), __shfl_xor(bn, off, 64), __shfl_xor(bd, off, 64));
    const int best = __builtin_amdgcn_readfirstlane(bi);
    if (tid == 0) best_out[0] = best;
    if (best < 0) {
        for (int i = tid; i < E * G; i += kPickThreads) place[i] = 0;
        return;
    }
    drawing_order(counts, s_cnt, s_order, E);
    uint32_t* s_rows = (uint32_t*)(s_cnt + E);      // [4][E], every row the winner's (G <= kMaxEnumG)
    uint32_t* s_key = G <= kMaxEnumG && E <= kPickKeys ? s_rows + 4 * E : nullptr;
    if (s_key != nullptr) draw_keys(s_order, s_key, 16, E, seed, (uint32_t)best);
    if (tid < 64) {
        if (G <= kMaxEnumG) draw_rows(s_order, s_key, 16, s_rows, E, G, seed, (uint32_t)best);
        else draw_candidate(s_order, s_mask, E, G, slots, seed, (uint32_t)best);
    }
    __syncthreads();
    for (int i = tid; i < E * G; i += kPickThreads)
        place[i] = (uint8_t)(((G <= kMaxEnumG ? (u64)s_rows[i / G] : s_mask[i / G]) >> (i % G)) & 1ull);
}

template <bool DRAW>
int launch_score(const fine_shape& s, const int32_t* load, const int32_t* counts, const uint8_t* place, int n, int slots,
                 uint32_t seed, int64_t* m_num, int32_t* m_den, hipStream_t st) {
    const bool share = share_candidate(n, s.G);
    auto k = share ? k_score<DRAW, true> : k_score<DRAW, false>;
    const size_t lds = ((size_t)(kScoreThreads / 64) * kTable + (kCandPerBlock + 3) * (size_t)s.E) * 4;
    hipLaunchKernelGGL(k, dim3(cdiv(n, share ? 1 : kCandPerBlock)), dim3(kScoreThreads), lds, st, load, counts, place, n, s.E,
                       s.G, slots, seed, m_num, m_den);
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

}  // namespace

// ---- symmetric placements from Cayley graphs (Appendix B): expert = edge {a, a + s} ----------------
struct CayleyDesc {
    int n_factors, n_gens, complete;
    int orders[kCayleyMaxFactors];
    int gen[kCayleyMaxGens][kCayleyMaxFactors];      // reduced modulo the orders
    int own_inverse[kCayleyMaxGens];
    int first[kCayleyMaxGens + 1];                    // first expert of each generator's edges
};

namespace {

__global__ __launch_bounds__(256) void k_cayley(CayleyDesc c, int E, int G, uint8_t* __restrict__ place) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= E * G) return;
    const int e = i / G, g = i - e * G;
    int a = 0, b = 0;
    const int pairs = G * (G - 1) / 2;
    if (e < c.complete * pairs) {
        // pair number t of the pairs a < b in lexicographic order
        int t = e % pairs;
        a = 0;
        while (t >= G - 1 - a) { t -= G - 1 - a; ++a; }
        b = a + 1 + t;
    } else {
        int j = 0;
        while (j + 1 < c.n_gens && e >= c.first[j + 1]) ++j;
        int t = e - c.first[j];
        // the t-th rank (ascending) that owns an edge of generator j
        for (a = 0; a < G; ++a) {
            int rest = a, w = 0, mul = 1;
            for (int f = c.n_factors - 1; f >= 0; --f) {           // last factor fastest
                const int n = c.orders[f], v = rest % n;
                rest /= n;
                w += ((v + c.gen[j][f]) % n) * mul;
                mul *= n;
            }
            b = w;
            if (c.own_inverse[j] && b < a) continue;
            if (t-- == 0) break;
        }
    }
    place[i] = (g == a || g == b) ? 1 : 0;
}

}  // namespace

int launch_cayley_placement(const fine_shape& s, int n_factors, const int32_t* orders, int n_gens, const int32_t* gens,
                            int complete, uint8_t* place, hipStream_t st) {
    CayleyDesc c{};
    c.n_factors = n_factors; c.n_gens = n_gens; c.complete = complete;
    long long G = 1;
    for (int f = 0; f < n_factors; ++f) {
        if (orders[f] < 1) return FINE_INVALID_ARG;
        c.orders[f] = orders[f];
        G *= orders[f];
        if (G > 64) return FINE_INVALID_ARG;
    }
    if (G != s.G) return FINE_INVALID_ARG;
    long long count = (long long)complete * s.G * (s.G - 1) / 2;
    for (int j = 0; j < n_gens; ++j) {
        bool zero = true, own = true;
        for (int f = 0; f < n_factors; ++f) {
            const int n = orders[f], v = ((gens[j * n_factors + f] % n) + n) % n;
            c.gen[j][f] = v;
            zero = zero && v == 0;
            own = own && (2 * v) % n == 0;
        }
        if (zero) return FINE_INVALID_ARG;                 // the identity is no generator
        c.own_inverse[j] = own;
        c.first[j] = (int)count;
        count += own ? s.G / 2 : s.G;
    }
    c.first[n_gens] = (int)count;
    if (count != s.E) return FINE_INVALID_ARG;
    hipLaunchKernelGGL(k_cayley, dim3(cdiv(s.E * s.G, 256)), dim3(256), 0, st, c, s.E, s.G, place);
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

int launch_replica_counts(const fine_shape& s, const int32_t* load, int slots, int32_t* counts, hipStream_t st) {
    hipLaunchKernelGGL(k_replica_counts, dim3(1), dim3(64), 0, st, load, s.E, s.G, slots, counts);
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

int launch_eval_placements(const fine_shape& s, int n, const uint8_t* place, const int32_t* load, int64_t* m_num,
                           int32_t* m_den, hipStream_t st) {
    if (n == 0) return FINE_OK;
    if (s.G > kMaxEnumG) {
        const size_t rest = 2 * (size_t)s.E * 4;
        if (!flow::size_allowed(s.E, s.G, 64 * 1024 - rest)) return FINE_UNSUPPORTED;
        const int xs = flow::x_stride(s.E, s.G, 64 * 1024 - rest);
        const size_t lds = flow::ctx_bytes(s.E, s.G, xs) + rest;
        auto k = flow::by_size(s.E, s.G, [](auto words, auto m) { return k_score_flow<false, decltype(m), words.value>; });
        hipLaunchKernelGGL(k, dim3(n), dim3(64), lds, st, load, (const int32_t*)nullptr, place, s.E, s.G, 0,
                           0u, xs, m_num, m_den);
        FINE_LAUNCH_CHECK();
        return FINE_OK;
    }
    return launch_score<false>(s, load, nullptr, place, n, 0, 0u, m_num, m_den, st);
}

int launch_place_search(const fine_shape& s, const int32_t* load, const int32_t* counts, int slots, int n, uint32_t seed,
                        int64_t* m_num, int32_t* m_den, int32_t* best, uint8_t* place, hipStream_t st) {
    if (s.G > kMaxEnumG) {
        const size_t rest = 2 * (size_t)s.E * 4;
        if (!flow::size_allowed(s.E, s.G, 64 * 1024 - rest)) return FINE_UNSUPPORTED;
        const int xs = flow::x_stride(s.E, s.G, 64 * 1024 - rest);
        const size_t lds = flow::ctx_bytes(s.E, s.G, xs) + rest;
        auto k = flow::by_size(s.E, s.G, [](auto words, auto m) { return k_score_flow<true, decltype(m), words.value>; });
        hipLaunchKernelGGL(k, dim3(n), dim3(64), lds, st, load, counts, (const uint8_t*)nullptr, s.E, s.G,
                           slots, seed, xs, m_num, m_den);
    } else {
        FINE_TRY(launch_score<true>(s, load, counts, nullptr, n, slots, seed, m_num, m_den, st));
    }
    FINE_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_pick, dim3(1), dim3(kPickThreads), ((size_t)8 * s.E + (s.E <= kPickKeys ? 16 * s.E : 0)) * 4, st, m_num, m_den, n, counts, s.E, s.G, slots, seed,
                       best, place);
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

}  // namespace fine
