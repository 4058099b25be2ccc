// Replica loads for a restricted placement: the canonical integer optimum of Eq. 1
// (Section 4.1), found with exact integer flows by ONE wavefront; the other waves of its block help to set the
// problem up and to write the result out.
//
// View used (the paper's graph abstraction, Section 5.1): ranks are vertices; an expert
// with units on rank a and a replica on rank b lets load move from a to b.  With G <= 64, vertex sets are 64-bit masks
// and a breadth-first search is a few ballots.
//
// Experts with one replica never move; the others form a list (flow_wave.h).
//
// Phase 1 (optimum value M*).  Start with every expert on its first replica and M =
// ceil(P/G).  While some rank a exceeds M, search from a for a rank below M and push the
// bottleneck amount along the path.  If the search finds none, the reached set S is closed
// (no expert with load in S has a replica outside S), so Eq. 3 gives the lower bound
// ceil(load(S)/|S|) > M; M jumps to it.  M only ever moves to lower bounds of the optimum
// and the loop ends with a feasible flow, hence M = M*.
//
// Phase 2 (canonical choice).  Variables are visited in order (e ascending, g ascending in
// G_EDP^e).  x[e][g] is raised as far as possible by taking units of e from its later
// replicas, first into free room on g, then along augmenting paths through loads that are
// still free to move (later variables only), ending on a rank with room or on the later
// replica the units came from.  When no such path exists x[e][g] is maximal given the
// earlier variables, i.e. the result is the lexicographically greatest optimum, which is
// unique: the order in which paths are found does not change it.
#include "route.h"

namespace fine {

namespace {

using namespace flow;

// Take `amount` units of listed expert j from the replicas in `from` (a subset of its later replicas, lowest first) to
// rank g.  Variable (j,g) itself is not free.
template <typename M, int NW, typename PM>
__device__ inline void pull_expert(Flow<M, NW, PM>& c, int j, int g, M from, int amount) {
    // lane q = source rank q: what the lower sources leave of `amount` is a prefix sum away
    const int q = lane();
    int* row = c.x + j * c.XS;
    const int m = (from & c.me) != 0 ? row[q] : 0;
    const int inc = wave_incl_scan_i(m);
    const int t = max(0, min(m, amount - (inc - m)));
    if (t > 0) {
        row[q] = m - t;
        c.ld -= t;
    }
    if (q == g) {
        row[g] += amount;
        c.ld += amount;
    }
    wave_sync();
    c.gave(j, t, m);
}

// Phases 1 and 2 by one wavefront; returns M*.  On return c.ld are the ranks' loads.
template <typename M, int NW, typename PM>
__device__ inline int solve(Flow<M, NW, PM>& c, int P) {
    const int l = lane();
    c.load_registers();
    // ---- phase 1: the optimum value ---------------------------------------------------------
    const int cap_rank = optimum_value(c, P);      // M*
    // ---- phase 2: the lexicographically greatest optimum ------------------------------------
    for (int j = 0; j < c.n; ++j) {
        M later = c.begin(j);                      // free replicas of j (including the one being removed next)
        while (true) {
            const int g = first_of(later);
            later &= later - 1;
            if (later == 0) break;                 // the last replica: nothing left to take units from (or to move them to)
            c.fix(j, g);
            while (true) {
                const bool mine = c.has_units(j);
                if (__ballot(mine) == 0ull) break;
                const int room = cap_rank - __builtin_amdgcn_readlane(c.ld, g);
                if (room > 0) {
                    pull_expert(c, j, g, later, min(room, wave_sum_i(c.units_of(j, mine))));
                    continue;
                }
                const auto way = c.bfs(g, (M)__ballot(l < c.G && c.ld < cap_rank) | (M)__ballot(mine));
                if (way.target < 0) break;
                const int avail = c.units_of(j, mine), room_r = cap_rank - __builtin_amdgcn_readlane(c.ld, way.target);
                if (room_r > 0) {
                    // the path may itself carry units of j between its later replicas, so
                    // the units are taken from whichever later replicas hold them afterwards
                    const int moved = push(c, way, min(room_r, wave_sum_i(avail)));
                    pull_expert(c, j, g, later, moved);
                } else {                           // all ranks on the way are full: exactly as much must come as goes
                    const int amount = min(way_capacity(c, way), __builtin_amdgcn_readlane(avail, way.target));
                    pull_expert(c, j, g, (M)1 << way.target, amount);
                    push(c, way, amount);
                }
            }
        }
    }
    return cap_rank;
}

// the ranks that hold a replica of expert e
__device__ inline u64 replica_mask(const uint8_t* __restrict__ place, int e, int G) {
    u64 m = 0ull;
    if (((reinterpret_cast<uintptr_t>(place) | (uintptr_t)G) & 15u) == 0) {      // 16 ranks per load, all of a row in flight
        uint4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const uint4*>(place + (size_t)e * G + min(16 * k, G - 16));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t d[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
            unsigned bits = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) bits |= (unsigned)(((d[i >> 2] >> (8 * (i & 3))) & 255u) != 0u) << i;
            if (16 * k < G) m |= (u64)bits << (16 * k);
        }
    } else {
        for (int g = 0; g < G; ++g)
            if (place[(size_t)e * G + g]) m |= 1ull << g;
    }
    return m;
}

constexpr int kXThreads = 1024, kXWaves = kXThreads / kW;

// LDS: the replica masks, whose place the experts' places (16 bits) take once the wavefront is done; one region for, in turn,
// the set-up's arrays (which experts are listed, a flag, the experts of the list in 16 bits), the sums of the edges and the
// waves' sums of the output; x and t.
__host__ __device__ inline size_t x_masks_bytes(int E, int mask_bytes) { return ((size_t)E * mask_bytes + 15) & ~(size_t)15; }
__host__ __device__ inline size_t x_shared_bytes(int E, int G) {
    const size_t setup = (size_t)(E + kW - 1) / kW * 8 + 8 + ((size_t)E * 2 + 3 & ~(size_t)3), sums = (size_t)kXWaves * G * 4;
    const size_t most = setup > sums ? setup : sums;
    return edge_bytes(E, G) > most ? edge_bytes(E, G) : most;
}
__host__ __device__ inline size_t x_bytes(int E, int G, int xs, int mask_bytes) {
    return x_masks_bytes(E, mask_bytes) + x_shared_bytes(E, G) + ((size_t)E * xs + G) * 4;
}

// prev (warm start, Section 4.1: between micro-batches only the loads change, so the previous solution is a good place
// to start from): every listed expert's previous row, restricted to its replicas, is scaled to the new load (rounded
// down, the rest to the first replica).  Any assignment of the loads to replicas is a valid start for phase 1, and the
// result of phase 2 does not depend on where it started, so `prev` may hold anything: negative entries read as 0, a row
// without units falls back to the first replica.  It may be x_out: it is read completely before that is written.
//
// 256 experts with 320 replicas on 32 ranks, warm: 173 -> 100 us (20 experts, 50 replicas, 5 ranks: 31 -> 23).  The search
// itself is bound by its count of dependent instructions (one wavefront issues one every 4-5 cycles, a value that goes from
// the vector to the scalar side waits several of those) and LDS round trips: some 95 searches of 430 cycles and 135 hops of
// pushes; a hop took 1200 cycles while the capacity of every edge was kept up to date, and takes some 500.  Set-up and
// output, 95 K of 433 K cycles when the one wavefront did them too, are 18 K with sixteen.
template <typename M, int MAXW>
__global__ __launch_bounds__(kXThreads) void k_general_x(const uint8_t* __restrict__ place, const int32_t* __restrict__ load,
                                                         const int32_t* prev, int E, int G, int xs, int P, int32_t* x_out,
                                                         int32_t* __restrict__ max_load, const int32_t* __restrict__ input_eg,
                                                         int locality, RouteTables route, int32_t* __restrict__ seg_off,
                                                         int32_t* __restrict__ rank_off) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    Problem<M> c;
    c.E = E; c.G = G; c.XS = xs;
    c.pm = reinterpret_cast<M*>(smem);
    char* const shared = smem + x_masks_bytes(E, sizeof(M));
    c.A = reinterpret_cast<int*>(shared);
    c.x = reinterpret_cast<int*>(shared + x_shared_bytes(E, G));
    c.t = c.x + (size_t)E * xs;
    u64* listed = reinterpret_cast<u64*>(shared);
    int* bad = reinterpret_cast<int*>(listed + (E + kW - 1) / kW);
    int16_t* expert = reinterpret_cast<int16_t*>(bad + 2);
    int* sums = reinterpret_cast<int*>(shared);        // [waves][G], after the solution
    int16_t* slot = reinterpret_cast<int16_t*>(smem);  // the same
    const int tid = threadIdx.x, l = lane(), wave = __builtin_amdgcn_readfirstlane(tid / kW);

    // ---- set-up: masks, the list, x, rank loads (a thread per expert: E <= kXThreads) --------------------
    for (int g = tid; g < G; g += kXThreads) c.t[g] = 0;
    if (tid == 0) *bad = 0;
    __syncthreads();
    const u64 mask = tid < E ? replica_mask(place, tid, G) : 0ull;
    const int mine = tid < E ? max(load[tid], 0) : 0, replicas = __popcll(mask);
    if (replicas == 1 && mine > 0) atomicAdd(&c.t[__ffsll((long long)mask) - 1], mine);
    const u64 in_list = __ballot(replicas > 1);
    if (l == 0 && tid < E) listed[wave] = in_list;
    if (replicas == 0 && mine > 0) *bad = 1;
    __syncthreads();
    if (*bad) {                                    // an expert with load and no replica: no schedule exists
        for (int i = tid; i < E * G; i += kXThreads) x_out[i] = 0;
        if (seg_off != nullptr) {
            for (int i = tid; i < G * (E + 1); i += kXThreads) seg_off[i] = 0;
            for (int i = tid; i < E * G; i += kXThreads) route.wait[i] = route.room_end[i] = 0;
            for (int i = tid; i <= G; i += kXThreads) rank_off[i] = 0;
        }
        if (tid == 0) max_load[0] = -1;
        return;
    }
    int n = 0, j = 0;
    for (int k = 0; k < (E + kW - 1) / kW; ++k) {
        if (k == wave) j = n;
        n += __popcll(listed[k]);
    }
    c.n = n;
    j += __popcll(in_list & ((1ull << l) - 1ull));
    // this thread's expert: its place in the list, or -1 - its only rank (G: on no rank)
    const int my_slot = replicas > 1 ? j : -1 - (replicas == 1 ? __ffsll((long long)mask) - 1 : G);
    if (replicas > 1) {
        c.pm[j] = (M)mask;
        expert[j] = (int16_t)tid;
    }
    __syncthreads();
    for (int i = wave; i < n; i += kXWaves) {      // a wave per listed expert, lane = rank
        const int e = expert[i], le = max(load[e], 0);
        const M m = c.pm[i];
        const bool here = l < G && has(m, l & (8 * (int)sizeof(M) - 1));
        int t = 0;
        if (prev != nullptr) {                     // (floating point: any split that adds up to the load will do)
            const float v = here ? (float)max(prev[(size_t)e * G + l], 0) : 0.f;
            float had = v;
            for (int o = 32; o > 0; o >>= 1) had += __shfl_xor(had, o, kW);
            t = had > 0.f ? (int)fminf(v * ((float)le / had), (float)le) : 0;
            t = max(0, min(t, le - (wave_incl_scan_i(t) - t)));
        }
        const int left = le - wave_sum_i(t);
        if (l == first_of(m)) t += left;
        if (l < G) c.x[i * xs + l] = t;
        if (t > 0) atomicAdd(&c.t[l], t);
    }
    __syncthreads();

    if (wave == 0) {
        int loads = 0;
        with_words<MAXW>(n, [&](auto words) {
            Flow<M, words.value, M> f(c);
            const int m_star = solve(f, P);
            if (l == 0) max_load[0] = m_star;
            loads = f.ld;
        });
        const int first = wave_incl_scan_i(loads) - loads;      // first row of every rank
        if (l < G) {
            c.t[l] = first;
            if (rank_off != nullptr) rank_off[l] = first;
            if (rank_off != nullptr && l == G - 1) rank_off[G] = first + loads;
        }
    }
    __syncthreads();
    if (tid < E) slot[tid] = (int16_t)my_slot;
    __syncthreads();

    // ---- out: a wave per run of experts, lane = rank; the rows of a rank's segments follow one another -------------
    const int per = (E + kXWaves - 1) / kXWaves, e0 = min(wave * per, E), count = min(per, E - e0);
    const int ours = min(e0 + l, E - 1);      // (count <= 64: one expert per lane)
    const int le = max(load[ours], 0), sl = slot[ours], q = min(l, G - 1);
    auto units = [&](int i) {
        const int s = __builtin_amdgcn_readlane(sl, i);
        const int on_list = c.x[max(s, 0) * xs + q];
        return s >= 0 ? on_list : -1 - s == q ? __builtin_amdgcn_readlane(le, i) : 0;
    };
    int sum = 0;
    for (int i = 0; i < count; ++i) sum += units(i);
    if (l < G) sums[wave * G + l] = sum;
    __syncthreads();
    int run = c.t[q];
    for (int w = 0; w < wave; ++w) run += sums[w * G + q];
    for (int i0 = 0; i0 < count; i0 += 4) {
        int in[4] = {0, 0, 0, 0};
        if (seg_off != nullptr)
#pragma unroll
            for (int k = 0; k < 4; ++k) in[k] = input_eg[(size_t)(e0 + min(i0 + k, count - 1)) * G + q];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = i0 + k, e = e0 + i;
            if (i >= count) break;
            const int v = units(i);
            if (l < G) x_out[(size_t)e * G + l] = v;
            if (seg_off != nullptr) {
                write_route(route, e, G, 0, locality, l < G ? in[k] : 0, l < G ? v : 0);
                if (l < G) seg_off[(size_t)l * (E + 1) + e] = run;
            }
            run += v;
        }
    }
    if (seg_off != nullptr && l < G && e0 + count == E && count > 0) seg_off[(size_t)l * (E + 1) + E] = run;
}

}  // namespace

// seg_off, rank_off: written too, with the queues of Algorithm 1 (route.h), unless NULL
int launch_general_x(const fine_shape& s, const uint8_t* place, const int32_t* load, const int32_t* x_prev,
                     int32_t* x_eg, int32_t* max_load, const int32_t* input_eg, const RouteTables& t, int32_t* seg_off,
                     int32_t* rank_off, hipStream_t st) {
    const int mask_bytes = s.G <= 32 ? 4 : 8;
    const size_t limit = 160 * 1024;
    if (!flow::size_allowed(s.E, s.G, limit)) return FINE_UNSUPPORTED;
    const int xs = x_bytes(s.E, s.G, s.G | 1, mask_bytes) <= limit ? s.G | 1 : s.G;
    const size_t lds = x_bytes(s.E, s.G, xs, mask_bytes);
    if (lds > limit) return FINE_UNSUPPORTED;
    static std::atomic<uint64_t> lds_set[2][kMaxWords + 1];
    auto k = flow::by_size(s.E, s.G, [](auto words, auto m) { return k_general_x<decltype(m), words.value>; });
    FINE_TRY(raise_lds_limit((const void*)k, (int)limit, lds_set[s.G <= 32][flow::words_for(s.E)]));
    hipLaunchKernelGGL(k, dim3(1), dim3(kXThreads), lds, st, place, load, x_prev, s.E, s.G, xs, s.T * s.K, x_eg, max_load,
                       input_eg, (s.flags & FINE_FLAG_LOCALITY) ? 1 : 0, t, seg_off, rank_off);
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

}  // namespace fine
