// Replica loads for a restricted placement: the canonical integer optimum of Eq. 1
// (Section 4.1), found with exact integer flows by ONE wavefront.
//
// View used (the paper's graph abstraction, Section 5.1): ranks are vertices; an expert
// with units on rank a and a replica on rank b lets load move from a to b.  A[a][b] is the
// total load that may move a -> b.  With G <= 64, vertex sets are 64-bit masks and a
// breadth-first search is a few ballots.
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
#include "flow_wave.h"

namespace fine {

namespace {

using namespace flow;

// Take `amount` units of listed expert j from the replicas in `from` (a subset of its later
// replicas `later`, lowest first) to rank g.  Variable (j,g) itself is not free, so only
// the rows of the source ranks change in A.
template <typename M>
__device__ inline void pull_expert(Ctx<M>& c, int j, int g, M later, M from, int amount) {
    // lane q = source rank q: what the lower sources leave of `amount` is a prefix sum away
    const int q = lane();
    int* row = c.x + j * c.XS;
    const int m = q < c.G && has(from, q & (8 * (int)sizeof(M) - 1)) ? row[q] : 0;
    const int inc = wave_incl_scan_i(m);
    const int t = max(0, min(m, amount - (inc - m)));
    if (t > 0) {
        row[q] = m - t;
        c.ld -= t;
    }
    // row s of A loses what source s gave towards every other later replica: lane q = column q
    const bool is_later = q < c.G && has(later, q & (8 * (int)sizeof(M) - 1));
    M givers = (M)__ballot(t > 0);
    int total = 0;
    while (givers) {
        const int s = first_of(givers);
        givers &= givers - 1;
        const int ts = __builtin_amdgcn_readlane(t, s);
        total += ts;
        if (q != s && is_later) {
            const int v = c.a(s, q) - ts;
            c.a(s, q) = v;
            c.in = (c.in & ~((M)1 << s)) | (M)(v > 0) << s;
        }
    }
    if (q == g) {                                      // g is not among the later replicas: nobody else writes these
        row[g] += total;
        c.ld += total;
    }
    wave_sync();
}

// Warm start (Section 4.1: between micro-batches only the loads change, so the previous solution is
// a good place to start from).  Every listed expert's previous row, restricted to its replicas, is scaled
// to the new load (rounded down, the rest to the first replica); x, A and the rank loads are
// filled from that.  Any assignment of the loads to replicas is a valid start for phase 1, and the
// result of phase 2 does not depend on where it started, so `prev` may hold anything: negative
// entries read as 0, a row without units falls back to the first replica.  `prev` is read completely before this
// function returns.  The rows of all experts are first copied into x, in wide batches of loads (a lane that walks
// its expert's row in global memory waits for every entry: 32 round trips for an expert on all of 32 ranks), then
// the listed ones are scaled and moved to their places in the list.
template <typename M>
__device__ inline void start_from_previous(Ctx<M>& c, const int32_t* __restrict__ load, const int32_t* prev) {
    const int l = lane();
    for (int i = l; i < c.G * c.AS; i += kW) c.A[i] = 0;
    if (l < c.G) c.t[l] = c.single;
    constexpr int kBatch = 16;
    const int per = kW / c.G, row0 = l / c.G, col = l - row0 * c.G;      // rows of E x G per wave instruction
    for (int r0 = row0; r0 < c.E; r0 += kBatch * per) {
        int v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) v[k] = prev[(size_t)min(r0 + k * per, c.E - 1) * c.G + col];
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
            if (row0 < per && r0 + k * per < c.E) c.x[(r0 + k * per) * c.XS + col] = v[k];
    }
    wave_sync();
    int n = 0;
    for (int base = 0; base < c.E; base += kW) {
        const u64 w = readlane_u64(c.listed, base / kW);
        const bool mine = (w >> l) & 1ull;
        const int e = base + l, j = n + __popcll(w & ((1ull << l) - 1ull));
        const u64 m = mine ? c.pm[j] : 0ull;
        if (mine) {
            int* row = c.x + e * c.XS;
            const int le = max(load[e], 0);
            const int first = __ffsll((long long)m) - 1;
            // (floating point: any split that adds up to the load will do)
            float had = 0.f;
            for (u64 r = m; r; r &= r - 1) had += (float)max(row[__ffsll((long long)r) - 1], 0);
            const float scale = had > 0.f ? (float)le / had : 0.f;
            int left = le;
            for (u64 r = m; r; r &= r - 1) {
                const int a = __ffsll((long long)r) - 1;
                const int t = (int)fminf((float)max(row[a], 0) * scale, (float)left);
                row[a] = min(t, left);
                left -= min(t, left);
            }
            row[first] += left;
            for (u64 r = m; r; r &= r - 1) {
                const int a = __ffsll((long long)r) - 1;
                const int t = row[a];
                if (t == 0) continue;
                atomicAdd(&c.t[a], t);
                for (u64 o = m & ~(1ull << a); o; o &= o - 1) atomicAdd(&c.a(a, (__ffsll((long long)o) - 1)), t);
            }
        }
        // to the rows of the list, in ascending order: row j is an expert's that is not listed or has moved already.
        wave_sync();
        for (u64 r = w; r; r &= r - 1) {
            const int k = __ffsll((long long)r) - 1;
            if (l < c.G) c.x[n * c.XS + l] = (readlane_u64(m, k) >> l) & 1ull ? c.x[(base + k) * c.XS + l] : 0;
            ++n;
        }
        wave_sync();
    }
    load_registers(c);
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

template <typename M>
__global__ __launch_bounds__(64) void k_general_x(const uint8_t* __restrict__ place, const int32_t* __restrict__ load,
                                                  const int32_t* prev, int E, int G, int xs, int P, int32_t* x_out,
                                                  int32_t* __restrict__ max_load) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    Ctx<M> c = make_ctx<M>(smem, E, G, xs);
    const int l = lane();

    // ---- set-up: masks, the list, x, A, rank loads --------------------
    for (int e = l; e < E; e += kW) c.pm[e] = replica_mask(place, e, G);
    wave_sync();
    if (compact(c, load)) {                        // an expert with load and no replica: no schedule exists
        for (int i = l; i < E * G; i += kW) x_out[i] = 0;
        if (l == 0) max_load[0] = -1;
        return;
    }
    if (prev) start_from_previous(c, load, prev);
    else start_on_first_replicas(c, load);

    // ---- phase 1: the optimum value ---------------------------------------------------------
    const int cap_rank = optimum_value(c, P);      // M*
    if (l == 0) max_load[0] = cap_rank;

    // ---- phase 2: the lexicographically greatest optimum ------------------------------------
    for (int j = 0; j < c.n; ++j) {
        M todo = (M)c.pm[j];
        M F = todo;                         // free replicas of j (including the one being removed next)
        const int* row = c.x + j * c.XS;
        while (todo) {
            const int g = first_of(todo);
            todo &= todo - 1;
            // variable (j,g) leaves the free set: its units can no longer move to the other free
            // replicas, nor theirs to g (lane q updates the two entries that involve replica q)
            F &= ~((M)1 << g);
            const M later = F;
            if (later == 0) continue;        // the last replica: nothing left to take units from
            const bool is_later = l < G && has(later, l & (8 * (int)sizeof(M) - 1));
            int back = 0;
            if (is_later) {
                const int to_me = c.a(g, l) - row[g];
                back = c.a(l, g) - row[l];
                c.a(g, l) = to_me;
                c.a(l, g) = back;
                c.in = (c.in & ~((M)1 << g)) | (M)(to_me > 0) << g;
            }
            const M still = (M)__ballot(back > 0);
            if (l == g) c.in = (c.in & ~later) | still;
            wave_sync();
            while (true) {
                const int avail = is_later ? row[l] : 0;
                if (__ballot(avail > 0) == 0ull) break;
                const int total_avail = wave_sum_i(avail);
                const int room = cap_rank - __builtin_amdgcn_readlane(c.ld, g);
                if (room > 0) {
                    pull_expert(c, j, g, later, later, min(room, total_avail));
                    continue;
                }
                const bool want = l < G && (c.ld < cap_rank || avail > 0);
                M visited; int parent, cap;
                const int r = bfs(c, g, want, &visited, &parent, &cap);
                if (r < 0) break;
                const int room_r = cap_rank - __builtin_amdgcn_readlane(c.ld, r);
                if (room_r > 0) {
                    // the path may itself carry units of j between its later replicas, so
                    // the units are taken from whichever later replicas hold them afterwards
                    const int amount = min(min(room_r, cap), total_avail);
                    push_path(c, g, r, parent, amount, j, g);
                    pull_expert(c, j, g, later, later, amount);
                } else {
                    const int amount = min(cap, __builtin_amdgcn_readlane(avail, r));
                    pull_expert(c, j, g, later, (M)1 << r, amount);
                    push_path(c, g, r, parent, amount, j, g);
                }
            }
        }
    }
    // ---- out: rows of the list; the load on the only replica for the others (their masks were dropped) --------
    int n = 0;
    const int per = kW / G, row0 = l / G, col = l - row0 * G;      // rows of E x G per wave instruction
    for (int base = 0; base < E; base += kW) {
        const u64 w = readlane_u64(c.listed, base / kW);
        const int e = min(base + l, E - 1);
        const int only = __ffsll((long long)replica_mask(place, e, G)) - 1, le = max(load[e], 0);
        const int rows = min(kW, E - base);
        for (int r = 0; r < rows; r += per) {
            const int k = min(r + row0, kW - 1);
            const int rank_k = __shfl(only, k, kW), load_k = __shfl(le, k, kW);
            const int j = n + __popcll(w & ((1ull << k) - 1ull));
            const int v = (w >> k) & 1ull ? c.x[j * c.XS + col] : rank_k == col ? load_k : 0;
            if (row0 < per && r + row0 < rows) x_out[(size_t)(base + k) * G + col] = v;
        }
        n += __popcll(w);
    }
}

}  // namespace

int launch_general_x(const fine_shape& s, const uint8_t* place, const int32_t* load, const int32_t* x_prev,
                     int32_t* x_eg, int32_t* max_load, hipStream_t st) {
    const int xs = flow::x_stride(s.E, s.G, 160 * 1024);
    const size_t lds = flow::ctx_bytes(s.E, s.G, xs);
    if (lds > 160 * 1024) return FINE_UNSUPPORTED;
    static std::atomic<uint64_t> lds_set32{0}, lds_set64{0};
    auto k = s.G <= 32 ? k_general_x<uint32_t> : k_general_x<u64>;
    FINE_TRY(raise_lds_limit((const void*)k, 160 * 1024, s.G <= 32 ? lds_set32 : lds_set64));
    hipLaunchKernelGGL(k, dim3(1), dim3(64), lds, st, place, load, x_prev, s.E, s.G, xs, s.T * s.K, x_eg, max_load);
    FINE_LAUNCH_CHECK();
    return FINE_OK;
}

}  // namespace fine
