// One-wavefront integer flows on the placement graph (Section 5.1's graph abstraction): ranks are
// vertices, an expert with units on rank a and a replica on rank b lets load move from a to b,
// A[a][b] is the total load that may move a -> b.  With G <= 64 a vertex set is a 64-bit mask and a
// breadth-first search is a few ballots.  Shared by the scheduler's replica-load solver and by the
// placement scoring for more than 16 ranks.
#pragma once

#include "common.h"

namespace fine {
namespace flow {

constexpr int kW = 64;
typedef unsigned long long u64;

// Only experts with several replicas can move: they are kept in a compact list, in ascending order (256 experts
// with 320 replicas: at most 64 of them, one per lane).  What a rank needs at every step is in the registers of its
// lane: its load and the set of ranks that load may come from; A, which is only read where an edge is used, is in LDS.
// M: a set of ranks, 32 bits where that is enough (the search is a chain of instructions of one wavefront, and 64-bit
// shifts and selects are several each).
template <typename M>
struct Ctx {
    int* x;        // [n][XS] units of listed expert j on every rank
    u64* pm;       // [n] replica masks of the listed experts (before compact(): of all experts)
    int* A;        // [G][AS], stored by destination: a(from, to) = A[to * AS + from]
    int* t;        // [G] scratch
    int E, G;
    int AS, XS;    // row strides (odd where they fit, so that a column's entries fall into different banks)
    int n;         // listed experts
    u64 listed;    // lane i: which of the experts 64 i .. 64 i + 63 are listed
    int single;    // lane = rank: load of the experts whose only replica is here
    int ld;        // lane = rank: its load
    M in;          // lane = rank: the ranks `a` with a(a, lane) > 0
    __device__ int& a(int from, int to) const { return A[to * AS + from]; }
};

__device__ inline int lane() { return threadIdx.x; }
__device__ inline u64 readlane_u64(u64 v, int src) {
    const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)v, src), hi = __builtin_amdgcn_readlane((int)(unsigned)(v >> 32), src);
    return ((u64)hi << 32) | lo;
}
template <typename M>
__device__ inline int first_of(M m) {
    if constexpr (sizeof(M) == 4) return __ffs((int)m) - 1;
    else return __ffsll((long long)m) - 1;
}
template <typename M>
__device__ inline M readlane_set(M v, int src) {
    if constexpr (sizeof(M) == 4) return (M)__builtin_amdgcn_readlane((int)v, src);
    else return readlane_u64(v, src);
}
template <typename M>
__device__ inline bool has(M m, int i) { return (m >> i) & (M)1; }
// LDS accesses of one wavefront are performed in order: only the compiler has to keep the order
__device__ inline void wave_sync() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Wave-wide scan and sum by DPP (data-parallel primitives: an operand taken from another lane of
// the same ALU instruction), six steps and no LDS traffic: shifts by 1, 2, 4, 8 inside each row of
// 16 lanes, then lane 15 of rows 0 and 2 added to rows 1 and 3, then lane 31 to rows 2 and 3.  A lane
// whose source lies outside its row takes the first argument (0).  All 64 lanes must be active.
template <int CTRL, int ROW_MASK>
__device__ inline int dpp_from(int identity, int v) {
    return __builtin_amdgcn_update_dpp(identity, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ inline int wave_incl_scan_i(int v) {
    v += dpp_from<0x111, 0xf>(0, v);     // row_shr:1
    v += dpp_from<0x112, 0xf>(0, v);     // row_shr:2
    v += dpp_from<0x114, 0xf>(0, v);     // row_shr:4
    v += dpp_from<0x118, 0xf>(0, v);     // row_shr:8
    v += dpp_from<0x142, 0xa>(0, v);     // row_bcast:15 into rows 1 and 3
    v += dpp_from<0x143, 0xc>(0, v);     // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ inline int wave_sum_i(int v) { return __builtin_amdgcn_readlane(wave_incl_scan_i(v), kW - 1); }

// Move `amount` units of free load from rank a to rank b (listed experts in ascending order; free: replicas above
// g_cur of j_cur and all of the experts after it; j_cur < 0: everything).  A lane past the last expert reads the last
// expert's entries (in bounds, no branch, so the LDS reads go out together) and takes no part.  Every rank q that is
// a replica of a giving expert loses what it could get from a and gains it from b: summed over the givers in
// lane q's register, then one update of its two entries.
template <typename M>
__device__ inline void move_units(Ctx<M>& c, int a, int b, int amount, int j_cur, int g_cur) {
    int remaining = amount, D = 0;
    const int q = lane();
    for (int base = (j_cur < 0 ? 0 : j_cur); base < c.n && remaining > 0; base += kW) {
        const int j = base + q;                       // >= j_cur: earlier experts are never looked at
        const bool in = j < c.n;
        const int jj = in ? j : c.n - 1;
        const M pm = (M)c.pm[jj];
        const int xa = c.x[jj * c.XS + a], xb = c.x[jj * c.XS + b];
        const M F = (j == j_cur) ? (pm & ~(((M)2 << g_cur) - (M)1)) : pm;
        const int m = (in && has(F, a) && has(F, b)) ? xa : 0;
        if (__ballot(m > 0) == 0ull) continue;        // no expert of this chunk links a to b (wave-uniform)
        const int inc = wave_incl_scan_i(m);
        const int t = max(0, min(m, remaining - (inc - m)));
        if (t > 0) {
            c.x[j * c.XS + a] = xa - t;
            c.x[j * c.XS + b] = xb + t;
        }
        u64 givers = __ballot(t > 0);
        while (givers) {
            const int src = __ffsll((long long)givers) - 1;
            givers &= givers - 1;
            const int ts = __builtin_amdgcn_readlane(t, src);
            if (has(readlane_set(F, src), q & (8 * (int)sizeof(M) - 1))) D += ts;
        }
        remaining -= min(remaining, __builtin_amdgcn_readlane(inc, kW - 1));
    }
    if (D > 0 && q < c.G) {
        const int va = q != a ? c.a(a, q) - D : 0, vb = q != b ? c.a(b, q) + D : 0;
        if (q != a) c.a(a, q) = va;
        if (q != b) c.a(b, q) = vb;
        c.in = (c.in & ~((M)1 << a) & ~((M)1 << b)) | (M)(va > 0) << a | (M)(vb > 0) << b;
    }
    c.ld += q == b ? amount : q == a ? -amount : 0;
    wave_sync();
}

// Breadth-first search from `src` over edges with A > 0.  Stops at the first level that
// holds a rank of `want` (a per-lane predicate, lane = rank).  Returns the chosen rank
// (lowest of that level) or -1; *visited_out = every rank reached; *parent_out (lane = rank) = where the search came
// from; *cap_out = the smallest capacity on the way.
template <typename M>
__device__ inline int bfs(const Ctx<M>& c, int src, bool want, M* visited_out, int* parent_out, int* cap_out) {
    const int b = lane();
    M visited = (M)1 << src, frontier = visited;
    int parent = -1, target = -1;
    while (true) {
        const M hit = c.in & frontier;                           // (lanes that are no ranks have nothing in `in`)
        const bool fresh = hit != 0 && parent < 0 && b != src;
        if (fresh) parent = first_of(hit);
        const M next = (M)__ballot(fresh);
        if (next == 0) break;
        visited |= next;
        const M good = (M)__ballot(fresh && want);
        if (good) { target = first_of(good); break; }
        frontier = next;
    }
    *visited_out = visited;
    *parent_out = parent;
    if (target < 0) return -1;
    // every reached rank reads the capacity of its own edge; the way back is then two lane reads per step
    const int edge = parent >= 0 ? c.a(parent, b) : 0;
    int cap = 0x7fffffff, cur = target;
    while (cur != src) {
        cap = min(cap, __builtin_amdgcn_readlane(edge, cur));
        cur = __builtin_amdgcn_readlane(parent, cur);
    }
    *cap_out = cap;
    return target;
}

// Moves `amount` units along the way found by bfs, last edge first (an edge's capacity depends on the units on its
// source only, and the ranks of a shortest way are distinct: the order of the edges does not matter).
template <typename M>
__device__ inline void push_path(Ctx<M>& c, int src, int target, int parent, int amount, int j_cur, int g_cur) {
    int cur = target;
    while (cur != src) {
        const int p = __builtin_amdgcn_readlane(parent, cur);
        move_units(c, p, cur, amount, j_cur, g_cur);
        cur = p;
    }
}

// From the replica masks of all experts in c.pm: the list of those with several replicas (their masks move to the
// front of c.pm), and the loads of the others on their only rank.  Returns (to every lane) whether some expert with
// load has no replica.
template <typename M>
__device__ inline bool compact(Ctx<M>& c, const int32_t* __restrict__ load) {
    const int l = lane();
    int bad = 0, n = 0;
    c.listed = 0ull;
    if (l < c.G) c.t[l] = 0;
    wave_sync();
    for (int base = 0; base < c.E; base += kW) {
        const int e = base + l;
        const u64 m = e < c.E ? c.pm[e] : 0ull;
        const int le = e < c.E ? max(load[e], 0) : 0;
        const int replicas = __popcll(m);
        if (replicas == 0 && le > 0) bad = 1;
        if (replicas == 1 && le > 0) atomicAdd(&c.t[__ffsll((long long)m) - 1], le);
        const u64 w = __ballot(replicas > 1);
        if (l == base / kW) c.listed = w;
        wave_sync();                                  // this chunk's masks are in registers
        if (replicas > 1) c.pm[n + __popcll(w & ((1ull << l) - 1ull))] = m;      // never behind what is still to be read
        n += __popcll(w);
    }
    c.n = n;
    wave_sync();
    c.single = l < c.G ? c.t[l] : 0;
    return __ballot(bad) != 0ull;
}

// the rank loads from c.t and the sets of sources from A
template <typename M>
__device__ inline void load_registers(Ctx<M>& c) {
    const int l = lane();
    wave_sync();
    c.ld = l < c.G ? c.t[l] : 0;
    c.in = 0;
    if (l < c.G)
        for (int a = 0; a < c.G; ++a) c.in |= (M)(c.A[l * c.AS + a] > 0) << a;
}

// Everything on each expert's first replica: fills x, A and the rank loads from the list and the expert loads
// (negative reads as 0) times `scale`.
template <typename M>
__device__ inline void start_on_first_replicas(Ctx<M>& c, const int32_t* __restrict__ load, int scale = 1) {
    const int l = lane();
    for (int i = l; i < c.G * c.AS; i += kW) c.A[i] = 0;
    for (int i = l; i < c.n * c.XS; i += kW) c.x[i] = 0;
    if (l < c.G) c.t[l] = c.single * scale;
    wave_sync();
    int n = 0;
    for (int base = 0; base < c.E; base += kW) {
        const u64 w = readlane_u64(c.listed, base / kW);
        if ((w >> l) & 1ull) {
            const int j = n + __popcll(w & ((1ull << l) - 1ull));
            const u64 m = c.pm[j];
            const int le = max(load[base + l], 0) * scale;
            if (le > 0) {
                const int first = __ffsll((long long)m) - 1;
                c.x[j * c.XS + first] = le;
                atomicAdd(&c.t[first], le);
                u64 others = m & ~(1ull << first);
                while (others) { int q = __ffsll((long long)others) - 1; others &= others - 1; atomicAdd(&c.a(first, q), le); }
            }
        }
        n += __popcll(w);
    }
    load_registers(c);
}

// The optimum value M* = ceil(m) of Eq. 1 for P units in all.  Start with M = ceil(P/G).  While some
// rank a exceeds M, search from a for a rank below M and push the bottleneck amount along the path.
// If the search finds none, the reached set S is closed (no expert with load in S has a replica
// outside S), so Eq. 3 gives the lower bound ceil(load(S)/|S|) > M; M jumps to it.  M only ever moves
// to lower bounds of the optimum and the loop ends with a feasible flow, hence M = M*.
template <typename M>
__device__ inline int optimum_value(Ctx<M>& c, int P) {
    const int l = lane();
    int best = (P + c.G - 1) / c.G;
    while (true) {
        const int mine = c.ld;
        const u64 over = __ballot(l < c.G && mine > best);
        if (over == 0ull) break;
        const int a = __ffsll((long long)over) - 1;
        M visited; int parent, cap;
        const int r = bfs(c, a, (l < c.G) && (mine < best), &visited, &parent, &cap);
        if (r < 0) {
            const bool in = (l < c.G) && has(visited, l & (8 * (int)sizeof(M) - 1));
            const int tot = wave_sum_i(in ? mine : 0);
            const int cnt = __popcll(visited);
            best = (tot + cnt - 1) / cnt;
            continue;
        }
        const int amount = min(min(__builtin_amdgcn_readlane(mine, a) - best, best - __builtin_amdgcn_readlane(mine, r)), cap);
        push_path(c, a, r, parent, amount, -1, 0);
    }
    return best;
}

// m of Eq. 3, the maximum density over sets of ranks, as a fraction num / den with den <= G (not
// reduced), for P units in all with P * G < 2^31.  lambda starts at P / G, the density of the set of
// all ranks, and only ever moves to the density of an actual set, so it never exceeds m.  With every
// load multiplied by den, "can all loads be placed with rank loads <= lambda" is an integer flow
// with capacity num per rank.  A search from a rank above capacity that finds no rank below it
// returns a closed set S: every expert with units in S has all its replicas in S and every other
// expert has none there, so the units in S are den * load(S), no rank of S is below capacity and one
// is above: load(S) / |S| > lambda.  lambda moves there and the flow starts again in the new scale.
// When no rank is above capacity the loads fit under lambda, so m <= lambda, hence m = lambda.
template <typename M>
__device__ inline void exact_density(Ctx<M>& c, const int32_t* __restrict__ load, int P, int* num_out, int* den_out) {
    const int l = lane();
    int num = P, den = c.G;
    while (true) {
        start_on_first_replicas(c, load, den);
        bool moved = false;
        while (true) {
            const int mine = c.ld;
            const u64 over = __ballot(l < c.G && mine > num);
            if (over == 0ull) break;
            const int a = __ffsll((long long)over) - 1;
            M visited; int parent, cap;
            const int r = bfs(c, a, (l < c.G) && (mine < num), &visited, &parent, &cap);
            if (r < 0) {
                const bool in = (l < c.G) && has(visited, l & (8 * (int)sizeof(M) - 1));
                num = wave_sum_i(in ? mine : 0) / den;
                den = __popcll(visited);
                moved = true;
                break;
            }
            push_path(c, a, r, parent,
                      min(min(__builtin_amdgcn_readlane(mine, a) - num, num - __builtin_amdgcn_readlane(mine, r)), cap), -1, 0);
        }
        if (!moved) break;
    }
    *num_out = num;
    *den_out = den;
}

// bytes of LDS behind a Ctx for E experts on G ranks, with x in rows of `xs`
__host__ __device__ inline size_t ctx_bytes(int E, int G, int xs) {
    return (((size_t)E * 8 + 15) & ~(size_t)15) + ((size_t)G * (G | 1) + (size_t)E * xs + G) * 4;
}
// row stride of x: odd where that fits into `limit` bytes
__host__ __device__ inline int x_stride(int E, int G, size_t limit) { return ctx_bytes(E, G, G | 1) <= limit ? G | 1 : G; }

// the arrays of a Ctx laid out from `smem` (16-byte aligned)
template <typename M>
__device__ inline Ctx<M> make_ctx(char* smem, int E, int G, int xs) {
    Ctx<M> c;
    c.E = E; c.G = G; c.AS = G | 1; c.XS = xs;
    c.pm = reinterpret_cast<u64*>(smem);
    c.A = reinterpret_cast<int*>(smem + (((size_t)E * 8 + 15) & ~(size_t)15));
    c.x = c.A + (size_t)G * c.AS;
    c.t = c.x + (size_t)E * xs;
    c.n = 0; c.listed = 0ull; c.single = 0; c.ld = 0; c.in = 0;
    return c;
}

}  // namespace flow
}  // namespace fine
