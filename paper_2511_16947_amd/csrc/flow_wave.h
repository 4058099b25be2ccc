// One-wavefront integer flows on the placement graph (Section 5.1's graph abstraction): ranks are
// vertices, an expert with units on rank a and a replica on rank b lets load move from a to b.  With G <= 64 a vertex
// set is a 64-bit mask and a breadth-first search is a few ballots.  Shared by the scheduler's replica-load solver and by
// the placement scoring for more than 16 ranks.
#pragma once

#include <type_traits>

#include "common.h"

namespace fine {
namespace flow {

constexpr int kW = 64;
typedef unsigned long long u64;

// Only experts with several replicas can move: they are kept in a compact list, in ascending order (256 experts
// with 320 replicas: at most 64 of them).
// PM: as the replica masks are stored.
template <typename PM = u64>
struct Problem {
    int* x;        // [n][XS] units of listed expert j on every rank
    PM* pm;        // [n] replica masks of the listed experts (before compact(): of all experts)
    int* t;        // [G] scratch
    int* A;        // long lists: [G][G | 1] sums of the edges
    int E, G;
    int XS;        // row stride (odd where it fits, so that a column's entries fall into different banks)
    int n;         // listed experts
    u64 listed;    // lane i: which of the experts 64 i .. 64 i + 63 are listed
    int single;    // lane = rank: load of the experts whose only replica is here
};

__device__ inline int lane() { return threadIdx.x & (kW - 1); }
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

// What a search needs, in the registers of the ranks' lanes: sets of ranks (M: 32 bits where that is enough; the search is a
// chain of instructions of one wavefront, and 64-bit shifts and selects are several each).
template <typename M, typename PM>
struct Ranks : Problem<PM> {
    int ld;                      // lane = rank: its load
    M me;                        // this rank as a set (no rank: the empty set)
    M in;                        // the ranks from which units may move here

    __device__ inline Ranks(const Problem<PM>& p) : Problem<PM>(p) {}
    // loads from c.t, no edges
    __device__ inline void load_ranks() {
        const int l = lane();
        wave_sync();
        me = l < this->G ? (M)1 << (l & (8 * (int)sizeof(M) - 1)) : (M)0;
        ld = l < this->G ? this->t[l] : 0;
        in = 0;
    }
    // Breadth-first search from `src`.  Stops at the first level that holds a rank of `want`.  The sets of ranks are scalar;
    // what the way back needs is one set per level.
    struct Way {
        int src, target, levels;     // target: lowest rank of `want` on the first level that has one, or -1
        M visited;                   // every rank reached
        M trail;                     // lane = level: the ranks first reached there
    };
    __device__ inline Way bfs(int src, M want) const {
        const int b = lane();
        Way w{src, -1, 0, (M)1 << src, 0};
        M level = w.visited;
        while (true) {
            if (b == w.levels) w.trail = level;
            level = (M)__ballot((in & level) != 0) & ~w.visited;      // (lanes that are no ranks have nothing in `in`)
            if (level == 0) break;
            w.visited |= level;
            const M good = level & want;
            if (good) { w.target = first_of(good); break; }
            ++w.levels;
        }
        return w;
    }
    // where the search came to `rank` from, on level `level` (lowest such rank)
    __device__ inline int before(const Way& w, int rank, int level) const {
        return first_of(readlane_set(in, rank) & readlane_set(w.trail, level));
    }
};

// Short lists: a move works on sets of listed experts (NW words of 64) in the registers of the ranks' lanes.  An edge from a
// to b exists while some free expert has units on a and a free replica on b, i.e. while units_a and free_b meet; how much
// may move along it is added up from x where it is used.  (Keeping the edges' sums, or each rank's set of neighbours as a
// union over its experts, costs every move and every variable that stops being free a chain of updates or of wave-wide
// reductions; here they are a few instructions per word.)
template <typename M, int NW, typename PM = u64>
struct Flow : Ranks<M, PM> {
    using Ranks<M, PM>::me;
    using Ranks<M, PM>::in;
    using Ranks<M, PM>::ld;
    u64 free[NW];                // experts that have a free replica here
    u64 units[NW];               // those of them that have units on it

    __device__ inline Flow(const Problem<PM>& p) : Ranks<M, PM>(p) {}
    // whether free experts of `set` (scalar words) have a replica on the lane's rank
    __device__ inline bool meets_free(const u64 (&set)[NW]) const {
        u64 v = 0ull;
#pragma unroll
        for (int w = 0; w < NW; ++w) v |= set[w] & free[w];
        return v != 0ull;
    }
    __device__ inline void read_units(int a, u64 (&set)[NW]) const {
#pragma unroll
        for (int w = 0; w < NW; ++w) set[w] = readlane_u64(units[w], a);
    }
    // the edges out of rank a, whose units are those of `set`
    __device__ inline void set_out(int a, const u64 (&set)[NW]) {
        const M bit = (M)1 << a;
        const bool edge = meets_free(set) && (me & bit) == 0;
        in = (in & ~bit) | (edge ? bit : (M)0);
    }
    // expert j has free units on the lane's rank
    __device__ inline bool has_units(int j) const {
        bool v = false;
#pragma unroll
        for (int w = 0; w < NW; ++w) v = v || (NW == 1 || w == j >> 6) && ((units[w] >> (j & 63)) & 1ull);
        return v;
    }
    // how many (here: has_units)
    __device__ inline int units_of(int j, bool here) const { return here ? this->x[j * this->XS + lane()] : 0; }
    // the free replicas of expert j, whose turn it is
    __device__ inline M begin(int j) const {
        bool v = false;
#pragma unroll
        for (int w = 0; w < NW; ++w) v = v || (NW == 1 || w == j >> 6) && ((free[w] >> (j & 63)) & 1ull);
        return (M)__ballot(v);
    }
    // expert j has no units left on the lane's rank, where `here`
    __device__ inline void clear_units(int j, bool here) {
#pragma unroll
        for (int w = 0; w < NW; ++w)
            if (here && (NW == 1 || w == j >> 6)) units[w] &= ~(1ull << (j & 63));
    }
    // replica (j, g) stops being free: its units can no longer move, nor others of j to it
    __device__ inline void fix(int j, int g) {
        const bool here = lane() == g;
        clear_units(j, here);
        u64 fg[NW], ug[NW];
        read_units(g, ug);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if (here && (NW == 1 || w == j >> 6)) free[w] &= ~(1ull << (j & 63));
            fg[w] = readlane_u64(free[w], g);
        }
        set_out(g, ug);
        u64 v = 0ull;
#pragma unroll
        for (int w = 0; w < NW; ++w) v |= units[w] & fg[w];
        const M from = (M)__ballot(v != 0ull) & ~((M)1 << g);
        if (here) in = from;
    }
    // the lane's rank has given `given` of its `had` units of expert j
    __device__ inline void gave(int j, int given, int had) {
        const bool none_left = given > 0 && given == had;
        clear_units(j, none_left);
        M gone = (M)__ballot(none_left);
        while (gone) {
            const int a = first_of(gone);
            gone &= gone - 1;
            u64 set[NW];
            read_units(a, set);
            set_out(a, set);
        }
    }
    // the registers from c.t (loads), the masks and x: everything free
    __device__ inline void load_registers() {
        const int l = lane();
        this->load_ranks();
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            free[w] = units[w] = 0ull;
            if (64 * w >= this->n) continue;
            const int j = min(64 * w + l, this->n - 1);      // lane = expert
            const M pm = 64 * w + l < this->n ? (M)this->pm[j] : (M)0;
#pragma unroll 8
            for (int a = 0; a < this->G; ++a) {
                const bool on = has(pm, a);
                const u64 f = __ballot(on), u = __ballot(on && this->x[j * this->XS + a] > 0);
                if (l == a) {
                    free[w] = f;
                    units[w] = u;
                }
            }
        }
        for (int a = 0; a < this->G; ++a) {
            u64 set[NW];
            read_units(a, set);
            set_out(a, set);
        }
    }
    // Moves up to `amount` units of free load from rank a to rank b (listed experts in ascending order) and returns how
    // many there were.
    __device__ inline int move_units(int a, int b, int amount) {
        const int l = lane();
        int remaining = amount;
        u64 ua[NW], ub[NW], lost = 0ull, gained = 0ull;
        read_units(a, ua);
        read_units(b, ub);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const u64 may = ua[w] & readlane_u64(free[w], b);
            if (may == 0ull || remaining == 0) continue;
            const bool on = (may >> l) & 1ull;
            int* row = this->x + min(64 * w + l, this->n - 1) * this->XS;
            const int xa = row[a], xb = row[b];
            int t, had;                              // what the lane's expert gives; what all of them have
            if ((may & (may - 1)) == 0ull) {         // one expert, as most edges have: no scan
                had = __builtin_amdgcn_readlane(xa, __builtin_ctzll(may));
                t = on ? min(had, remaining) : 0;
            } else {
                const int m = on ? xa : 0, inc = wave_incl_scan_i(m);
                had = __builtin_amdgcn_readlane(inc, kW - 1);
                t = max(0, min(m, remaining - (inc - m)));
            }
            if (t > 0) {
                row[a] = xa - t;
                row[b] = xb + t;
            }
            const u64 some = __ballot(t > 0), all = some & __ballot(t == xa);
            lost |= all;
            gained |= some & ~ub[w];
            ua[w] &= ~all;
            ub[w] |= some;
            if (l == a) units[w] = ua[w];
            if (l == b) units[w] = ub[w];
            remaining -= min(remaining, had);
        }
        if (lost) set_out(a, ua);
        if (gained) set_out(b, ub);
        const int moved = amount - remaining;
        ld += l == b ? moved : l == a ? -moved : 0;
        wave_sync();
        return moved;
    }
    // how many free units of rank a may move to rank b
    __device__ inline int edge_capacity(int a, int b) const {
        const int l = lane();
        int sum = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const u64 may = readlane_u64(units[w], a) & readlane_u64(free[w], b);
            if (may == 0ull) continue;
            const int xa = this->x[min(64 * w + l, this->n - 1) * this->XS + a];
            sum += (may >> l) & 1ull ? xa : 0;
        }
        return wave_sum_i(sum);
    }
};

// Long lists: the sums of the edges instead of sets, A[b][a] = units that may move from a to b, kept up to date.  A move
// looks through the list, 64 experts at a time, and then changes the entries of every rank that is a replica of a giving
// expert, summed over the givers in that rank's lane.  What a variable that stops being free costs does not depend on the
// length of the list.
template <typename M, typename PM>
struct Flow<M, 0, PM> : Ranks<M, PM> {
    using Ranks<M, PM>::me;
    using Ranks<M, PM>::in;
    using Ranks<M, PM>::ld;
    int cur = -1;                // the expert whose turn it is: those before it can no longer move
    M later = 0;                 // its free replicas
    int mine = 0;                // its units on the lane's

    __device__ inline Flow(const Problem<PM>& p) : Ranks<M, PM>(p) {}
    __device__ inline int& sum(int a, int b) const { return this->A[b * (this->G | 1) + a]; }
    __device__ inline M begin(int j) {
        cur = j;
        later = readlane_set((M)this->pm[j], 0);
        return later;
    }
    __device__ inline bool has_units(int j) {
        mine = 0;
        if ((later & me) != 0) mine = this->x[j * this->XS + lane()];
        return mine > 0;
    }
    __device__ inline int units_of(int, bool) const { return mine; }
    __device__ inline void fix(int j, int g) {
        const int l = lane(), *row = this->x + j * this->XS;
        later &= ~((M)1 << g);
        int back = 0;
        if ((later & me) != 0) {      // lane = one of the other replicas
            const int to_me = sum(g, l) - row[g];
            back = sum(l, g) - row[l];
            sum(g, l) = to_me;
            sum(l, g) = back;
            in = (in & ~((M)1 << g)) | (M)(to_me > 0) << g;
        }
        const M still = (M)__ballot(back > 0);
        if (l == g) in = (in & ~later) | still;
        wave_sync();
    }
    __device__ inline void gave(int, int given, int) {
        const int q = lane();
        M givers = (M)__ballot(given > 0);
        while (givers) {
            const int a = first_of(givers);
            givers &= givers - 1;
            const int t = __builtin_amdgcn_readlane(given, a);
            if (q != a && (later & me) != 0) {
                const int v = sum(a, q) - t;
                sum(a, q) = v;
                in = (in & ~((M)1 << a)) | (M)(v > 0) << a;
            }
        }
        wave_sync();
    }
    __device__ inline void load_registers() {
        const int l = lane();
        this->load_ranks();
        for (int i = l; i < this->G * (this->G | 1); i += kW) this->A[i] = 0;
        wave_sync();
        for (int j = l; j < this->n; j += kW) {
            const M m = (M)this->pm[j];
            for (M r = m; r; r &= r - 1) {
                const int a = first_of(r), units = this->x[j * this->XS + a];
                if (units > 0)
                    for (M o = m & ~((M)1 << a); o; o &= o - 1) atomicAdd(&sum(a, first_of(o)), units);
            }
        }
        wave_sync();
        if (l < this->G)
            for (int a = 0; a < this->G; ++a) in |= (M)(sum(a, l) > 0) << a;
    }
    __device__ inline int move_units(int a, int b, int amount) {
        const int q = lane();
        int remaining = amount, D = 0;
        for (int base = max(cur, 0); base < this->n && remaining > 0; base += kW) {
            // (a lane past the last expert reads the last one's entries and takes no part: the reads go out together)
            const int j = base + q, jj = min(j, this->n - 1);
            const M pm = (M)this->pm[jj];
            int* row = this->x + jj * this->XS;
            const int xa = row[a], xb = row[b];
            const M F = j == cur ? later : pm;
            const int m = j < this->n && has(F, a) && has(F, b) ? xa : 0;
            if (__ballot(m > 0) == 0ull) continue;
            const int inc = wave_incl_scan_i(m), t = max(0, min(m, remaining - (inc - m)));
            if (t > 0) {
                row[a] = xa - t;
                row[b] = xb + t;
            }
            u64 givers = __ballot(t > 0);
            while (givers) {
                const int src = first_of(givers);
                givers &= givers - 1;
                const int ts = __builtin_amdgcn_readlane(t, src);
                if ((readlane_set(F, src) & me) != 0) D += ts;
            }
            remaining -= min(remaining, __builtin_amdgcn_readlane(inc, kW - 1));
        }
        if (D > 0) {
            const int va = q != a ? sum(a, q) - D : 0, vb = q != b ? sum(b, q) + D : 0;
            if (q != a) sum(a, q) = va;
            if (q != b) sum(b, q) = vb;
            in = (in & ~((M)1 << a) & ~((M)1 << b)) | (M)(va > 0) << a | (M)(vb > 0) << b;
        }
        const int moved = amount - remaining;
        ld += q == b ? moved : q == a ? -moved : 0;
        wave_sync();
        return moved;
    }
    __device__ inline int edge_capacity(int a, int b) const { return __builtin_amdgcn_readfirstlane(sum(a, b)); }
};

// smallest capacity on the way
template <typename F, typename W>
__device__ inline int way_capacity(const F& c, const W& w) {
    int cap = 0x7fffffff, cur = w.target;
    for (int level = w.levels; level >= 0; --level) {
        const int p = c.before(w, cur, level);
        cap = min(cap, c.edge_capacity(p, cur));
        cur = p;
    }
    return cap;
}
// Moves up to `amount` units along the way, last edge first, and returns how many left its source (at least one).  An
// edge takes what the edge after it took, or less if it has not as many: a rank on the way never ends with more than
// it had.  (The edges not yet used are as the search found them: the ranks of a shortest way are distinct.)
template <typename F, typename W>
__device__ inline int push(F& c, const W& w, int amount) {
    int cur = w.target;
    for (int level = w.levels; level >= 0; --level) {
        const int p = c.before(w, cur, level);
        amount = c.move_units(p, cur, amount);
        cur = p;
    }
    return amount;
}

// Calls f(number of words; 0: sums of the edges) with what suits n listed experts; MAXW = words_for(E).  Every word costs every
// step of the sets, while the sums hardly feel the length.  Whole scheduler, 4096 tokens x 8, us (geometric mean of six
// placements; started from first replicas / warm), sets of 4 or 16 words : sums.  On 8 ranks 129 experts of two replicas 267 :
// 265 / 155 : 136, of four 357 : 328 / 259 : 224; 256 of two 398 : 359 / 256 : 211, of eight 1078 : 968 / 1007 : 847; 512 of four
// 3116 : 1170 / 2382 : 802; on 32 ranks 256 of four 1253 : 1224 / 794 : 719; 1024 of two 5619 : 3083 / 3095 : 1342.  The sets
// stay ahead only from first replicas with two each on many ranks (256 on 32 697 : 748 / 453 : 437, on 64 749 : 837 / 516 : 514).
constexpr int kMaxWords = 2;
constexpr int words_for(int E) { return E <= 64 ? 1 : E <= 64 * kMaxWords ? kMaxWords : 0; }
template <int MAXW, typename F>
__device__ inline void with_words(int n, F f) {
    if constexpr (MAXW == 0)
        if (n > 64 * kMaxWords) { f(std::integral_constant<int, 0>{}); return; }
    if constexpr (MAXW != 1)
        if (n > 64) { f(std::integral_constant<int, kMaxWords>{}); return; }
    f(std::integral_constant<int, 1>{});
}
// pick(words_for(E), a value of the type for sets of ranks), on the host
template <typename F>
inline auto by_size(int E, int G, F pick) {
    auto with = [&](auto m) {
        switch (words_for(E)) {
            case 1: return pick(std::integral_constant<int, 1>{}, m);
            case kMaxWords: return pick(std::integral_constant<int, kMaxWords>{}, m);
            default: return pick(std::integral_constant<int, 0>{}, m);
        }
    };
    return G <= 32 ? with(uint32_t{}) : with(u64{});
}

// From the replica masks of all experts in c.pm: the list of those with several replicas (their masks move to the
// front of c.pm), and the loads of the others on their only rank.  Returns (to every lane) whether some expert with
// load has no replica.
template <typename PM>
__device__ inline bool compact(Problem<PM>& c, const int32_t* __restrict__ load) {
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
        if (replicas > 1) c.pm[n + __popcll(w & ((1ull << l) - 1ull))] = (PM)m;      // never behind what is still to be read
        n += __popcll(w);
    }
    c.n = n;
    wave_sync();
    c.single = l < c.G ? c.t[l] : 0;
    return __ballot(bad) != 0ull;
}

// Everything on each expert's first replica: fills x and the rank loads from the list and the expert loads
// (negative reads as 0) times `scale`.
template <typename M, int NW, typename PM>
__device__ inline void start_on_first_replicas(Flow<M, NW, PM>& c, const int32_t* __restrict__ load, int scale = 1) {
    const int l = lane();
    for (int i = l; i < c.n * c.XS; i += kW) c.x[i] = 0;
    if (l < c.G) c.t[l] = c.single * scale;
    wave_sync();
    int n = 0;
    for (int base = 0; base < c.E; base += kW) {
        const u64 w = readlane_u64(c.listed, base / kW);
        if ((w >> l) & 1ull) {
            const int j = n + __popcll(w & ((1ull << l) - 1ull));
            const int le = max(load[base + l], 0) * scale, first = first_of((M)c.pm[j]);
            c.x[j * c.XS + first] = le;
            if (le > 0) atomicAdd(&c.t[first], le);
        }
        n += __popcll(w);
    }
    c.load_registers();
}

// The optimum value M* = ceil(m) of Eq. 1 for P units in all.  Start with M = ceil(P/G).  While some
// rank a exceeds M, search from a for a rank below M and push along the path what it takes.
// If the search finds none, the reached set S is closed (no expert with load in S has a replica
// outside S), so Eq. 3 gives the lower bound ceil(load(S)/|S|) > M; M jumps to it.  M only ever moves
// to lower bounds of the optimum and the loop ends with a feasible flow, hence M = M*.
template <typename M, int NW, typename PM>
__device__ inline int optimum_value(Flow<M, NW, PM>& c, int P) {
    const int l = lane();
    int best = (P + c.G - 1) / c.G;
    while (true) {
        const int mine = c.ld;
        const u64 over = __ballot(l < c.G && mine > best);
        if (over == 0ull) break;
        const int a = __ffsll((long long)over) - 1;
        const auto way = c.bfs(a, (M)__ballot(l < c.G && mine < best));
        if (way.target < 0) {
            const int tot = wave_sum_i((way.visited & c.me) != 0 ? mine : 0);
            const int cnt = __popcll(way.visited);
            best = (tot + cnt - 1) / cnt;
            continue;
        }
        const int amount = min(__builtin_amdgcn_readlane(mine, a) - best, best - __builtin_amdgcn_readlane(mine, way.target));
        push(c, way, amount);
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
template <typename M, int NW, typename PM>
__device__ inline void exact_density(Flow<M, NW, PM>& c, const int32_t* __restrict__ load, int P, int* num_out, int* den_out) {
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
            const auto way = c.bfs(a, (M)__ballot(l < c.G && mine < num));
            if (way.target < 0) {
                num = wave_sum_i((way.visited & c.me) != 0 ? mine : 0) / den;
                den = __popcll(way.visited);
                moved = true;
                break;
            }
            push(c, way, min(__builtin_amdgcn_readlane(mine, a) - num, num - __builtin_amdgcn_readlane(mine, way.target)));
        }
        if (!moved) break;
    }
    *num_out = num;
    *den_out = den;
}

// bytes of LDS behind a Problem for E experts on G ranks, with x in rows of `xs`
__host__ __device__ inline size_t edge_bytes(int E, int G) { return words_for(E) == 0 ? (size_t)G * (G | 1) * 4 : 0; }
__host__ __device__ inline size_t ctx_bytes(int E, int G, int xs) {
    return (((size_t)E * 8 + 15) & ~(size_t)15) + edge_bytes(E, G) + ((size_t)E * xs + G) * 4;
}
// The contract's limit on (E, G): with the edges' sums, whether they are kept or not.
inline bool size_allowed(int E, int G, size_t limit) {
    return (((size_t)E * 8 + 15) & ~(size_t)15) + ((size_t)G * (G | 1) + (size_t)E * G + G) * 4 <= limit;
}
// row stride of x: odd where that fits into `limit` bytes
__host__ __device__ inline int x_stride(int E, int G, size_t limit) { return ctx_bytes(E, G, G | 1) <= limit ? G | 1 : G; }

// the arrays of a Problem laid out from `smem` (16-byte aligned)
__device__ inline Problem<> make_problem(char* smem, int E, int G, int xs) {
    Problem<> c;
    c.E = E; c.G = G; c.XS = xs;
    c.pm = reinterpret_cast<u64*>(smem);
    c.A = reinterpret_cast<int*>(smem + (((size_t)E * 8 + 15) & ~(size_t)15));
    c.x = c.A + edge_bytes(E, G) / 4;
    c.t = c.x + (size_t)E * xs;
    c.n = 0; c.listed = 0ull; c.single = 0;
    return c;
}

}  // namespace flow
}  // namespace fine
