// Algorithm 1 (Section 4.2) as positions in queues, shared by the kernels that prepare it and the one that reads it.
//
// The local pass gives min(input, x) to the own rank.  What is left meets in ascending order on both sides: the waiting
// tokens of an expert's sources are one queue, the free loads of its replicas another, and they are paired head to
// head.  So all that Algorithm 1 hands out is in the prefix sums of the two queues: a token's position in the
// first is its position in the second, and where that lies is its replica.  No table of transfers per (source, replica)
// is needed.  (It was: [E][G][G] twice, 2 MB for 256 experts on 32 ranks, and every pair walked its row of it.)
//
// With nodes (Appendix A.1's routing order: same GPU, same node, then any GPU; rpn consecutive ranks form a node, rpn <= 1:
// no nodes) every node has such a pair of queues of its own first, and what lies beyond the other queue's end goes on
// into the queues over all ranks.
#pragma once

#include "flow_wave.h"

namespace fine {

// int32 [E][G] each: tokens of lower sources waiting for the pass over all ranks; free loads of the replicas up to and
// including this one; the same inside a node
struct RouteTables {
    int32_t *wait, *room_end;
    int32_t *node_wait, *node_room_end;
};

__device__ inline int clamp_to(int v, int hi) { return min(max(v, 0), hi); }

// one wave per expert e, lane = rank: its tokens in_g and its replica load x_g (0 past the last rank)
__device__ inline void write_route(const RouteTables& t, int e, int G, int rpn, int locality, int in_g, int x_g) {
    const int lane = threadIdx.x & 63;
    const int loc = locality ? min(in_g, x_g) : 0;
    int ri = in_g - loc, rx = x_g - loc;
    if (rpn > 1) {
        const int first = (lane / rpn) * rpn, last = min(first + rpn, 64) - 1;
        const int sI = flow::wave_incl_scan_i(ri), sX = flow::wave_incl_scan_i(rx);
        const int bI = __shfl(sI - ri, first, 64), bX = __shfl(sX - rx, first, 64);
        const int tI = __shfl(sI, last, 64) - bI, tX = __shfl(sX, last, 64) - bX;      // the node's queues are this long
        const int nI = sI - ri - bI, nX = sX - rx - bX;
        if (lane < G) {
            t.node_wait[(size_t)e * G + lane] = nI;
            t.node_room_end[(size_t)e * G + lane] = nX + rx;
        }
        ri -= clamp_to(tX - nI, ri);
        rx -= clamp_to(tI - nX, rx);
    }
    const int I = flow::wave_incl_scan_i(ri), X = flow::wave_incl_scan_i(rx);
    if (lane < G) {
        t.wait[(size_t)e * G + lane] = I - ri;
        t.room_end[(size_t)e * G + lane] = X;
    }
}

// how many entries of the ascending row [0, n) are <= p.  All of them are read: independent loads take one round trip, a
// binary search one per step (G = 32: 6.2 us for the kernel, 9.1 when it walked its transfers one by one).
__device__ inline int count_le(const int32_t* __restrict__ row, int n, int p) {
    int c = 0;
    if ((((uintptr_t)row | (uintptr_t)(n * 4)) & 15u) == 0) {
        for (int h = 0; h < n; h += 16) {
            int4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const int4*>(row + min(h + 4 * i, n - 4));
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (h + 4 * i < n) c += (v[i].x <= p) + (v[i].y <= p) + (v[i].z <= p) + (v[i].w <= p);
        }
    } else {
        for (int h = 0; h < n; h += 8) {
            int v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = row[min(h + i, n - 1)];
#pragma unroll
            for (int i = 0; i < 8; ++i) c += h + i < n && v[i] <= p;
        }
    }
    return c;
}

// Destination (-1: no schedule exists) of the r-th token of (expert, source g) and its place in the destination's segment;
// in, x and the tables: the expert's rows
__device__ inline int route_token(const RouteTables& t, const int32_t* __restrict__ in, const int32_t* __restrict__ x, size_t row0,
                                  int G, int rpn, int locality, int g, int r, int* place) {
    const int32_t *wait = t.wait + row0, *room_end = t.room_end + row0;
    const int loc = locality ? min(in[g], x[g]) : 0;
    const bool nodes = rpn > 1;
    const int32_t *nw = t.node_wait + row0, *nre = t.node_room_end + row0;
    auto local_of = [&](int h) { return locality ? min(in[h], x[h]) : 0; };
    auto node_of = [&](int h) { return h / rpn; };
    auto node_end = [&](int h) { return min((node_of(h) + 1) * rpn, G) - 1; };
    // the units of replica h in the node's queues: those that its node's tokens fill, and where they begin
    auto node_begin = [&](int h) { return h % rpn ? nre[h - 1] : 0; };
    auto node_used = [&](int h) {
        const int end = node_end(h), tI = nw[end] + in[end] - local_of(end);
        return clamp_to(tI - node_begin(h), nre[h] - node_begin(h));
    };
    const int my_wait = wait[g];
    // units of replica h taken in the pass over all ranks by sources before g
    auto taken_before = [&](int h) {
        const int begin = h ? room_end[h - 1] : 0;
        return clamp_to(my_wait - begin, room_end[h] - begin);
    };
    if (r < loc) {
        *place = r + taken_before(g) + (nodes ? clamp_to(nw[g] - node_begin(g), node_used(g)) : 0);
        return g;
    }
    r -= loc;
    if (nodes) {
        const int n0 = node_of(g) * rpn, nn = node_end(g) + 1 - n0;
        const int inside = clamp_to(nre[n0 + nn - 1] - nw[g], in[g] - loc);      // of g's tokens
        if (r < inside) {
            const int p = nw[g] + r, h = n0 + count_le(nre + n0, nn, p);
            *place = p - node_begin(h) + taken_before(h) + (h < g ? local_of(h) : 0);
            return h;
        }
        r -= inside;
    }
    const int p = my_wait + r, h = count_le(room_end, G, p);
    if (h >= G) return -1;
    *place = p - (h ? room_end[h - 1] : 0) + (h < g ? local_of(h) : 0);
    if (nodes && node_of(h) <= node_of(g)) *place += node_of(h) < node_of(g) ? node_used(h) : clamp_to(nw[g] - node_begin(h), node_used(h));
    return h;
}

}  // namespace fine
