// Routed evaluation: every workgroup keeps one piece of a grid in LDS and
// takes the points that fall into it (types, and the plan of the pieces that
// the host checks and the kernel follows).
#pragma once

#include "pdfx_internal.h"

namespace pdfx {

// How one grid is cut: along the split axis (0: x, 1: Q^2) into pieces of at
// most `most` intervals, of which the whole axis needs `pieces` (0: no cut
// fits the LDS).
struct RoutePlan {
    int split, most, pieces;
};

// Bytes of one knot in LDS for n_u requested rows of vsize-byte values: planes
// of 16-byte nodes (16 / vsize rows each) and one narrower plane for the rest
// (FP64: 8 bytes; FP32: 4, 8 or 16).
__host__ __device__ inline int route_tail_bytes(int n_u, int vsize)
{
    const int t = n_u % (16 / vsize) * vsize;
    return t == 12 ? 16 : t;
}
__host__ __device__ inline int route_node_bytes(int n_u, int vsize)
{
    return n_u / (16 / vsize) * 16 + route_tail_bytes(n_u, vsize);
}

__host__ __device__ inline int route_round16(int b) { return (b + 15) / 16 * 16; }

// LDS bytes of the search tables of an axis part of cnt intervals: knots,
// interval constants (32 bytes each) and the axis' bucket seeds.
__host__ __device__ inline int route_axis_bytes(int cnt, int nbuckets)
{
    return route_round16((cnt + 1) * 8) + cnt * 32 + route_round16(nbuckets * 2);
}

// The fewest pieces whose knots, tables and alpha_s values (as_bytes) fit the
// LDS, cutting either axis; x when both need as many.
__host__ __device__ inline RoutePlan route_plan(int nx, int nq, int nbx, int nbq, int n_u,
                                                int vsize, int as_bytes)
{
    RoutePlan best{0, 0, 0};
    if (nx < 4 || nq < 4 || n_u < 1)
        return best;
    const int nb = route_node_bytes(n_u, vsize);
    for (int s = 0; s < 2; ++s) {
        const int n = s ? nq : nx, other = s ? nx : nq;
        const int nb_s = s ? nbq : nbx, nb_o = s ? nbx : nbq;
        const int64_t room = (int64_t)kLdsLimit - route_round16(as_bytes) -
                             route_axis_bytes(other - 1, nb_o) -
                             route_axis_bytes(0, nb_s) - 48;
        const int64_t fixed = (int64_t)3 * other * nb;
        if (room <= fixed)
            continue;
        const int64_t most = (room - fixed) / ((int64_t)other * nb + 40);
        if (most < 1)
            continue;
        const int p = most >= n - 1 ? 1 : (int)((n - 1 + most - 1) / most);
        if (best.pieces == 0 || p < best.pieces)
            best = RoutePlan{s, most >= n - 1 ? n - 1 : (int)most, p};
    }
    return best;
}

// Which intervals the pieces of a unit hold and how many workgroups sweep
// each, from a sample of the points: piece k holds intervals [cut[k], cut[k+1])
// of the split axis.  Intervals outside [cut[0], cut[pieces]) hold no sample and
// no piece.
constexpr int kRouteMaxPieces = 32;
struct RouteCut {
    int pieces;
    int cut[kRouteMaxPieces + 1];
    int width[kRouteMaxPieces];
};

// One launch: units of (member, range of points), each shared out among the
// workgroups of a team (the workgroups of one XCD by block index) as (piece,
// part of the piece's points).
struct RouteArgs {
    const MemberDev *mem;         // [n_mem] on the device, or null: `one`
    MemberDev one;
    int n_mem;
    RouteCut *cuts;               // [n_mem] on the device: where each member is cut, or null
    int longest;                  // knots of the longest axis
    int raw;                      // values are [nf][nx][nq] without a border
    int teams, team_size;
    int ranges;                   // ranges of points per member
    int n_units;                  // members * ranges
    int64_t range_pts;
    int n_u;                      // requested rows, each one output column
    int urow[kMaxReq];
    const double *x, *q;
    int q_is_q;
    int64_t n;
    void *out;                    // [n_mem][n][n_u]
    int domain_mode;
    unsigned long long *dom_count;
    const void *as_vals;          // padded alpha_s knot values, or null
    void *as_out;
};

// Which kernel takes a call.  Its load is its points times the request's flavour groups
// (11 partons: 6 in FP64, 3 in FP32).
//
// Up to kDirectMost the direct kernel, whose gathers come from the L2, then the group
// kernel, which copies a group's nodes into LDS first.  100 x 50 knots, FP64 / FP32 us,
// 11 partons: 8 thousand points 6.2 / 5.1 and 5.5 / 5.2, 16 thousand 6.8 / 5.4 and 6.3 /
// 5.7, 32 thousand 10.0 / 6.6 and 7.6 / 6.3, 100 thousand 27 / 15 and 13.3 / 8.9 (the
// double-buffered kernel 18.8 / 13.3); 2 partons: 32 thousand 5.6 / 5.7 and 5.6 / 5.5.
// Caller values are read by the direct kernel as they are and repacked for the group
// kernel: the line is their points times partons (11: 16 thousand 7.8 / 6.4 and 9.6 / 8.2,
// 32 thousand 11.8 / 8.7 and 10.7 / 8.7; 2: 100 thousand 7.4 / 7.9 and 10.5 / 8.5).
constexpr int64_t kDirectMost = 60000, kDirectMostRaw = 250000;
// From kRouteMin the routed kernel, whose placing of the pieces takes 20 us: 11 partons,
// group and routed: 400 thousand points 41 / 22.5 and 46 / 36, 600 thousand 58 / 30 and
// 55 / 43, 1 million 90 / 46 and 73 / 52, 2 million 167 / 87 and 115 / 77; 110 x 70 knots:
// 600 thousand 55 / 31 and 58 / 44, 1 million 90 / 47 and 78 / 56; 5 partons: 600 thousand
// 31 / 21 and 41 / 29, 2 million 87 / 55 and 74 / 52.
constexpr int64_t kRouteMin = 3000000;
// Calls that cannot be routed: 12 columns with a repeated pid, double-buffered and group,
// 2 million points 206 / 127 and 199 / 120, 10 million 944 / 583 and 1222 / 575; 60 x 25
// knots 2 million 169 / 109 and 183 / 116; 3 columns 10 million 488 / 297 and 282 / 153.
constexpr int64_t kGroupMostDma = 6000000;
// Grids whose group does not fit the group kernel, and requests of more flavours than it
// takes: points from which they are routed, the direct kernel (if it takes them) before.
// 190 x 75 knots: 100 thousand points 29.4 / 16.6 by the direct kernel and 47.6 / 29.1 by
// the single-buffer one, 128 thousand 38 / 30 routed and 45 / 24, 256 thousand 47 / 36 and
// 81 / 43.
constexpr int64_t kRouteMinDma = 400000, kRouteMinOther = 200000;
// The same for a set: points per member and points over all members.  101
// members in FP64 / FP32 by the class kernels and routed: 32 thousand points
// 359 / 238 us and 415 / 280, 64 thousand 724 / 450 and 558 / 368; 8 members:
// 64 thousand points 71 / 51 us and 59 / 47; 3 members: 128 thousand points 61
// / 42 us and 73 / 60.  Calls whose member blocks are not 16-byte aligned have
// only the single-slab kernel beside it (8 members, 32001 points: 74 / 41 us and
// 45 / 39; 101 members 888 / 382 and 412 / 298).
constexpr int64_t kRouteMinSet = 48000, kRouteMinSetAll = 500000;
constexpr int64_t kRouteMinSetOdd = 16000, kRouteMinSetOddAll = 200000;

hipError_t launch_route(const RouteArgs &a, bool f32, hipStream_t s);

}  // namespace pdfx
