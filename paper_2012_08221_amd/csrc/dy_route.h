// Routed integrand kernel: arguments shared by the host runtime and dy_route.hip.
#pragma once

#include "route_internal.h"

namespace pdfx {

struct DyRouteArgs {
    AxisDev ax, aq;               // the alpha_s axis is the Q^2 axis
    int nx, nq;
    const void *vals;             // value (f, i, k) at f * flav_stride + i * x_stride + k
    size_t flav_stride;
    int x_stride;
    const void *as_vals;          // padded alpha_s knot values, precision's type
    int np;                       // quark-antiquark pairs (1 .. 5)
    int row[10];                  // grid rows: np quarks, then their antiquarks
    int most;                     // intervals a piece holds at most
    int teams, team_size;
    int64_t range_pts;            // points of a team
    const double *u1, *u2;
    int64_t n;
    double lnxmin, lnrange, s, L2;
    void *out;                    // [n] or null
    double *block_sums;           // [teams * team_size] or null
    unsigned long long *dom_count;
};

// Q^2 intervals a piece can hold, 0 if not even one fits the LDS.
int dy_route_most(int nx, int nq, int nbx, int nbq, int np, bool f32);
hipError_t launch_dy_route(const DyRouteArgs &a, bool f32, hipStream_t s);

// Points from which the integrand is routed, where the Q^2 axis makes up to 5
// pieces and where it makes more (whose extra columns then outweigh their own).
// 100 x 50 knots, FP64 / FP32, the other kernels' default shape and routed: 300
// thousand points 50 / 38 us and 50 / 41, 1 million 113 / 86 and 85 / 62, 10
// million 973 / 726 and 480 / 292.  180 x 27 (FP64: 8 pieces): 1 million points
// 110 and 119 us, 10 million 965 and 773.
constexpr int64_t kDyRouteMin = 400000, kDyRouteMinMany = 2000000;

}  // namespace pdfx
