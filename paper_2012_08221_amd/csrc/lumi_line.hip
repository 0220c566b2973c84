// Flavour-pair luminosity at one Q^2 for every point (the single-top example of
// Fig. 4): with Q^2 fixed, the sum over the four Q^2 knots of a stencil is the same
// for every point of an x interval, so a workgroup forms it once per x knot and
// parton and a parton at a point is 4 values instead of 16.
//
// The line of a parton is kept as the cubic of every interval in t, made from
// differences: three multiply-adds a parton, and no folded weights a point.  Bound by
// the vector ALU: two FP64 logarithms, bins and a division a point.  4 pairs, 1e7 points,
// sum only: 96 us FP32 (112 with the knots' values and folded weights, 568 by the
// kernel that walks the flavour groups); 4e6 points FP64 66 -> 55, 25 pairs 227 -> 180.
// The error against extended precision, by the largest knot of a stencil, is smaller
// than with folded weights (FP32 9.9e-8 -> 6.9e-8 root mean square, FP64 2.6e-16 -> 2.3e-16).
#include "lumi_internal.h"
#include "piece_axis.h"

#include <algorithm>

namespace pdfx {

namespace {

using namespace piece;

constexpr int kLineBlock = 512;

// Placement in LDS: the partons' cubics [n_row][nx - 1], the x tables, and the lines
// [n_row][nx], in FP64, that the cubics are made from.
size_t line_lds(int nx, int nbx, int n_row, bool f32)
{
    const int vs = f32 ? 4 : 8;
    return (size_t)n_row * (nx - 1) * 4 * vs + route_axis_bytes(nx - 1, nbx) + (size_t)n_row * nx * 8;
}

template <typename V>
__global__ __launch_bounds__(kLineBlock) void lumi_line_kernel(const LumiLineArgs a)
{
    constexpr bool F32 = sizeof(V) == 4;
    constexpr int C = 16 / (int)sizeof(V);   // pairs stored at once
    extern __shared__ uint4 smem4[];
    char *sm = reinterpret_cast<char *>(smem4);
    typedef V Cubic __attribute__((ext_vector_type(4)));
    Cubic *const cubic = reinterpret_cast<Cubic *>(sm);
    const int tid = threadIdx.x;
    const int nx = a.nx, nq = a.nq;

    int off = a.n_row * (nx - 1) * (int)sizeof(Cubic);
    const PieceAxis px = place_axis(sm, off, a.ax, 0, nx - 1);
    {
        const PieceAxis both[2] = {px, px};
        const AxisDev *const axes[2] = {&a.ax, &a.ax};
        load_axes<F32>(both, axes, kLineBlock);
    }
    double *const line = reinterpret_cast<double *>(sm + off);

    // Q^2: inside, clamped into the grid, or (every point outside) the first knot
    double q2 = a.q2_fixed;
    const bool q_in = q2 >= a.aq.lo && q2 <= a.aq.hi;
    if (!q_in)
        q2 = a.domain_mode == 1 ? fmin(fmax(q2, a.aq.lo), a.aq.hi) : a.aq.lo;
    double wq[4];
    const double lnq = ln(q2);
    const int cq = window4(far_weights<double>(a.aq, q2, lnq, wq), nq, wq);
    const V *const src = reinterpret_cast<const V *>(a.vals);
    for (int e = tid; e < a.n_row * nx; e += kLineBlock) {
        const int r = e / nx, i = e - r * nx;
        const V *v = src + (size_t)a.row[r] * a.flav_stride + (size_t)i * a.x_stride + cq;
        double t = wq[0] * (double)v[0];
        t = fma(wq[1], (double)v[1], t);
        t = fma(wq[2], (double)v[2], t);
        t = fma(wq[3], (double)v[3], t);
        line[e] = t;
    }
    __syncthreads();
    for (int e = tid; e < a.n_row * (nx - 1); e += kLineBlock) {
        const int r = e / (nx - 1), i = e - r * (nx - 1);
        const double *v = line + r * nx;
        const IntervalRec<double> c = a.ax.rec64[i];
        const double v0 = c.pl != 0.0 ? v[i - 1] : v[i], v1 = v[i], v2 = v[i + 1];
        const double v3 = c.pr != 0.0 ? v[i + 2] : v2, d = v2 - v1;
        // slopes at both ends, times the width
        const double s1 = fma(c.pl, v1 - v0, c.ql * d), s2 = fma(c.pr, v3 - v2, c.qr * d);
        cubic[e] = Cubic{(V)v1, (V)s1, (V)(3.0 * d - 2.0 * s1 - s2), (V)(s1 + s2 - 2.0 * d)};
        // infinite values (a caller's): the weights are below 0 at the outer two knots, so
        // this is what the sum of the products is inside the interval
        if (!(fabs(s1) + fabs(s2) < 1.0 / 0.0))
            cubic[e] = Cubic{(V)(v1 + v2 - (c.pl != 0.0 ? v0 : 0.0) - (c.pr != 0.0 ? v3 : 0.0)), V(0),
                             V(0), V(0)};
    }
    __syncthreads();

    V *const out_pair = reinterpret_cast<V *>(a.out_pair);
    V *const out_sum = reinterpret_cast<V *>(a.out_sum);
    const int n_pair = a.n_pair;
    const int64_t step = (int64_t)gridDim.x * kLineBlock;
    int64_t p = (int64_t)blockIdx.x * kLineBlock + tid;
    const int64_t n_wave = (a.n + 63) / 64 * 64;   // whole waves, for the counting
    double nx1 = load_point(a.x1, p, a.n), nx2 = load_point(a.x2, p, a.n);
    for (; p < n_wave; p += step) {
        double x1 = nx1, x2 = nx2;
        nx1 = load_point(a.x1, p + step, a.n);
        nx2 = load_point(a.x2, p + step, a.n);
        const bool nan_in = (x1 != x1) || (x2 != x2);
        bool ok = x1 >= px.lo && x1 <= px.hi && x2 >= px.lo && x2 <= px.hi && q_in;
        if (!ok) {
            if (a.domain_mode == 1 && !nan_in) {
                ok = true;
                x1 = fmin(fmax(x1, px.lo), px.hi);
                x2 = fmin(fmax(x2, px.lo), px.hi);
            } else {
                x1 = x2 = px.lo;
            }
        }
        const bool live = p < a.n;
        fwd::count_flagged(live && !ok, a.dom_count);
        const double ln1 = ln(x1), ln2 = ln(x2);
        const int i1 = piece_bin(px, x1, ln1), i2 = piece_bin(px, x2, ln2);
        auto coordinate = [&](int i, double l) {
            const double2 c = *reinterpret_cast<const double2 *>(px.cst + i * 32);   // z, 1/d
            return (V)((l - c.x) * c.y);
        };
        const V t1 = coordinate(i1, ln1), t2 = coordinate(i2, ln2);
        V inv = (V)(1.0 / (x1 * x2));
        inv = ok ? inv : fwd::quiet_nan<V>();
        auto at = [&](int row, int i, V t) {
            const Cubic c = cubic[row * (nx - 1) + i];
            return fma(fma(fma(c.w, t, c.z), t, c.y), t, c.x);
        };
        V sum = V(0), fa = V(0);
        int row_a = -1;
        for (int k0 = 0; k0 < n_pair; k0 += C) {
            V l[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                l[c] = V(0);
                if (k0 + c < n_pair) {
                    const int ia = a.ia[k0 + c], ib = a.ib[k0 + c];
                    if (ia >= 0) {
                        if (ia != row_a)
                            fa = at(ia, i1, t1);
                        row_a = ia;
                        l[c] = fa * at(ib, i2, t2) * inv;
                    }
                    sum = fma((V)a.coef[k0 + c], l[c], sum);
                }
            }
            if (out_pair && live) {
                V *dst = out_pair + p * n_pair + k0;
                if (k0 + C <= n_pair) {
                    typedef V vec __attribute__((ext_vector_type(C), aligned(sizeof(V))));
                    vec v;
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        v[c] = l[c];
                    *reinterpret_cast<vec *>(dst) = v;
                } else {
#pragma unroll
                    for (int c = 0; c < C - 1; ++c)
                        if (k0 + c < n_pair)
                            dst[c] = l[c];
                }
            }
        }
        if (out_sum && live)
            out_sum[p] = ok ? sum : fwd::quiet_nan<V>();
    }
}

}  // namespace

hipError_t launch_lumi_line(const LumiLineArgs &a, bool f32, int cus, hipStream_t s)
{
    const size_t lds = line_lds(a.nx, a.ax.nbuckets, a.n_row, f32);
    int64_t grid = (a.n + kLineBlock - 1) / kLineBlock;
    // up to 32 waves a compute unit, as many as its LDS has room for
    const int64_t most = (int64_t)cus * std::max<int64_t>(1, std::min<int64_t>(4, kLdsLimit / lds));
    if (grid > most)
        grid = most;
    if (grid < 1)
        return hipSuccess;
    auto go = [&](auto fn) -> hipError_t {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(kLineBlock), lds, s, a);
        return hipGetLastError();
    };
    return f32 ? go(lumi_line_kernel<float>) : go(lumi_line_kernel<double>);
}

bool lumi_line_fits(int nx, int nbx, int n_row, bool f32)
{
    return line_lds(nx, nbx, n_row, f32) <= kLdsLimit;
}

}  // namespace pdfx
