// Forward kernels for calls below the routed kernel's: the direct kernel (small calls,
// without the grid in LDS) and the group kernel (medium ones, a flavour group in LDS).
//
// A call of a few thousand points is latency: the kernels that bring the grid into
// LDS copy 160 KB per workgroup and walk the flavour groups one after another.
// Here a workgroup takes 64 points and has one wave per flavour group: every wave
// locates the 64 points (search tables in LDS, loaded while the coordinates
// arrive), gathers its group's 16 nodes of 16 bytes a point out of the L2, all at
// once, and stores its columns.  Same bins, weights and order of sums as the
// other forward kernels, so the same bits.
//
// Bound by its chain of memory latencies up to some 16 thousand points (1000
// points, 11 partons and alpha_s on 100 x 50 knots: 16.9 -> 6.2 us FP64 and 12.4 ->
// 5.6 us FP32 against the double-buffered kernel; 190 x 75 knots 42 -> 6.5 and 25 ->
// 5.8 us), by the location done once per group and the gathers beyond.  Having a
// quad of lanes read one point's four neighbouring nodes together and exchange
// them touches a quarter of the lines and was slower (32 thousand points FP64:
// 9.6 -> 11.8 us).
#include "piece_axis.h"
#include "xfx_dma_impl.h"

#include <algorithm>

namespace pdfx {

namespace {

using namespace piece;

// The columns of group `stage` at point p (live: of the call), and alpha_s and the zero
// columns with group 0.  RAW: caller values [nf][nx][nq] instead of the bordered group
// nodes `group`.
template <typename V, bool AS, bool RAW>
__device__ __forceinline__ void group_columns(const XfxArgs &a, const PieceAxis &px,
                                              const PieceAxis &pq, const uint4 *group, int stage,
                                              int64_t p, bool live, double xv, double qv)
{
    constexpr bool F32 = sizeof(V) == 4;
    constexpr int G = 16 / (int)sizeof(V);
    if (a.q_is_q)
        qv = qv * qv;
    const bool x_in = xv >= px.lo && xv <= px.hi;   // false for NaN
    const bool q_in = qv >= pq.lo && qv <= pq.hi;
    bool ok = x_in && q_in, q_ok = true;
    if (!ok) {
        const bool x_nan = xv != xv, q_nan = qv != qv;
        if (a.domain_mode == 1) {
            ok = !x_nan && !q_nan;
            q_ok = !q_nan;
            xv = x_nan ? px.lo : fmin(fmax(xv, px.lo), px.hi);
            qv = q_nan ? pq.lo : fmin(fmax(qv, pq.lo), pq.hi);
        } else {
            q_ok = q_in;
            xv = x_in ? xv : px.lo;
            qv = q_in ? qv : pq.lo;
        }
    }
    if (stage == 0) {
        fwd::count_flagged(live && !ok, a.dom_count);
        if constexpr (AS)
            fwd::count_flagged(live && !q_ok, a.dom_count);
    }
    const double lnx = ln(xv), lnq = ln(qv);
    V wx[4], wq[4];
    const int ix = piece_bin(px, xv, lnx), kq = piece_bin(pq, qv, lnq);
    piece_weights<V>(px, ix, lnx, wx);
    piece_weights<V>(pq, kq, lnq, wq);
    V *const row = reinterpret_cast<V *>(a.out) + p * a.n_req;
    if (AS && stage == 0) {
        const V *av = reinterpret_cast<const V *>(a.as_vals) + kq;   // padded by one knot
        V s = wq[0] * av[0];
        s = fma(wq[1], av[1], s);
        s = fma(wq[2], av[2], s);
        s = fma(wq[3], av[3], s);
        if (live)
            reinterpret_cast<V *>(a.as_out)[p] = q_ok ? s : fwd::quiet_nan<V>();
    }
    if (stage == 0 && live)
        for (int z = 0; z < a.n_zero; ++z)
            row[a.zcols[z]] = V(0);
    if (stage >= a.n_stage)
        return;
    // a point outside the grid: NaN weights make all its values NaN
#pragma unroll
    for (int k = 0; k < 4; ++k)
        wx[k] = ok ? wx[k] : fwd::quiet_nan<V>();

    V acc[G];
    if constexpr (RAW) {
        const int sx = window4(ix, a.nx, wx), sq = window4(kq, a.nq, wq);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int r = a.sgrp[stage] * G + g;
            const V *v = reinterpret_cast<const V *>(a.vals) +
                         ((size_t)(r < a.nf ? r : a.nf - 1) * a.nx + sx) * a.nq + sq;
#pragma unroll
            for (int jx = 0; jx < 4; ++jx, v += a.nq) {
                V t = wq[0] * v[0];
                t = fma(wq[1], v[1], t);
                t = fma(wq[2], v[2], t);
                t = fma(wq[3], v[3], t);
                acc[g] = (jx == 0) ? wx[0] * t : fma(wx[jx], t, acc[g]);
            }
        }
    } else {
        const int nqp = a.nq + 2;
        const uint4 *nodes = group + ix * nqp + kq;
        uint4 d[4][4];
#pragma unroll
        for (int jx = 0; jx < 4; ++jx)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                d[jx][k] = nodes[jx * nqp + k];
#pragma unroll
        for (int jx = 0; jx < 4; ++jx) {
            V t[G];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                V v[G];
                __builtin_memcpy(v, &d[jx][k], 16);
#pragma unroll
                for (int g = 0; g < G; ++g)
                    t[g] = (k == 0) ? wq[0] * v[g] : fma(wq[k], v[g], t[g]);
            }
#pragma unroll
            for (int g = 0; g < G; ++g)
                acc[g] = (jx == 0) ? wx[0] * t[g] : fma(wx[jx], t[g], acc[g]);
        }
    }
    if (!live)
        return;
    const int c0 = a.slot_col[stage * G];
    bool side_by_side = c0 >= 0 && a.n_dup == 0;
#pragma unroll
    for (int g = 1; g < G; ++g)
        side_by_side = side_by_side && a.slot_col[stage * G + g] == c0 + g;
    // one store a lane; FP64 caller values are faster without (32 thousand points
    // 14.8 against 12.1 us)
    if ((F32 || !RAW) && side_by_side) {
        typedef V vec __attribute__((ext_vector_type(G), aligned(4)));
        vec v;
#pragma unroll
        for (int g = 0; g < G; ++g)
            v[g] = acc[g];
        *reinterpret_cast<vec *>(row + c0) = v;
        return;
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int c = a.slot_col[stage * G + g];
        if (c < 0)
            continue;
        row[c] = acc[g];
        for (int d = 0; d < a.n_dup; ++d)
            if (a.dup_src[d] == c)
                row[a.dup_dst[d]] = acc[g];
    }
}

template <typename V, bool AS, bool RAW>
__global__ __launch_bounds__(64 * kGrpMaxSlots / 2) void xfx_direct_kernel(const XfxArgs a)
{
    extern __shared__ uint4 smem4[];
    char *sm = reinterpret_cast<char *>(smem4);
    const int lane = threadIdx.x & 63;
    const int stage = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t p = (int64_t)blockIdx.x * 64 + lane;
    const double xv = load_point(a.x, p, a.n), qv = load_point(a.q, p, a.n);
    int off = 0;
    const PieceAxis px = place_axis(sm, off, a.ax, 0, a.nx - 1);
    const PieceAxis pq = place_axis(sm, off, a.aq, 0, a.nq - 1);
    {
        const PieceAxis both[2] = {px, pq};
        const AxisDev *const axes[2] = {&a.ax, &a.aq};
        load_axes<sizeof(V) == 4>(both, axes, blockDim.x);
    }
    __syncthreads();
    const uint4 *const group = reinterpret_cast<const uint4 *>(a.gvals) +
                               (RAW ? 0 : (size_t)a.sgrp[stage < a.n_stage ? stage : 0] * a.gstride);
    group_columns<V, AS, RAW>(a, px, pq, group, stage, p, p < a.n, xv, qv);
}

// The same for more points, one group a workgroup: its nodes in LDS, a share of
// `per` points.  The workgroups of a share run on one XCD, whose L2 joins their parts of
// the output rows.  A compute unit copies one group, not all of them (the double-buffered
// kernel, whose time up to 100 thousand points is those copies), for a location per group
// and point; from half a million points on the parts of the rows bound it.  100 thousand
// points x 11 partons on 100 x 50 knots with alpha_s: 18.8 -> 13.3 us FP64, 13.3 -> 8.9 us
// FP32; 300 thousand 44 -> 32 and 29 -> 17.5 us.
constexpr int kGroupBlock = 1024;

template <typename V, bool AS>
__global__ __launch_bounds__(kGroupBlock) void xfx_group_kernel(const XfxArgs a, int per)
{
    extern __shared__ uint4 smem4[];
    char *sm = reinterpret_cast<char *>(smem4);
    const int at = blockIdx.x / 8;
    const int stage = at % a.n_stage;
    const int64_t p0 = (int64_t)(at / a.n_stage * 8 + blockIdx.x % 8) * per;
    if (p0 >= a.n)
        return;
    const int64_t p1 = p0 + per < a.n ? p0 + per : a.n;
    const int nodes = (a.nx + 2) * (a.nq + 2);
    fwd::dma_slab<kGroupBlock>(smem4, reinterpret_cast<const uint4 *>(a.gvals) +
                                          (size_t)a.sgrp[stage] * a.gstride, nodes);
    int64_t p = p0 + threadIdx.x;
    double xv = load_point(a.x, p, p1), qv = load_point(a.q, p, p1);
    int off = nodes * 16;
    const PieceAxis px = place_axis(sm, off, a.ax, 0, a.nx - 1);
    const PieceAxis pq = place_axis(sm, off, a.aq, 0, a.nq - 1);
    {
        const PieceAxis both[2] = {px, pq};
        const AxisDev *const axes[2] = {&a.ax, &a.aq};
        load_axes<sizeof(V) == 4>(both, axes, kGroupBlock);
    }
    fwd::wait_vm();
    __syncthreads();
    // whole waves leave together
    for (; p - (threadIdx.x & 63) < p1; p += kGroupBlock) {
        const double x = xv, q = qv;
        xv = load_point(a.x, p + kGroupBlock, p1);
        qv = load_point(a.q, p + kGroupBlock, p1);
        group_columns<V, AS, false>(a, px, pq, smem4, stage, p, p < p1, x, q);
    }
}

size_t direct_lds(const XfxArgs &a)
{
    return (size_t)route_axis_bytes(a.nx - 1, a.ax.nbuckets) +
           route_axis_bytes(a.nq - 1, a.aq.nbuckets);
}

}  // namespace

static size_t group_lds(const XfxArgs &a)
{
    return (size_t)(a.nx + 2) * (a.nq + 2) * 16 + direct_lds(a);
}

bool xfx_group_fits(const XfxArgs &a)
{
    return a.nx >= 4 && a.nq >= 4 && a.n_stage > 0 && group_lds(a) <= kLdsLimit;
}

hipError_t launch_xfx_group(const XfxArgs &a, bool f32, int cus, hipStream_t s)
{
    auto go = [&](auto fn) -> hipError_t {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)group_lds(a));
        if (e != hipSuccess)
            return e;
        // one workgroup a compute unit, and a multiple of 8 shares
        const int64_t shares = std::max(cus / a.n_stage / 8 * 8, 8);
        const int64_t per = ((a.n + shares - 1) / shares + 63) / 64 * 64;
        hipLaunchKernelGGL(fn, dim3((unsigned)(shares * a.n_stage)), dim3(kGroupBlock), group_lds(a), s,
                           a, (int)per);
        return hipGetLastError();
    };
    if (a.as_out)
        return f32 ? go(xfx_group_kernel<float, true>) : go(xfx_group_kernel<double, true>);
    return f32 ? go(xfx_group_kernel<float, false>) : go(xfx_group_kernel<double, false>);
}

bool xfx_direct_fits(const XfxArgs &a)
{
    return a.nx >= 4 && a.nq >= 4 && direct_lds(a) <= 64 * 1024;
}

hipError_t launch_xfx_direct(const XfxArgs &a, bool f32, bool raw, hipStream_t s)
{
    auto go = [&](auto fn) -> hipError_t {
        const int64_t blocks = (a.n + 63) / 64;
        hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(64 * (a.n_stage > 0 ? a.n_stage : 1)),
                           direct_lds(a), s, a);
        return hipGetLastError();
    };
    if (a.as_out)
        return f32 ? (raw ? go(xfx_direct_kernel<float, true, true>)
                          : go(xfx_direct_kernel<float, true, false>))
                   : (raw ? go(xfx_direct_kernel<double, true, true>)
                          : go(xfx_direct_kernel<double, true, false>));
    return f32 ? (raw ? go(xfx_direct_kernel<float, false, true>)
                      : go(xfx_direct_kernel<float, false, false>))
               : (raw ? go(xfx_direct_kernel<double, false, true>)
                      : go(xfx_direct_kernel<double, false, false>));
}

}  // namespace pdfx
