// Search tables of a part of an axis in LDS: bins, folded weights and windows of
// the kernels that keep their part of the grid resident.
#pragma once

#include "route_internal.h"
#include "set_internal.h"
#include "xfx_fwd_impl.h"

namespace pdfx {
namespace piece {

// One axis of a piece in LDS: knots [0 .. cnt] of its cnt intervals, their
// constants, and the bucket seeds of the whole axis (a: its first interval).
struct PieceAxis {
    const double *k;
    const char *cst;
    const uint16_t *seed;
    int cnt, a, n, nb;
    double lo, hi, ln_lo, inv_hb;
};

// Largest local interval i with k[i] <= v, kept in the piece: the bucket's seed
// and the two knots after it settle nearly every point at once; the others walk.
__device__ __forceinline__ int piece_bin(const PieceAxis &p, double v, double lnv)
{
    const double fb = (lnv - p.ln_lo) * p.inv_hb;
    const int b = fb <= 0.0 ? 0 : (fb >= (double)(p.nb - 1) ? p.nb - 1 : (int)fb);
    const int top = p.cnt - 1;
    int i = (int)p.seed[b] - p.a;
    i = min(max(i, 0), top);
    const double k0 = p.k[i], k1 = p.k[i + 1], k2 = p.k[min(i + 2, p.cnt)];
    const bool up1 = i < top && k1 <= v, up2 = up1 && i + 1 < top && k2 <= v;
    i += (int)up1 + (int)up2;
    if (up2 || k0 > v) {
        while (i < top && p.k[i + 1] <= v)
            ++i;
        while (i > 0 && p.k[i] > v)
            --i;
    }
    return i;
}

// Folded weights of local interval i from its constants: z and 1/d (FP64),
// then pl, pr (FP64) or pl, pl-ql, qr-pr, pr (FP32); ql and qr are 1/2 inside
// the subgrid and 1 at its ends, where pl or pr is 0.
template <typename W>
__device__ __forceinline__ void piece_weights(const PieceAxis &p, int i, double lnv, W w[4]);
template <>
__device__ __forceinline__ void piece_weights<double>(const PieceAxis &p, int i, double lnv,
                                                      double w[4])
{
    const double2 c = *reinterpret_cast<const double2 *>(p.cst + i * 32);
    const double2 e = *reinterpret_cast<const double2 *>(p.cst + i * 32 + 16);
    const double t = (lnv - c.x) * c.y;
    const double ql = e.x != 0.0 ? 0.5 : 1.0, qr = e.y != 0.0 ? 0.5 : 1.0;
    fwd::fold<double>(t, e.x, e.x - ql, ql, qr, qr - e.y, e.y, w);
}
template <>
__device__ __forceinline__ void piece_weights<float>(const PieceAxis &p, int i, double lnv,
                                                     float w[4])
{
    const double2 c = *reinterpret_cast<const double2 *>(p.cst + i * 32);
    const float4 e = *reinterpret_cast<const float4 *>(p.cst + i * 32 + 16);
    const float t = (float)((lnv - c.x) * c.y);
    const float ql = e.x != 0.f ? 0.5f : 1.f, qr = e.w != 0.f ? 0.5f : 1.f;
    fwd::fold<float>(t, e.x, e.y, ql, qr, e.z, e.w, w);
}

// Window of global interval i on an axis of n knots (as the double-buffered
// kernel): its first knot, the weights moved along at the ends.
template <typename W>
__device__ __forceinline__ int window4(int i, int n, W w[4])
{
    int st = i - 1;
    if (st < 0) {
        st = 0;
        w[0] = w[1];
        w[1] = w[2];
        w[2] = w[3];
        w[3] = W(0);
    } else if (st > n - 4) {
        st = n - 4;
        w[3] = w[2];
        w[2] = w[1];
        w[1] = w[0];
        w[0] = W(0);
    }
    return st;
}

// Places one axis part (intervals a .. a + cnt - 1) in LDS at *off.
__device__ __forceinline__ PieceAxis place_axis(char *sm, int &off, const AxisDev &ax, int a,
                                                int cnt)
{
    PieceAxis p;
    p.k = reinterpret_cast<const double *>(sm + off);
    off += route_round16((cnt + 1) * 8);
    p.cst = sm + off;
    off += cnt * 32;
    p.seed = reinterpret_cast<const uint16_t *>(sm + off);
    off += route_round16(ax.nbuckets * 2);
    p.cnt = cnt;
    p.a = a;
    p.n = ax.n;
    p.nb = ax.nbuckets;
    p.lo = ax.lo;
    p.hi = ax.hi;
    p.ln_lo = ax.ln_lo;
    p.inv_hb = ax.inv_hb;
    return p;
}

// Copies the tables of both axis parts into LDS; all loads of a thread are
// issued before its first write.
template <bool F32, int BLOCK>
__device__ __forceinline__ void load_axes(const PieceAxis (&p)[2], const AxisDev *const (&ax)[2])
{
    const int most = max(max(p[0].cnt + 1, p[0].nb / 2), max(p[1].cnt + 1, p[1].nb / 2));
    for (int i = threadIdx.x; i < most; i += BLOCK) {
        double k[2], z[2][2], c64[2][2];
        float c32[2][4];
        unsigned int sd[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int a = p[s].a, ik = min(i, p[s].cnt), ic = min(i, p[s].cnt - 1);
            gptr<double> r64 = (gptr<double>)(ax[s]->rec64 + a + ic);
            k[s] = ((gptr<double>)ax[s]->knots)[a + ik];
            z[s][0] = r64[0];
            z[s][1] = r64[1];
            if constexpr (F32) {
                gptr<float> r32 = (gptr<float>)(ax[s]->rec32 + a + ic);
                c32[s][0] = r32[2];
                c32[s][1] = r32[3];
                c32[s][2] = r32[6];
                c32[s][3] = r32[7];
            } else {
                c64[s][0] = r64[2];
                c64[s][1] = r64[7];
            }
            sd[s] = ((gptr<unsigned int>)ax[s]->seed)[min(i, p[s].nb / 2 - 1)];   // nb % 4 == 0
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            double *d = reinterpret_cast<double *>(const_cast<char *>(p[s].cst) + i * 32);
            if (i <= p[s].cnt)
                const_cast<double *>(p[s].k)[i] = k[s];
            if (i < p[s].cnt) {
                d[0] = z[s][0];
                d[1] = z[s][1];
                if constexpr (F32) {
                    float *f = reinterpret_cast<float *>(d + 2);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        f[j] = c32[s][j];
                } else {
                    d[2] = c64[s][0];
                    d[3] = c64[s][1];
                }
            }
            if (i < p[s].nb / 2)
                reinterpret_cast<unsigned int *>(const_cast<uint16_t *>(p[s].seed))[i] = sd[s];
        }
    }
}

// Bin and folded weights from the tables in global memory, for a point
// outside every piece.
template <typename W>
__device__ __forceinline__ int far_weights(const AxisDev &ax, double v, double lnv, W w[4])
{
    const double fb = (lnv - ax.ln_lo) * ax.inv_hb;
    const int b = fb <= 0.0 ? 0 : (fb >= (double)(ax.nbuckets - 1) ? ax.nbuckets - 1 : (int)fb);
    gptr<double> k = (gptr<double>)ax.knots;
    int i = ((gptr<uint16_t>)ax.seed)[b];
    while (i < ax.n - 2 && k[i + 1] <= v)
        ++i;
    while (i > 0 && k[i] > v)
        --i;
    gptr<double> d = (gptr<double>)(ax.rec64 + i);
    if constexpr (sizeof(W) == 8) {
        const double t = (lnv - d[0]) * d[1];
        fwd::fold<double>(t, d[2], d[3], d[4], d[5], d[6], d[7], w);
    } else {
        gptr<float> f = (gptr<float>)(ax.rec32 + i);
        const float t = (float)((lnv - d[0]) * d[1]);
        fwd::fold<float>(t, f[2], f[3], f[4], f[5], f[6], f[7], w);
    }
    return i;
}

}  // namespace piece
}  // namespace pdfx
