// alpha_s(Q^2): 1-D cubic Hermite in ln Q^2 over the alpha_s knots, subgrids
// split at repeated knots (same search, tie and weight rules as the PDF axis).
// Persistent workgroups; the axis tables live in LDS, and with them the cubic of every
// interval, made by each workgroup from the records and the knot values: a point reads
// 48 bytes (FP64) and takes three multiply-adds, where the folded weights took 7
// constants at a 64-byte stride (26 us of LDS time with its conflicts) and 18
// operations.  Bound by vector instructions, half of them the logarithm: 8e6 points FP64
// 39 us (47 with the folded weights), the memory's share 23.
#include "xfx_fwd_impl.h"

namespace pdfx {

namespace {

constexpr int kAsBlock = 256;
constexpr int kAsPpt = 4;

// An interval: its coordinate t = (ln Q^2 - z) inv_d and the cubic in t that the folded
// weights and the four knot values make there.
template <typename V>
struct AsCubic {
    double z, inv_d;
    V c[4];
};

template <typename V>
__global__ __launch_bounds__(kAsBlock) void alphas_kernel(const AlphasArgs a, AxisLds lo)
{
    extern __shared__ uint4 smem4[];
    char *sm = reinterpret_cast<char *>(smem4);
    AsCubic<V> *const cubic = reinterpret_cast<AsCubic<V> *>(sm + lo.rec64);
    const int64_t tile = (int64_t)kAsBlock * kAsPpt;
    // a tile's points are loaded a tile ahead (clamped indices keep these global
    // loads; a select with a default value would make them flat loads)
    double next[kAsPpt];
    auto load = [&](int64_t t0) {
#pragma unroll
        for (int j = 0; j < kAsPpt; ++j)
            next[j] = load_point(a.q2, t0 + (int64_t)j * kAsBlock + threadIdx.x, a.n);
    };
    load((int64_t)blockIdx.x * tile);
    fwd::copy_words<kAsBlock>(sm + lo.knots, a.a.knots, a.a.n * 8);
    fwd::copy_words<kAsBlock>(sm + lo.seed, a.a.seed, a.a.nbuckets * 2);
    // padded values: vals[k'] holds knot k'-1, so interval k's four are vals[k ..]
    const V *const vals = reinterpret_cast<const V *>(a.vals);
    for (int k = threadIdx.x; k < a.a.n - 1; k += kAsBlock) {
        const IntervalRec<double> r = a.a.rec64[k];
        const double v0 = vals[k], v1 = vals[k + 1], v2 = vals[k + 2], v3 = vals[k + 3];
        // the rise and the slopes at both ends (times the width), from differences,
        // which lose nothing
        const double d = v2 - v1;
        const double s1 = fma(r.pl, v1 - v0, r.ql * d), s2 = fma(r.pr, v3 - v2, r.qr * d);
        cubic[k] = AsCubic<V>{r.z, r.inv_d, {(V)v1, (V)s1, (V)(3.0 * d - 2.0 * s1 - s2), (V)(s1 + s2 - 2.0 * d)}};
    }
    __syncthreads();
    fwd::LAxis la;
    la.k = reinterpret_cast<const double *>(sm + lo.knots);
    la.seed = reinterpret_cast<const uint16_t *>(sm + lo.seed);
    la.n = a.a.n;
    la.nb = a.a.nbuckets;
    la.ln_lo = a.a.ln_lo;
    la.inv_hb = a.a.inv_hb;
    V *out = reinterpret_cast<V *>(a.out);
    for (int64_t t0 = (int64_t)blockIdx.x * tile; t0 < a.n; t0 += (int64_t)gridDim.x * tile) {
        double qs[kAsPpt];
#pragma unroll
        for (int j = 0; j < kAsPpt; ++j)
            qs[j] = next[j];
        if (t0 + (int64_t)gridDim.x * tile < a.n)
            load(t0 + (int64_t)gridDim.x * tile);
#pragma unroll
        for (int j = 0; j < kAsPpt; ++j) {
            const int64_t p = t0 + (int64_t)j * kAsBlock + threadIdx.x;
            const bool live = p < a.n;
            double qv = qs[j];
            if (a.q_is_q)
                qv = qv * qv;
            const bool nan_in = qv != qv;
            bool ok = true;
            if (!(qv >= a.a.lo && qv <= a.a.hi)) {
                if (a.domain_mode == 1 && !nan_in) {
                    qv = fmin(fmax(qv, a.a.lo), a.a.hi);
                } else {
                    ok = false;
                    qv = a.a.lo;
                }
            }
            fwd::count_flagged(live && !ok, a.dom_count);
            const double lq = ln(qv);
            const AsCubic<V> c = cubic[fwd::lbin(la, qv, lq)];
            const V t = (V)((lq - c.z) * c.inv_d);
            const V v = fma(fma(fma(c.c[3], t, c.c[2]), t, c.c[1]), t, c.c[0]);
            if (live)
                out[p] = ok ? v : fwd::quiet_nan<V>();
        }
    }
}

}  // namespace

hipError_t launch_alphas(const AlphasArgs &a, bool f32, hipStream_t s)
{
    AxisLds lo;
    size_t off = 0;
    auto take = [&](size_t bytes, size_t align) {
        off = (off + align - 1) / align * align;
        size_t r = off;
        off += bytes;
        return (int)r;
    };
    lo.knots = take((size_t)a.a.n * 8, 16);
    lo.seed = take((size_t)a.a.nbuckets * 2, 16);
    lo.rec64 = take((size_t)(a.a.n - 1) * (f32 ? sizeof(AsCubic<float>) : sizeof(AsCubic<double>)), 16);
    const size_t lds = off;
    if (lds > kLdsLimit)
        return hipErrorInvalidValue;
    const int64_t tile = (int64_t)kAsBlock * kAsPpt;
    int64_t blocks = (a.n + tile - 1) / tile;
    if (blocks > 2048)
        blocks = 2048;
    if (blocks < 1)
        blocks = 1;
    if (f32)
        hipLaunchKernelGGL(alphas_kernel<float>, dim3((unsigned)blocks), dim3(kAsBlock), lds, s, a, lo);
    else
        hipLaunchKernelGGL(alphas_kernel<double>, dim3((unsigned)blocks), dim3(kAsBlock), lds, s, a, lo);
    return hipGetLastError();
}

}  // namespace pdfx
