// Double-buffered forward kernel of the Drell-Yan-like integrand (same
// integrand as dy.hip) for grids that fit the double-buffered xf kernel and
// hold the 11 partons in the standard order (-5 .. -1, g, 1 .. 5).
//
// The flavour groups of the grid are walked once per tile: with that order,
// the groups up to the one holding -1 are evaluated at (x2, Q^2) and the ones
// from the group holding 1 on at (x1, Q^2) (FP32: the middle group {-1, g, 1,
// 2} at both), so every result lands in a register slot fixed at compile
// time and the partner products need no indexing.  The luminosity sum runs
// over q = 1 .. 5 in the same order and with the same operations as the
// single-slab kernel, so both give the same per-point values.
//
// Staging, LDS layout and the overlap of the next tile's point location with
// the stencil stages follow the double-buffered xf kernel; alpha_s is located
// by bisection over its knots in LDS, its interval records and values are
// read from global memory.
#include "xfx_dma_impl.h"
#include "fixed_point.h"
#include "scatter_order.h"

namespace pdfx {

namespace {

using fwd::kDmaKnots;
using fwd::kDmaNodes;
using fwd::kDmaSeeds;

// Largest i in [0, n-2] with k[i] <= v, for v in [k[0], k[n-1]].
__device__ __forceinline__ int bisect(const double *k, int n, double v)
{
    int lo = 0, hi = n - 2;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (k[mid] <= v)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Per-point state: bins and weights of (x1, Q^2), (x2, Q^2), alpha_s.
template <typename V>
struct DyPoint {
    V w1[4], w2[4], wq[4];
    int b1, b2;
    V as;
    bool ok;
};

template <typename V, int BLOCK, int PPT>
__global__ __launch_bounds__(BLOCK) void dy_dma_kernel(const DyArgs a)
{
    constexpr int G = 16 / (int)sizeof(V);
    constexpr int NS = 12 / G;   // groups of the 11-parton grid
    __shared__ uint4 slab0[kDmaNodes];
    __shared__ uint4 slab1[kDmaNodes];
    __shared__ double knots[kDmaKnots];
    __shared__ uint16_t seeds[kDmaSeeds];
    const int tid = threadIdx.x;

    const int nx = a.nx, nq = a.nq, na = a.aa.n;
    const int nodes = nx * nq;
    const uint4 *gsrc = reinterpret_cast<const uint4 *>(a.gvals);
    V *out = reinterpret_cast<V *>(a.out);
    const V *asv = reinterpret_cast<const V *>(a.as_vals);
    const int64_t tile_pts = (int64_t)BLOCK * PPT;
    const int64_t ntiles = (a.n + tile_pts - 1) / tile_pts;

    if ((int64_t)blockIdx.x < ntiles)
        fwd::dma_slab<BLOCK>(slab0, gsrc, nodes);   // first group of the first tile
    fwd::copy_words<BLOCK>(reinterpret_cast<char *>(knots), a.ax.knots, nx * 8);
    fwd::copy_words<BLOCK>(reinterpret_cast<char *>(knots + nx), a.aq.knots, nq * 8);
    fwd::copy_words<BLOCK>(reinterpret_cast<char *>(knots + nx + nq), a.aa.knots, na * 8);
    fwd::copy_words<BLOCK>(reinterpret_cast<char *>(seeds), a.ax.seed, a.ax.nbuckets * 2);
    fwd::copy_words<BLOCK>(reinterpret_cast<char *>(seeds + a.ax.nbuckets), a.aq.seed,
                           a.aq.nbuckets * 2);
    __syncthreads();
    fwd::LAxis lx, lq;
    lx.k = knots;
    lx.seed = seeds;
    lx.n = nx;
    lx.nb = a.ax.nbuckets;
    lx.ln_lo = a.ax.ln_lo;
    lx.inv_hb = a.ax.inv_hb;
    lq.k = knots + nx;
    lq.seed = seeds + a.ax.nbuckets;
    lq.n = nq;
    lq.nb = a.aq.nbuckets;
    lq.ln_lo = a.aq.ln_lo;
    lq.inv_hb = a.aq.inv_hb;
    const double *ka_knots = knots + nx + nq;

    auto locate = [&](double ua, double ub, int64_t p, DyPoint<V> &st) {
        const double l1 = a.lnxmin + ua * a.lnrange;
        const double l2 = a.lnxmin + ub * a.lnrange;
        double x1 = exp(l1), x2 = exp(l2);
        double q2 = x1 * x2 * a.s;
        q2 = q2 < a.aq.lo ? a.aq.lo : (q2 > a.aq.hi ? a.aq.hi : q2);
        st.ok = x1 >= a.ax.lo && x1 <= a.ax.hi && x2 >= a.ax.lo && x2 <= a.ax.hi &&
                q2 >= a.aa.lo && q2 <= a.aa.hi;
        fwd::count_flagged(p < a.n && !st.ok, a.dom_count);
        // ln x is the exponent itself (the bins compare raw x, so a last-bit
        // difference from log(x) cannot change them)
        double lnx1 = l1, lnx2 = l2;
        if (!st.ok) {
            x1 = x2 = a.ax.lo;
            lnx1 = lnx2 = a.ax.ln_lo;
            q2 = a.aq.lo > a.aa.lo ? a.aq.lo : a.aa.lo;
        }
        const double lnq = ln(q2);
        const int i1 = fwd::lbin(lx, x1, lnx1);
        const int i2 = fwd::lbin(lx, x2, lnx2);
        const int kq = fwd::lbin(lq, q2, lnq);
        fwd::weights_gmem<V>(a.ax, i1, lnx1, st.w1);
        fwd::weights_gmem<V>(a.ax, i2, lnx2, st.w2);
        fwd::weights_gmem<V>(a.aq, kq, lnq, st.wq);
        const int cq = fwd::window(kq, nq, st.wq);
        st.b1 = fwd::window(i1, nx, st.w1) * nq + cq;
        st.b2 = fwd::window(i2, nx, st.w2) * nq + cq;
        const int ka = bisect(ka_knots, na, q2);
        V wa[4];
        fwd::weights_gmem<V>(a.aa, ka, lnq, wa);
        V av = wa[0] * asv[ka];
        av = fma(wa[1], asv[ka + 1], av);
        av = fma(wa[2], asv[ka + 2], av);
        av = fma(wa[3], asv[ka + 3], av);
        st.as = av;
    };

    // Stencil of one group at one point (window base b, weights wx, wq).
    auto stencil = [&](const uint4 *slab, int b, const V (&wx)[4], const V (&wq)[4], V (&r)[G]) {
        V acc[G];
#pragma unroll
        for (int jx = 0; jx < 4; ++jx) {
            const uint4 *rowp = slab + b + jx * nq;
            V rr[G];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                V v[G];
                fwd::Node<V>::get(rowp + k, v);
#pragma unroll
                for (int g = 0; g < G; ++g)
                    rr[g] = (k == 0) ? wq[0] * v[g] : fma(wq[k], v[g], rr[g]);
            }
#pragma unroll
            for (int g = 0; g < G; ++g)
                acc[g] = (jx == 0) ? wx[0] * rr[g] : fma(wx[jx], rr[g], acc[g]);
        }
#pragma unroll
        for (int g = 0; g < G; ++g)
            r[g] = acc[g];
    };

    // Point state of the current tile and of the next one; the next tile's
    // points are located during the current tile's stencil stages (point j
    // in stage j), whose time goes to LDS traffic.
    DyPoint<V> cur[PPT], nxt[PPT];
    double unext[PPT], vnext[PPT];
    if ((int64_t)blockIdx.x < ntiles) {
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            const int64_t p = (int64_t)blockIdx.x * tile_pts + tid + (int64_t)j * BLOCK;
            locate(load_point(a.u1, p, a.n), load_point(a.u2, p, a.n), p, cur[j]);
            const int64_t pn = p + (int64_t)gridDim.x * tile_pts;
            unext[j] = load_point(a.u1, pn, a.n);
            vnext[j] = load_point(a.u2, pn, a.n);
        }
    }

    double part = 0.0;   // this thread's FP64 partial sum of I
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t t0 = tile * tile_pts;
        const bool more = tile + gridDim.x < ntiles;
        const int64_t pnext0 = t0 + (int64_t)gridDim.x * tile_pts + tid;
        auto locate_next = [&](int j) {
            const int64_t pn = pnext0 + (int64_t)j * BLOCK;
            locate(unext[j], vnext[j], pn, nxt[j]);
            const int64_t pnn = pn + (int64_t)gridDim.x * tile_pts;
            unext[j] = load_point(a.u1, pnn, a.n);
            vnext[j] = load_point(a.u2, pnn, a.n);
        };

        fwd::wait_vm();
        __syncthreads();   // the tile's first group has landed

        // x2-side values by grid row (antiquarks -5 .. -1 are rows 0 .. 4;
        // the gluon slot is not used) and the luminosity sum.
        V at2[PPT][12], lum[PPT];
#pragma unroll
        for (int j = 0; j < PPT; ++j)
            lum[j] = V(0);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            // (a.n_seq is 10 for this kernel: the test is always true; as a
            // runtime test it keeps each stage's arithmetic in the stage's
            // own block instead of letting it drift to the end of the tile,
            // where the loaded nodes would all have to stay live)
            if (a.n_seq < 2 * s)
                continue;
            const uint4 *cs = (s & 1) ? slab1 : slab0;
            uint4 *ns = (s & 1) ? slab0 : slab1;
            if (s + 1 < NS)
                fwd::dma_slab<BLOCK>(ns, gsrc + (size_t)(s + 1) * a.gstride, nodes);
            else if ((s & 1) && more)
                fwd::dma_slab<BLOCK>(slab0, gsrc, nodes);   // slab0 is free during the last stage
            if (s < PPT)
                locate_next(s);
            // rows s*G .. s*G+G-1: antiquarks are rows 0 .. 4, quarks rows 6 .. 10
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                V r[G];
                if (s * G <= 4) {
                    stencil(cs, cur[j].b2, cur[j].w2, cur[j].wq, r);
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        at2[j][s * G + g] = r[g];
                }
                if (s * G + G - 1 >= 6) {
                    stencil(cs, cur[j].b1, cur[j].w1, cur[j].wq, r);
                    // quark q = row - 5 meets its antiquark (row 5 - q) at x2,
                    // in the order q = 1 .. 5
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const int q = s * G + g - 5;
                        if (q >= 1 && q <= 5)
                            lum[j] = fma(r[g], at2[j][5 - q], lum[j]);
                    }
                }
            }
            if (s + 1 < NS) {
                fwd::wait_vm();
                __syncthreads();
            }
        }
#pragma unroll
        for (int j = NS; j < PPT; ++j)
            locate_next(j);   // more points per thread than stages
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            const V I = (V)a.L2 * cur[j].as * lum[j];
            const int64_t p = t0 + tid + (int64_t)j * BLOCK;
            if (p < a.n) {
                if (out)
                    out[p] = cur[j].ok ? I : fwd::quiet_nan<V>();
                part += cur[j].ok ? (double)I : __builtin_nan("");
            }
            cur[j] = nxt[j];
        }
        if ((NS & 1) && more) {
            // the last stage read slab0: start the next tile's first group now
            __syncthreads();
            fwd::dma_slab<BLOCK>(slab0, gsrc, nodes);
        }
    }

    // workgroup sum of the partial sums (fixed order: deterministic)
    fwd::wait_vm();
    __syncthreads();
    double *red = reinterpret_cast<double *>(slab1);
    red[tid] = part;
    __syncthreads();
    for (int w = BLOCK / 2; w > 0; w >>= 1) {
        if (tid < w)
            red[tid] += red[tid + w];
        __syncthreads();
    }
    if (tid == 0 && a.block_sums)
        a.block_sums[blockIdx.x] = red[0];
}

template <typename V>
hipError_t dy_dma_typed(const DyArgs &a, LaunchShape ls, int cus, hipStream_t s, int *n_blocks)
{
    auto go = [&](auto fn, int block, int ppt) -> hipError_t {
        const int64_t tile_pts = (int64_t)block * ppt;
        const int64_t ntiles = (a.n + tile_pts - 1) / tile_pts;
        int per_cu = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, reinterpret_cast<const void *>(fn), block, 0);
        if (e != hipSuccess || per_cu < 1)
            per_cu = 1;
        int64_t grid = (int64_t)per_cu * cus;
        if (grid > ntiles)
            grid = ntiles;
        if (grid > kDyMaxBlocks)
            grid = kDyMaxBlocks;
        if (grid < 1)
            grid = 1;
        hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(block), 0, s, a);
        *n_blocks = (int)grid;
        return hipGetLastError();
    };
    if (ls.block == 512 && ls.ppt == 1)
        return go(dy_dma_kernel<V, 512, 1>, 512, 1);
    if (ls.block == 512 && ls.ppt == 2)
        return go(dy_dma_kernel<V, 512, 2>, 512, 2);
    if (ls.block == 256 && ls.ppt == 2)
        return go(dy_dma_kernel<V, 256, 2>, 256, 2);
    if constexpr (sizeof(V) == 4) {
        if (ls.block == 512 && ls.ppt == 4)
            return go(dy_dma_kernel<V, 512, 4>, 512, 4);
    }
    return hipErrorInvalidValue;
}

// ---- backward, one quark-antiquark pair per workgroup ----
//
// dI/dv_q[i][k]  = L^2 alpha_s xf_-q(x2) w1_i wq_k and
// dI/dv_-q[i][k] = L^2 alpha_s xf_q(x1)  w2_i wq_k, summed over the points.
// A workgroup takes one pair (q, -q) and one chunk of points: both value
// slabs and both gradient slabs (borderless) sit in LDS, so each point's
// state (bins, local coordinates, alpha_s from the state pass) is read and its
// weights folded once for the two flavours, and each partner value comes from
// a 16-tap stencil of the other flavour's slab.  The LDS gradients are added
// to the FP64 accumulator at the end.  The 32 adds of a point are made in its lane's
// own order over a blocked layout (scatter_order.h), so that the lanes of an add hit
// different banks, and so are its 32 reads (its stencil sums of a point then depend on
// its lane in the last bit); the constants that the weights need are in LDS.  The sums
// are kept in 64-bit fixed point (integer LDS adds run ~1.9x faster than FP64 ones, and
// integer sums are exact and independent of the order of the adds).  1e7 points, 100 x
// 50 knots, FP64: 857 us, 590 of them vector instructions and 433 LDS; in one order, with
// the points dealt to lanes by the bank of the quark's stencil and the interval records
// gathered from global memory, 1076 us (926 of them LDS).  1e5 points 28 us (31).
// The scale is a power of two per workgroup and array,
// from a bound on the terms: |alpha_s| <= B_a max|alpha knot|, a partner value
// <= B_x B_q max|row value|, one weight product <= B_x B_q, with B the largest
// sum of |weights| over an axis' intervals (1 + 4/27 times the sum of the
// interval's |fold constants|, as |h10|, |h11| <= 4/27 and h00 + h01 = 1).
// Every term is then below 2^50 and every sum of the chunk's terms below 2^61.
// Non-finite inputs make the two rows' gradients NaN.

constexpr int kPairBlock = 1024;

// Where the pair's knots lie: the quark's in strips of 4 lines upwards from word 0, the
// antiquark's in strips downwards from `down`.  If the last strip holds 1 or 2 lines,
// the two flavours' share its words, so that 100 x 50 FP64 knots fit with strips of a
// multiple of 16 words (BlockLayout; else windows across two strips meet other lanes'
// words: the kernel's LDS time 671 us instead of 433 at 1e7 points).
struct PairLayout {
    int strip, down, words;   // words: of both flavours
    bool swapped;             // strips along Q^2 instead of x
    bool pairs;               // the intervals' FoldPair fit, too
};

__device__ __forceinline__ int pair_word(const PairLayout &y, bool anti, int ix, int kq)
{
    const int a = y.swapped ? kq : ix, b = y.swapped ? ix : kq;
    return (anti ? y.down - (a >> 2) * y.strip : (a >> 2) * y.strip) + b * 4 + (a & 3);
}

// LDS: the gradients of the two flavours, then their values in the same layout (FP32
// ones widened), then the FoldPair of the intervals of the x axis and of the Q^2 axis.
template <typename V, bool SWAPPED>
__global__ __launch_bounds__(kPairBlock) void dy_pair_adjoint_kernel(const DyArgs a, const PairLayout y)
{
    constexpr int G = 16 / (int)sizeof(V);
    extern __shared__ unsigned long long gq[];
    double *const vals = reinterpret_cast<double *>(gq + y.words);
    FoldPair *const cx = reinterpret_cast<FoldPair *>(gq + 2 * y.words);
    FoldPair *const cq = cx + a.nx - 1;
    const int q = blockIdx.y + 1;          // quark q: row 5 + q; antiquark: row 5 - q
    const int rq = 5 + q, rqb = 5 - q;
    const int nx = a.nx, nq = a.nq, nodes = nx * nq;
    const V *src = reinterpret_cast<const V *>(a.gvals);
    // m[0..5]: max |quark value|, max |antiquark value|, weight-sum bounds of
    // the x, Q^2 and alpha_s axes, max |alpha_s knot value|
    double m[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    // (five at once: a grid of up to 5000 knots loads all its values before it waits)
    for (int e0 = threadIdx.x; e0 < nodes; e0 += 5 * kPairBlock) {
        V u[5], ub[5];
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            const int e = min(e0 + t * kPairBlock, nodes - 1);
            u[t] = src[((size_t)(rq / G) * a.gstride + e) * G + rq % G];
            ub[t] = src[((size_t)(rqb / G) * a.gstride + e) * G + rqb % G];
        }
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            const int e = min(e0 + t * kPairBlock, nodes - 1);
            const int i = e / nq, k = e - i * nq;
            vals[pair_word(y, false, i, k)] = (double)u[t];
            vals[pair_word(y, true, i, k)] = (double)ub[t];
            m[0] = nan_max(m[0], fabs((double)u[t]));
            m[1] = nan_max(m[1], fabs((double)ub[t]));
        }
    }
    for (int i = threadIdx.x; i < nx - 1; i += kPairBlock) {
        const IntervalRec<double> r = a.ax.rec64[i];
        m[2] = fmax(m[2], weight_sum_bound(r));
        if (y.pairs)
            cx[i] = FoldPair{r.pl, r.pr};
    }
    for (int i = threadIdx.x; i < nq - 1; i += kPairBlock) {
        const IntervalRec<double> r = a.aq.rec64[i];
        m[3] = fmax(m[3], weight_sum_bound(r));
        if (y.pairs)
            cq[i] = FoldPair{r.pl, r.pr};
    }
    for (int i = threadIdx.x; i < a.aa.n - 1; i += kPairBlock)
        m[4] = fmax(m[4], weight_sum_bound(a.aa.rec64[i]));
    for (int i = threadIdx.x; i < a.aa.n + 2; i += kPairBlock)
        m[5] = fmax(m[5], fabs(a.as_vals64[i]));
    block_max<6, kPairBlock / 64>(m, reinterpret_cast<double *>(gq));   // in the gradients' place
    __syncthreads();
    for (int e = threadIdx.x; e < y.words; e += kPairBlock)
        gq[e] = 0ull;
    __syncthreads();
    const int64_t p_begin = (int64_t)blockIdx.x * a.chunk;
    const int64_t p_end = p_begin + a.chunk < a.n ? p_begin + a.chunk : a.n;
    // quark terms carry the antiquark value and the reverse
    const double kc = fabs(a.scale * a.L2) * m[4] * m[5] * m[2] * m[2] * m[3] * m[3];
    const double bnd_q = kc * m[1], bnd_qb = kc * m[0];
    const bool finite = bnd_q < 1.0 / 0.0 && bnd_qb < 1.0 / 0.0;   // false for NaN too
    const int e_q = finite ? fixed_exponent(bnd_q, p_end - p_begin) : 0;
    const int e_qb = finite ? fixed_exponent(bnd_qb, p_end - p_begin) : 0;
    const double f_q = ldexp(1.0, e_q), f_qb = ldexp(1.0, e_qb);
    const int key = threadIdx.x & 15;
    // The next step's state is loaded a step ahead (clamped to the chunk).
    struct State {
        int i1, i2;
        double t1, t2, tq, as;
    };
    auto load_state = [&](int64_t p) {
        const int64_t pc = p < p_end ? p : p_end - 1;
        return State{a.st_i1[pc], a.st_i2[pc], a.st_t1[pc], a.st_t2[pc], a.st_tq[pc], a.st_as[pc]};
    };
    int64_t p = p_begin + threadIdx.x;
    State nxt = load_state(p);
    for (; finite && p < p_end; p += kPairBlock) {
        const State st = nxt;
        nxt = load_state(p + kPairBlock);
        if (st.i1 < 0)   // outside the grid
            continue;
        const int i1 = st.i1 & 0xffff, kq = st.i1 >> 16, i2 = st.i2;
        FoldPair c1, c2, cc;
        if (y.pairs) {
            c1 = cx[i1];
            c2 = cx[i2];
            cc = cq[kq];
        } else {
            c1 = FoldPair{a.ax.rec64[i1].pl, a.ax.rec64[i1].pr};
            c2 = FoldPair{a.ax.rec64[i2].pl, a.ax.rec64[i2].pr};
            cc = FoldPair{a.aq.rec64[kq].pl, a.aq.rec64[kq].pr};
        }
        double w1[4], w2[4], wq[4];
        fold_pair(st.t1, c1, w1);
        fold_pair(st.t2, c2, w2);
        fold_pair(st.tq, cc, wq);
        const int sq = visit_start(kq, nq), s1 = visit_start(i1, nx), s2 = visit_start(i2, nx);
        // everything below in the lane's order: u[i] the weights along x, uq[k] along Q^2
        double u1[4], u2[4], uq[4];
        int l1[4], l2[4], lq1[4], lq2[4];
        if constexpr (SWAPPED) {
            visit_weights(wq, kq, key, uq);
            visit_weights(w1, i1, key >> 2, u1);
            visit_weights(w2, i2, key >> 2, u2);
            visit_rows<8>(sq, y.strip, key, lq1);
            visit_rows<8>(sq, -y.strip, key, lq2);
            visit_cols<8>(s1, key, l1);
            visit_cols<8>(s2, key, l2);
        } else {
            visit_weights(wq, kq, key >> 2, uq);
            visit_weights(w1, i1, key, u1);
            visit_weights(w2, i2, key, u2);
            visit_rows<8>(s1, y.strip, key, l1);
            visit_rows<8>(s2, -y.strip, key, l2);
            visit_cols<8>(sq, key, lq1);
            visit_cols<8>(sq, key, lq2);
        }
        // partner values: xf_q(x1) for the antiquark, xf_-q(x2) for the quark
        auto partner = [&](int first, const int (&l)[4], const int (&lq)[4], const double (&u)[4]) {
            double f = 0.0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                double r = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    r = fma(uq[k], __longlong_as_double((long long)*visit_word(gq + first, l[i], lq[k])), r);
                f = fma(u[i], r, f);
            }
            return f;
        };
        auto scatter = [&](int first, const int (&l)[4], const int (&lq)[4], const double (&u)[4],
                           double m) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double mi = m * u[i];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    atomicAdd((unsigned long long *)visit_word(gq + first, l[i], lq[k]),
                              to_fixed(mi, uq[k]));
            }
        };
        const double c = a.scale * a.L2 * st.as;
        const double mq = c * partner(y.words + y.down, l2, lq2, u2) * f_q;   // f_*: powers of two
        const double mqb = c * partner(y.words, l1, lq1, u1) * f_qb;
        scatter(0, l1, lq1, u1, mq);
        scatter(y.down, l2, lq2, u2, mqb);
    }
    __syncthreads();
    double *dq = a.gacc + (size_t)rq * nodes;
    double *dqb = a.gacc + (size_t)rqb * nodes;
    const double i_q = ldexp(1.0, -e_q), i_qb = ldexp(1.0, -e_qb);
    for (int e = threadIdx.x; e < nodes; e += kPairBlock) {
        if (!finite) {
            unsafeAtomicAdd(&dq[e], __builtin_nan(""));
            unsafeAtomicAdd(&dqb[e], __builtin_nan(""));
            continue;
        }
        const int i = e / nq, k = e - i * nq;
        const long long sq = (long long)gq[pair_word(y, false, i, k)];
        const long long sqb = (long long)gq[pair_word(y, true, i, k)];
        if (sq != 0)
            unsafeAtomicAdd(&dq[e], (double)sq * i_q);
        if (sqb != 0)
            unsafeAtomicAdd(&dqb[e], (double)sqb * i_qb);
    }
}

}  // namespace

// The first that fits: with the constants in LDS, then strips of a multiple of 16 words,
// then strips along x.  Without any of them every grid of launch_dy_dma_forward fits.
static bool pair_layout(int nx, int nq, PairLayout *y)
{
    auto up = [](int n) { return (n + 3) / 4 * 4; };
    const int room = (int)(kLdsLimit / 16), pairs = nx + nq - 2;   // in 16 bytes
    for (int t = 0; t < 8; ++t) {
        const bool swapped = t & 1, packed = t & 2, far = t & 4;
        const int na = swapped ? nq : nx, nb = swapped ? nx : nq;
        const int strips = up(na) / 4, rest = na % 4;
        const int strip = 4 * (packed ? nb : up(nb));
        const int down = rest == 1 || rest == 2 ? 2 * (strips - 1) * strip + 2 : (2 * strips - 1) * strip;
        const int least = 6 * (kPairBlock / 64);   // the waves' maxima
        const int words = down + strip < least ? least : up(down + strip);
        if (words + (far ? 0 : pairs) <= room) {
            *y = PairLayout{strip, down, words, swapped, !far};
            return true;
        }
    }
    return false;
}

// Pair-wise integrand adjoint (standard parton order, grid fits the
// double-buffered layout): one workgroup per (point chunk, q), one resident
// workgroup per compute unit.
hipError_t launch_dy_pair_adjoint(const DyArgs &a0, bool f32, int cus, hipStream_t s)
{
    DyArgs a = a0;
    int64_t nchunk = cus / 5 > 0 ? cus / 5 : 1;
    int64_t chunk = (a.n + nchunk - 1) / nchunk;
    if (chunk < kPairBlock)
        chunk = kPairBlock;
    nchunk = (a.n + chunk - 1) / chunk;
    a.chunk = (int)chunk;
    PairLayout y;
    if (!pair_layout(a.nx, a.nq, &y))
        return hipErrorInvalidValue;
    const size_t lds = (size_t)16 * y.words + (y.pairs ? (size_t)(a.nx + a.nq - 2) * sizeof(FoldPair) : 0);
    auto go = [&](auto fn) -> hipError_t {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(fn, dim3((unsigned)nchunk, 5u), dim3(kPairBlock), lds, s, a, y);
        return hipGetLastError();
    };
    if (f32)
        return y.swapped ? go(dy_pair_adjoint_kernel<float, true>) : go(dy_pair_adjoint_kernel<float, false>);
    return y.swapped ? go(dy_pair_adjoint_kernel<double, true>) : go(dy_pair_adjoint_kernel<double, false>);
}

bool dy_shape_supported(LaunchShape ls, bool f32)
{
    return (ls.block == 512 && (ls.ppt == 1 || ls.ppt == 2)) || (ls.block == 256 && ls.ppt == 2) ||
           (f32 && ls.block == 512 && ls.ppt == 4);
}

bool dy_dma_supported(int nx, int nq, int na, int nbx, int nbq)
{
    return nx >= 4 && nq >= 4 && na >= 2 && nx * nq <= kDmaNodes && nx + nq + na <= kDmaKnots &&
           nbx + nbq <= kDmaSeeds;
}

hipError_t launch_dy_dma_forward(const DyArgs &a, bool f32, LaunchShape ls, int cus,
                                 hipStream_t s, int *n_blocks)
{
    return f32 ? dy_dma_typed<float>(a, ls, cus, s, n_blocks)
               : dy_dma_typed<double>(a, ls, cus, s, n_blocks);
}

}  // namespace pdfx
