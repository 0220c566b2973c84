// Routed forward kernel of the Drell-Yan-like integrand (same integrand as
// dy.hip and dy_dma.hip) for large calls: the grid is cut along Q^2 into pieces
// that hold the quarks and antiquarks over all x and stay in LDS, and a workgroup
// takes the points whose Q^2 falls into its piece.  Both stencils of a point,
// at (x1, Q^2) and (x2, Q^2), lie in that one piece, so each point is located and
// evaluated once, with no barrier between the waves and nothing copied per tile.
//
// ln Q^2 is a sum of the inputs, so the points are sorted out by it; Q^2 itself
// may fall on the other side of a knot in its last bits, so a piece holds one
// interval more at either end (two where the first has no width, at a threshold).  Sharing out the work, scanning and the queue of
// points are as in the routed x f kernel; bins, weights and the order of sums are
// those of the other integrand kernels, so each point's value is the same bits.
// Bound by the LDS gathers (160 values a point in FP64: 1280 bytes).  10 million
// points, 100 x 50 knots: 973 -> 438 us FP64, 726 -> 273 us FP32 against the
// double-buffered kernel's default shape.
#include "dy_route.h"
#include "piece_axis.h"

namespace pdfx {

namespace {

using namespace piece;

constexpr int kDyRouteBlock = 768;   // 12 waves of up to 168 registers
constexpr int kDyRouteWaves = kDyRouteBlock / 64;
constexpr int kDyScan = 4;

// The np values of one side (quarks or antiquarks) at byte address p of its first
// plane: full planes of 16 / sizeof(V) rows, then the rest.
template <typename V, typename Use>
__device__ __forceinline__ void side_values(const char *p, int np, int plane, const char *pt,
                                            int qn, const V wx[4], const V wq[4], Use use)
{
    constexpr int G = 16 / (int)sizeof(V);
    const int full = np / G, left = np - full * G;
#pragma unroll
    for (int g = 0; g < 5 / G; ++g)
        if (g < full) {
            V v[G];
            plane_stencil<V, G>(p + g * plane, qn * 16, wx, wq, v);
#pragma unroll
            for (int k = 0; k < G; ++k)
                use(g * G + k, v[k]);
            asm volatile("" ::: "memory");
        }
    if (left == 1) {
        V v[1];
        plane_stencil<V, 1>(pt, qn * (int)sizeof(V), wx, wq, v);
#pragma unroll
        for (int u = 0; u < 5; ++u)
            if (u == full * G)
                use(u, v[0]);
    } else if constexpr (G == 4) {
        if (left == 2) {
            V v[2];
            plane_stencil<V, 2>(pt, qn * 8, wx, wq, v);
            use(0, v[0]);
            use(1, v[1]);
        } else if (left == 3) {
            V v[4];
            plane_stencil<V, 4>(pt, qn * 16, wx, wq, v);
            use(0, v[0]);
            use(1, v[1]);
            use(2, v[2]);
        }
    }
}

template <typename V>
__global__ __launch_bounds__(kDyRouteBlock) void dy_route_kernel(const DyRouteArgs a)
{
    constexpr bool F32 = sizeof(V) == 4;
    constexpr int G = 16 / (int)sizeof(V);
    extern __shared__ uint4 smem4[];
    char *sm = reinterpret_cast<char *>(smem4);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = blockIdx.x % a.teams, place = blockIdx.x / a.teams;
    const int nx = a.nx, nq = a.nq, np = a.np;
    const int64_t p0 = (int64_t)team * a.range_pts;
    const int64_t rest = a.n - p0;
    const int npts = rest <= 0 ? 0 : (int)(rest < a.range_pts ? rest : a.range_pts);
    const double ln_s = log(a.s);
    auto ln_q2 = [&](double ua, double ub) {
        return (a.lnxmin + ua * a.lnrange) + (a.lnxmin + ub * a.lnrange) + ln_s;
    };

    // the piece's intervals [ia, ib) by ln Q^2
    int ia = 0, ib = nq - 1, piece = 0, part = place, width = a.team_size;
    int cut_lo = 0, cut_hi = nq - 1;
    if (a.most < nq - 1) {
        RouteCut *rc = reinterpret_cast<RouteCut *>(sm);
        double *kn = reinterpret_cast<double *>(sm + route_round16(sizeof(RouteCut)));
        make_cut<kDyRouteBlock>(
            rc, kn, reinterpret_cast<int *>(kn + nq), nq, a.most, a.team_size,
            [&](int i) { return log(a.aq.knots[i]); },
            [&](int k) {
                const int64_t i = k * a.n / kRouteSamples;
                return ln_q2(a.u1[i], a.u2[i]);
            });
        while (part >= rc->width[piece]) {
            part -= rc->width[piece];
            ++piece;
        }
        width = __builtin_amdgcn_readfirstlane(rc->width[piece]);
        ia = __builtin_amdgcn_readfirstlane(rc->cut[piece]);
        ib = __builtin_amdgcn_readfirstlane(rc->cut[piece + 1]);
        cut_lo = __builtin_amdgcn_readfirstlane(rc->cut[0]);
        cut_hi = __builtin_amdgcn_readfirstlane(rc->cut[rc->pieces]);
        piece = __builtin_amdgcn_readfirstlane(piece);
        part = __builtin_amdgcn_readfirstlane(part);
        __syncthreads();   // read before the values are written over it
    }
    const bool first = ia == 0, last = ib == nq - 1;
    const double s_lo = log(a.aq.knots[ia]), s_hi = last ? __builtin_inf() : log(a.aq.knots[ib]);
    const bool far_lo = piece == 0 && cut_lo > 0, far_hi = piece == 0 && cut_hi < nq - 1;
    const bool far_any = far_lo || far_hi;
    const double f_hi = far_hi ? log(a.aq.knots[cut_hi]) : __builtin_inf();

    // one interval with a width more at either end, and the knots of their windows
    int ja = max(ia - 1, 0), jb = min(ib + 1, nq - 1);
    if (ja > 0 && a.aq.knots[ja] == a.aq.knots[ja + 1])
        --ja;
    if (jb < nq - 1 && a.aq.knots[jb - 1] == a.aq.knots[jb])
        ++jb;
    auto start = [&](int i) { return i - 1 < 0 ? 0 : i - 1 > nq - 4 ? nq - 4 : i - 1; };
    const int q0 = start(ja), qn = start(jb - 1) + 4 - q0;
    const int nodes = nx * qn, plane = nodes * 16;
    const int full = np / G, tail = route_tail_bytes(np, (int)sizeof(V));
    const int side = route_round16(full * plane + nodes * tail);   // quarks, then antiquarks

    const V *const src = reinterpret_cast<const V *>(a.vals);
    {
        const int lane = tid & 63;
        for (int u = 0; u < 2 * np; ++u) {
            const int v = u < np ? u : u - np;
            char *dst = sm + (u < np ? 0 : side) + (v / G) * plane + (v % G) * (int)sizeof(V);
            const int step = v >= full * G ? tail : 16;
            const V *g = src + (size_t)a.row[u] * a.flav_stride + q0;
            for (int i0 = wave; i0 < nx; i0 += 8 * kDyRouteWaves)
                for (int k = lane; k < qn; k += 64) {
                    V t[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int i = i0 + j * kDyRouteWaves;
                        t[j] = g[(i < nx ? i : i0) * a.x_stride + k];
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int i = i0 + j * kDyRouteWaves;
                        if (i < nx)
                            *reinterpret_cast<V *>(dst + (i * qn + k) * step) = t[j];
                    }
                }
        }
    }
    int off = 2 * side;
    const PieceAxis px = place_axis(sm, off, a.ax, 0, nx - 1);
    const PieceAxis pq = place_axis(sm, off, a.aq, ja, jb - ja);
    {
        const PieceAxis both[2] = {px, pq};
        const AxisDev *const axes[2] = {&a.ax, &a.aq};
        load_axes<F32>(both, axes, kDyRouteBlock);
    }
    const V *asv = reinterpret_cast<const V *>(sm + off) + 1;   // padded by one on each side
    for (int i = tid; i < nq + 2; i += kDyRouteBlock)
        reinterpret_cast<V *>(sm + off)[i] = reinterpret_cast<const V *>(a.as_vals)[i];
    __syncthreads();

    V *const out = reinterpret_cast<V *>(a.out);
    const double *const up = a.u1 + p0, *const vp = a.u2 + p0;
    const int ntile = (npts + 63) / 64;
    const int stride = width * kDyRouteWaves;
    double sum = 0.0;   // this thread's FP64 partial sum of I

    // Tiles of 64 points, scanned kDyScan at a time (see the routed x f kernel).
    const int t_first = part * kDyRouteWaves + wave;
    int t_load = t_first, t_use = t_first, held = 0;
    double un[kDyScan], wn[kDyScan];
    unsigned int bits = 0, bits_next = 0;
    bool raw = false, far_seen = false;
    auto load_tiles = [&]() {
        const int lane = fresh_lane();
#pragma unroll
        for (int k = 0; k < kDyScan; ++k) {
            const int rel = min((t_load + k * stride) * 64 + lane, npts - 1);
            un[k] = up[rel];
            wn[k] = vp[rel];
        }
        raw = true;
    };
    auto is_far = [&](double v) { return (far_lo && !(v >= s_lo)) || (far_hi && v >= f_hi); };
    auto make_bits = [&]() {
        const int lane = fresh_lane();
        bits_next = 0;
#pragma unroll
        for (int k = 0; k < kDyScan; ++k) {
            const int rel = (t_load + k * stride) * 64 + lane;
            const double v = ln_q2(un[k], wn[k]);
            if (rel < npts && (first || v >= s_lo) && !(v >= s_hi))
                bits_next |= 1u << k;
            if (far_any)
                far_seen = far_seen || is_far(v);
        }
        raw = false;
    };
    int n_wait = 0, wait = 0, over = 0;
    int b_n = 0, b_rel = 0;
    double b_u = 0.0, b_v = 0.0;
    auto next_batch = [&]() {
        const int lane = fresh_lane();
        while (n_wait < 64 && (held > 0 || t_load < ntile)) {
            if (held == 0) {
                if (raw)
                    make_bits();
                bits = bits_next;
                t_use = t_load;
                held = kDyScan;
                t_load += kDyScan * stride;
                if (t_load < ntile)
                    load_tiles();
            }
            const bool sel = bits & 1u;
            const unsigned long long mask = __ballot(sel);
            if (mask != 0ull) {
                const int hits = __popcll(mask);
                const int before = __builtin_amdgcn_mbcnt_hi(
                    (unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
                const int dest = n_wait + (sel ? before : hits + lane - before);
                over = __builtin_amdgcn_ds_permute((dest & 63) * 4, t_use * 64 + lane);
                wait = lane < n_wait ? wait : over;
                n_wait += hits;
            }
            bits >>= 1;
            t_use += stride;
            --held;
        }
        b_n = n_wait;
        b_rel = lane < n_wait ? wait : __builtin_amdgcn_readfirstlane(wait);
        wait = over;
        n_wait = n_wait > 64 ? n_wait - 64 : 0;
        b_u = up[b_rel];
        b_v = vp[b_rel];
    };
    // Location of a point: x1, x2 and Q^2 with their logarithms; false outside.
    auto place_point = [&](double ua, double ub, double &x1, double &x2, double &q2, double &l1,
                           double &l2) {
        l1 = a.lnxmin + ua * a.lnrange;
        l2 = a.lnxmin + ub * a.lnrange;
        x1 = exp(l1);
        x2 = exp(l2);
        q2 = x1 * x2 * a.s;
        q2 = q2 < pq.lo ? pq.lo : (q2 > pq.hi ? pq.hi : q2);
        const bool ok = x1 >= px.lo && x1 <= px.hi && x2 >= px.lo && x2 <= px.hi && q2 >= pq.lo &&
                        q2 <= pq.hi;
        if (!ok) {
            x1 = x2 = px.lo;
            l1 = l2 = px.ln_lo;
            q2 = pq.lo;
        }
        return ok;
    };
    auto alphas = [&](int sq, const V wq[4]) {
        const V *av = asv + sq;
        V s = wq[0] * av[0];
        s = fma(wq[1], av[1], s);
        s = fma(wq[2], av[2], s);
        return fma(wq[3], av[3], s);
    };
    auto finish = [&](int rel, bool live, bool ok, V as, V lum) {
        const V I = (V)a.L2 * as * lum;
        if (live) {
            if (out)
                out[p0 + rel] = ok ? I : fwd::quiet_nan<V>();
            sum += ok ? (double)I : __builtin_nan("");
        }
    };
    if (t_load < ntile)
        load_tiles();
    if (npts > 0)
        next_batch();
    while (b_n > 0) {
        const int lane = fresh_lane();
        const int n_now = b_n, rel = b_rel;
        const bool live = lane < n_now;
        const double ua = b_u, ub = b_v;
        next_batch();
        double x1, x2, q2, l1, l2;
        const bool ok = place_point(ua, ub, x1, x2, q2, l1, l2);
        fwd::count_flagged(live && !ok, a.dom_count);
        const double lnq = ln(q2);
        V w1[4], w2[4], wq[4];
        const int i1 = piece_bin(px, x1, l1), i2 = piece_bin(px, x2, l2);
        const int kq = piece_bin(pq, q2, lnq);
        piece_weights<V>(px, i1, l1, w1);
        piece_weights<V>(px, i2, l2, w2);
        piece_weights<V>(pq, kq, lnq, wq);
        const int s1 = window4(i1, nx, w1), s2 = window4(i2, nx, w2);
        const int sq = window4(kq + pq.a, nq, wq);
        const V as = alphas(sq, wq);
        // waited for before this batch's stores: memory operations complete in order
        asm volatile("" : "+v"(b_u), "+v"(b_v));
        if (raw)
            make_bits();
        const int n1 = s1 * qn + (sq - q0), n2 = s2 * qn + (sq - q0);
        V anti[5], lum = V(0);
#pragma unroll
        for (int u = 0; u < 5; ++u)
            anti[u] = V(0);
        side_values<V>(sm + side + n2 * 16, np, plane, sm + side + full * plane + n2 * tail, qn,
                       w2, wq, [&](int u, V v) { anti[u] = v; });
        side_values<V>(sm + n1 * 16, np, plane, sm + full * plane + n1 * tail, qn, w1, wq,
                       [&](int u, V v) { lum = fma(v, anti[u], lum); });
        finish(rel, live, ok, as, lum);
    }

    // Points outside every piece (the sample held none), from global memory.
    if (far_any && __ballot(far_seen) != 0ull) {
        const int lane = tid & 63;
        for (int t = t_first; t < ntile; t += stride) {
            const int rel = t * 64 + lane;
            const double ua = up[min(rel, npts - 1)], ub = vp[min(rel, npts - 1)];
            if (rel >= npts || !is_far(ln_q2(ua, ub)))
                continue;
            double x1, x2, q2, l1, l2;
            const bool ok = place_point(ua, ub, x1, x2, q2, l1, l2);
            if (!ok)   // only some lanes are here
                atomicAdd(a.dom_count, 1ull);
            const double lnq = ln(q2);
            V w1[4], w2[4], wq[4];
            const int s1 = window4(far_weights<V>(a.ax, x1, l1, w1), nx, w1);
            const int s2 = window4(far_weights<V>(a.ax, x2, l2, w2), nx, w2);
            const int sq = window4(far_weights<V>(a.aq, q2, lnq, wq), nq, wq);
            auto value = [&](int row, int sx, const V wx[4]) {
                const V *g = src + (size_t)row * a.flav_stride + (size_t)sx * a.x_stride + sq;
                V acc = V(0);
#pragma unroll
                for (int jx = 0; jx < 4; ++jx, g += a.x_stride) {
                    V r = wq[0] * g[0];
                    r = fma(wq[1], g[1], r);
                    r = fma(wq[2], g[2], r);
                    r = fma(wq[3], g[3], r);
                    acc = (jx == 0) ? wx[0] * r : fma(wx[jx], r, acc);
                }
                return acc;
            };
            V lum = V(0);
            for (int u = 0; u < np; ++u)
                lum = fma(value(a.row[u], s1, w1), value(a.row[np + u], s2, w2), lum);
            finish(rel, true, ok, alphas(sq, wq), lum);
        }
    }

    // workgroup sum of the partial sums (fixed order)
    __syncthreads();
    double *red = reinterpret_cast<double *>(sm);
    red[tid] = sum;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (tid < w && tid + w < kDyRouteBlock)
            red[tid] += red[tid + w];
        __syncthreads();
    }
    if (tid == 0 && a.block_sums)
        a.block_sums[blockIdx.x] = red[0];
}

}  // namespace

int dy_route_most(int nx, int nq, int nbx, int nbq, int np, bool f32)
{
    if (nx < 4 || nq < 4 || np < 1)
        return 0;
    const int vs = f32 ? 4 : 8;
    const int64_t node = 2 * route_node_bytes(np, vs);
    const int64_t room = (int64_t)kLdsLimit - route_round16((nq + 2) * vs) -
                         route_axis_bytes(nx - 1, nbx) - route_axis_bytes(0, nbq) - 64;
    // a piece of m intervals holds up to m + 4 of them and m + 7 knots
    const int64_t most = (room - 7 * nx * node - 160) / (nx * node + 40);
    if (room - 7 * nx * node - 160 <= 0 || most < 1)
        return 0;
    return most >= nq - 1 ? nq - 1 : (int)most;
}

hipError_t launch_dy_route(const DyRouteArgs &a, bool f32, hipStream_t s)
{
    auto go = [&](auto fn) -> hipError_t {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)kLdsLimit);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(fn, dim3((unsigned)(a.teams * a.team_size)), dim3(kDyRouteBlock),
                           kLdsLimit, s, a);
        return hipGetLastError();
    };
    return f32 ? go(dy_route_kernel<float>) : go(dy_route_kernel<double>);
}

}  // namespace pdfx
