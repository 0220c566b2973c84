// Routed forward kernel: batched x f(x, Q^2) of one grid or of every member
// of a set, with the grid cut into pieces that stay in LDS.
//
// A grid's values for all requested partons (440 KB in FP64 for 11 x 100 x 50)
// do not fit the 160 KB of a compute unit.  Instead of cycling flavour groups
// through LDS for every tile of points, the grid is cut along one axis into
// pieces (33 of 99 x intervals, with the 3 rows a window needs beyond them)
// that hold every requested parton, and a workgroup keeps one piece for the
// whole call.  It scans the points, takes those that fall into its piece (64
// at a time, so that no lane idles) and writes their complete rows: nothing is
// copied per tile, no barrier stands between the waves, and one wave's search
// and logarithms run beside another's gathers.
//
// The workgroups of an XCD (by block index) form a team that works through a
// range of points of one member; they are shared out among the pieces by the
// share of the points in each, estimated from 1024 of them (the estimate only
// decides who does what).  The pieces of a team sweep the range side by side,
// so that the rows of neighbouring points, which share 128-byte lines, meet in
// that XCD's L2.
//
// Same bins, weights and order of sums as the other forward kernels, so the
// same bits.
//
// Bound by the LDS in FP64 (its pipe is busy for three quarters of the kernel,
// two thirds of that in bank conflicts of the random 16-byte gathers) and by the
// vector ALU and the LDS alike in FP32; rows that are finished by two
// workgroups cost up to 60% more HBM writes than the rows' bytes.  10 million
// points, 11 partons and alpha_s on 100 x 50 knots: 934 -> 489 us FP64 and 588 ->
// 302 us FP32 against the double-buffered kernel's default shape; 3 million
// points, 5 partons on 150 x 60 knots, continued outside: 345 -> 125 us; 101
// members of 200003 points FP64: 4.37 -> 1.10 ms, of 1 million FP32: 5.97 -> 2.95.
#include "piece_axis.h"
#include "set_internal.h"

#include <type_traits>

namespace pdfx {

namespace {

using namespace piece;

// Workgroup size by precision, one workgroup a compute unit: 16 waves of 128
// registers in FP32; FP64, whose weights and gathers take twice the registers,
// spills there and runs 12 waves (10 million points, 11 partons: 588 us against 601).
template <typename V>
constexpr int kRouteBlock = sizeof(V) == 8 ? 768 : 1024;
constexpr int kRouteScan = 4;      // tiles of 64 points whose coordinates are loaded at once

template <int K, typename V>
__device__ __forceinline__ void store_values(V *dst, const V v[K])
{
    if constexpr (K == 4) {
        typedef V vec __attribute__((ext_vector_type(4), aligned(sizeof(V))));
        *reinterpret_cast<vec *>(dst) = vec{v[0], v[1], v[2], v[3]};
    } else if constexpr (K == 3) {
        typedef V vec __attribute__((ext_vector_type(3), aligned(sizeof(V))));
        *reinterpret_cast<vec *>(dst) = vec{v[0], v[1], v[2]};
    } else if constexpr (K == 2) {
        typedef V vec __attribute__((ext_vector_type(2), aligned(sizeof(V))));
        *reinterpret_cast<vec *>(dst) = vec{v[0], v[1]};
    } else {
#pragma unroll
        for (int g = 0; g < K; ++g)
            dst[g] = v[g];
    }
}

// Member m, read through the scalar cache (the table is constant).
typedef const __attribute__((address_space(4))) uint32_t *cptr32;
__device__ __forceinline__ MemberDev member(const RouteArgs &a, int m)
{
    MemberDev md = a.one;
    if (a.mem) {
        cptr32 g = (cptr32)(uintptr_t)(a.mem + m);
        uint32_t w[sizeof(MemberDev) / 4];
#pragma unroll
        for (int i = 0; i < (int)(sizeof(MemberDev) / 4); ++i)
            w[i] = g[i];
        __builtin_memcpy(&md, w, sizeof(MemberDev));
    }
    return md;
}

template <typename V, bool AS>
__global__ __launch_bounds__(kRouteBlock<V>) void xfx_route_kernel(const RouteArgs a)
{
    constexpr int BLOCK = kRouteBlock<V>, WAVES = BLOCK / 64;
    constexpr bool F32 = sizeof(V) == 4;
    constexpr int G = 16 / (int)sizeof(V);
    extern __shared__ uint4 smem4[];
    char *sm = reinterpret_cast<char *>(smem4);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = blockIdx.x % a.teams, place = blockIdx.x / a.teams;
    const int n_u = a.n_u;
    const int full = n_u / G;                                       // 16-byte planes
    const int tail = route_tail_bytes(n_u, (int)sizeof(V));         // bytes of the last plane

    for (int unit = team; unit < a.n_units; unit += a.teams) {
        const int m = unit / a.ranges;
        const MemberDev md = member(a, m);
        const int nx = md.nx, nq = md.nq;
        const int64_t p0 = (int64_t)(unit - m * a.ranges) * a.range_pts;
        const int64_t left = a.n - p0;
        const int npts = (int)(left < a.range_pts ? left : a.range_pts);
        const RoutePlan plan = route_plan(nx, nq, md.ax.nbuckets, md.aq.nbuckets, n_u,
                                          (int)sizeof(V), AS ? (nq + 2) * (int)sizeof(V) : 0);
        const bool by_q = plan.split != 0;
        const int ns = by_q ? nq : nx;                              // knots of the split axis
        gptr<double> ks = (gptr<double>)(by_q ? md.aq.knots : md.ax.knots);
        const double *sp = by_q ? a.q : a.x;
        const bool square = by_q && a.q_is_q;

        // this workgroup's piece [ia, ib), and which of the `width` workgroups
        // that sweep it this one is
        int ia = 0, ib = ns - 1, piece = 0, part = place, width = a.team_size;
        int cut_lo = 0, cut_hi = ns - 1;                            // intervals held by any piece
        __syncthreads();   // the previous unit has left LDS
        if (plan.pieces > 1) {
            RouteCut *rc = reinterpret_cast<RouteCut *>(sm);
            double *kn = reinterpret_cast<double *>(sm + route_round16(sizeof(RouteCut)));
            if (a.cuts) {
                // made by route_cut_kernel
                gptr<int> g = (gptr<int>)(a.cuts + m);
                if (tid < (int)(sizeof(RouteCut) / 4))
                    reinterpret_cast<int *>(rc)[tid] = g[tid];
                __syncthreads();
            } else {
                make_cut<BLOCK>(rc, kn, reinterpret_cast<int *>(kn + ns), ns, plan.most,
                                a.team_size, [&](int i) { return ks[i]; },
                                [&](int k) {
                                    const double v = sp[k * a.n / kRouteSamples];
                                    return square ? v * v : v;
                                });
            }
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
        // points of the piece: s_lo <= v < s_hi, without a bound at an end of
        // the axis (the lower end's piece takes NaN); piece 0 also takes the
        // points outside every piece
        const bool first = ia == 0, last = ib == ns - 1;
        const double s_lo = ks[ia], s_hi = last ? __builtin_inf() : ks[ib];
        const bool far_lo = piece == 0 && cut_lo > 0, far_hi = piece == 0 && cut_hi < ns - 1;
        const bool far_any = far_lo || far_hi;
        const double f_hi = far_hi ? ks[cut_hi] : __builtin_inf();

        // knots [w0, w0 + wn) of the split axis are in LDS
        auto start = [&](int i) { return i - 1 < 0 ? 0 : i - 1 > ns - 4 ? ns - 4 : i - 1; };
        const int w0 = start(ia), wn = start(ib - 1) + 4 - w0;
        const int x0 = by_q ? 0 : w0, xn = by_q ? nx : wn;
        const int q0 = by_q ? w0 : 0, qn = by_q ? wn : nq;
        const int nodes = xn * qn;
        const int plane = nodes * 16;                               // bytes of a full plane

        // values: wave by (row, x), lanes over Q^2
        const V *const src = reinterpret_cast<const V *>(F32 ? md.vals32 : md.vals64);
        const int rs = a.raw ? nq : nq + 2;
        const size_t fs = a.raw ? (size_t)nx * nq : (size_t)(F32 ? md.slab32 : md.slab64);
        const size_t o0 = a.raw ? 0 : (size_t)rs + 1;
        // (H rows of four x values at once, so that as many loads are in flight: 101 members
        // of 200003 points FP64 1131 us with 2, 1103 with 4; the FP64 instance with alpha_s
        // loses 2% of its 10 million points to what 4 does to its registers)
        constexpr int H = F32 || !AS ? 4 : 2;
        const int urow = lane < n_u ? a.urow[lane] : 0;
        for (int u = 0; u < n_u; u += H) {
            gptr<V> g[H];
            int dst[H], step[H];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int uh = min(u + h, n_u - 1);
                g[h] = (gptr<V>)(src + (size_t)__builtin_amdgcn_readlane(urow, uh) * fs + o0 +
                                 (size_t)x0 * rs + q0);
                dst[h] = (uh / G) * plane + (uh % G) * (int)sizeof(V);
                step[h] = uh >= full * G ? tail : 16;
            }
            for (int i0 = wave; i0 < xn; i0 += 4 * WAVES)
                for (int k = lane; k < qn; k += 64) {
                    V v[H][4];
#pragma unroll
                    for (int h = 0; h < H; ++h)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int i = i0 + j * WAVES;
                            v[h][j] = g[h][(i < xn ? i : i0) * rs + k];
                        }
#pragma unroll
                    for (int h = 0; h < H; ++h)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int i = i0 + j * WAVES;
                            if (i < xn)
                                *reinterpret_cast<V *>(sm + dst[h] + (i * qn + k) * step[h]) =
                                    v[h][j];
                        }
                }
        }
        int off = route_round16(full * plane + nodes * tail);
        const PieceAxis px = place_axis(sm, off, md.ax, by_q ? 0 : ia, by_q ? nx - 1 : ib - ia);
        const PieceAxis pq = place_axis(sm, off, md.aq, by_q ? ia : 0, by_q ? ib - ia : nq - 1);
        {
            const PieceAxis both[2] = {px, pq};
            const AxisDev *const axes[2] = {&md.ax, &md.aq};
            load_axes<F32>(both, axes, BLOCK);
        }
        const V *asv = reinterpret_cast<const V *>(sm + off) + 1;   // padded by one on each side
        if constexpr (AS) {
            gptr<V> gv = (gptr<V>)a.as_vals;
            for (int i = tid; i < nq + 2; i += BLOCK)
                reinterpret_cast<V *>(sm + off)[i] = gv[i];
        }
        __syncthreads();

        V *const out = reinterpret_cast<V *>(a.out) + ((int64_t)m * a.n + p0) * n_u;
        const double *const xp = a.x + p0, *const qp = a.q + p0, *const spp = sp + p0;
        const int ntile = (npts + 63) / 64;
        const int stride = width * WAVES;

        // Domain rule for the point (x, Q^2); x f is defined (ok), alpha_s is (q_ok).
        auto admit = [&](double &xv, double &qv, bool &q_ok) {
            const bool x_in = xv >= px.lo && xv <= px.hi;   // false for NaN
            const bool q_in = qv >= pq.lo && qv <= pq.hi;
            bool ok = x_in && q_in;
            q_ok = true;
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
            return ok;
        };
        auto alphas = [&](int rel, bool live, bool q_ok, int sq, const V wq[4]) {
            const V *av = asv + sq;
            V s = wq[0] * av[0];
            s = fma(wq[1], av[1], s);
            s = fma(wq[2], av[2], s);
            s = fma(wq[3], av[3], s);
            if (live)
                reinterpret_cast<V *>(a.as_out)[p0 + rel] = q_ok ? s : fwd::quiet_nan<V>();
        };

        // Tiles of 64 points t, t + stride, ... of this wave, scanned kRouteScan at
        // a time; bit k of `bits` tells that the lane's point of the k-th tile is
        // the piece's.  The next tiles' coordinates are loaded ahead (vn, `raw`
        // until they are made into bits).
        const int t_first = part * WAVES + wave;
        int t_load = t_first, t_use = t_first, held = 0;
        double vn[kRouteScan];
        unsigned int bits = 0, bits_next = 0;
        bool raw = false, far_seen = false;
        auto load_tiles = [&]() {
            const int lane = fresh_lane();
#pragma unroll
            for (int k = 0; k < kRouteScan; ++k) {
                const int rel = (t_load + k * stride) * 64 + lane;
                vn[k] = spp[rel < npts ? rel : npts - 1];
            }
            raw = true;
        };
        auto is_far = [&](double v) { return (far_lo && !(v >= s_lo)) || (far_hi && v >= f_hi); };
        auto make_bits = [&]() {
            const int lane = fresh_lane();
            bits_next = 0;
#pragma unroll
            for (int k = 0; k < kRouteScan; ++k) {
                const int rel = (t_load + k * stride) * 64 + lane;
                double v = vn[k];
                if (square)
                    v = v * v;
                if (rel < npts && (first || v >= s_lo) && !(v >= s_hi))
                    bits_next |= 1u << k;
                if (far_any)
                    far_seen = far_seen || is_far(v);
            }
            raw = false;
        };
        // The points waiting: lanes [0, n_wait) of `wait`, and past 64 those of `over`.
        int n_wait = 0, wait = 0, over = 0;
        // The next batch of 64; its coordinates are loaded at once.
        int b_n = 0, b_rel = 0;
        double b_x = 0.0, b_q = 0.0;
        auto next_batch = [&]() {
            const int lane = fresh_lane();
            while (n_wait < 64 && (held > 0 || t_load < ntile)) {
                if (held == 0) {
                    if (raw)
                        make_bits();
                    bits = bits_next;
                    t_use = t_load;
                    held = kRouteScan;
                    t_load += kRouteScan * stride;
                    if (t_load < ntile)
                        load_tiles();
                }
                const bool sel = bits & 1u;
                const unsigned long long mask = __ballot(sel);
                if (mask != 0ull) {
                    // the tile's points go to the lanes after those waiting, the
                    // other lanes fill up
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
            b_x = xp[b_rel];
            b_q = qp[b_rel];
        };
        if (t_load < ntile)
            load_tiles();
        next_batch();
        while (b_n > 0) {
            const int lane = fresh_lane();
            const int n_now = b_n, rel = b_rel;
            const bool live = lane < n_now;
            double xv = b_x, qv = b_q;
            next_batch();
            if (a.q_is_q)
                qv = qv * qv;
            bool q_ok;
            const bool ok = admit(xv, qv, q_ok);
            fwd::count_flagged(live && !ok, a.dom_count);
            if constexpr (AS)
                fwd::count_flagged(live && !q_ok, a.dom_count);
            const double lnx = ln(xv), lnq = ln(qv);
            V wx[4], wq[4];
            const int ix = piece_bin(px, xv, lnx);
            const int kq = piece_bin(pq, qv, lnq);
            piece_weights<V>(px, ix, lnx, wx);
            piece_weights<V>(pq, kq, lnq, wq);
            const int sx = window4(ix + px.a, nx, wx);
            const int sq = window4(kq + pq.a, nq, wq);
            // a point outside the grid: NaN weights make all its values NaN
#pragma unroll
            for (int k = 0; k < 4; ++k)
                wx[k] = ok ? wx[k] : fwd::quiet_nan<V>();
            // The loads ahead are waited for here, before this batch's stores:
            // memory operations complete in order, and a wait for a load that was
            // issued after them would wait for the stores as well.
            asm volatile("" : "+v"(b_x), "+v"(b_q));
            if (raw)
                make_bits();
            if constexpr (AS)
                alphas(rel, live, q_ok, sq, wq);
            const int node = (sx - x0) * qn + (sq - q0);
            const char *p = sm + node * 16;
            // C planes side by side: each row's C * 16 bytes leave from C
            // neighbouring lanes in one store, a quarter (C = 4) of the line
            // requests of a store of 16 bytes per lane and row
            auto planes = [&](int g, auto cc) {
                constexpr int C = decltype(cc)::value;
                uint4 c[C];
#pragma unroll
                for (int j = 0; j < C; ++j, p += plane) {
                    V acc[G];
                    plane_stencil<V, G>(p, qn * 16, wx, wq, acc);
                    __builtin_memcpy(&c[j], acc, 16);
                    asm volatile("" ::: "memory");
                }
                if constexpr (C >= 2)
#pragma unroll
                    for (int j = 0; j < C; j += 2)
                        swap_pieces<1>(lane, c[j], c[j + 1]);
                if constexpr (C == 4) {
                    swap_pieces<2>(lane, c[0], c[2]);
                    swap_pieces<2>(lane, c[1], c[3]);
                }
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    // row of the j-th of the C lanes, piece of this lane
                    int rj = rel;
                    if constexpr (C == 2)
                        rj = j ? quad_lane<0xF5>(rel) : quad_lane<0xA0>(rel);
                    else if constexpr (C == 4)
                        rj = j == 0   ? quad_lane<0x00>(rel)
                             : j == 1 ? quad_lane<0x55>(rel)
                             : j == 2 ? quad_lane<0xAA>(rel)
                                      : quad_lane<0xFF>(rel);
                    V v[G];
                    __builtin_memcpy(v, &c[j], 16);
                    if ((lane & ~(C - 1)) + j < n_now)
                        store_values<G>(out + (int64_t)rj * n_u + (g + (lane & (C - 1))) * G, v);
                }
            };
            int g = 0;
            for (; g + 4 <= full; g += 4)
                planes(g, std::integral_constant<int, 4>{});
            if (g + 2 <= full) {
                planes(g, std::integral_constant<int, 2>{});
                g += 2;
            }
            if (g < full)
                planes(g, std::integral_constant<int, 1>{});
            if (tail) {
                const int u0 = full * G, left = n_u - u0;
                V *const row = out + (int64_t)rel * n_u + u0;
                V acc[G];
                p = sm + full * plane + node * tail;
                if (left == 1) {
                    plane_stencil<V, 1>(p, qn * tail, wx, wq, acc);
                    if (live)
                        store_values<1>(row, acc);
                } else if constexpr (F32) {
                    if (left == 2) {
                        plane_stencil<V, 2>(p, qn * tail, wx, wq, acc);
                        if (live)
                            store_values<2>(row, acc);
                    } else {
                        plane_stencil<V, 4>(p, qn * tail, wx, wq, acc);
                        if (live)
                            store_values<3>(row, acc);
                    }
                }
            }
        }

        // Points outside every piece (the sample held none): again over the
        // tiles of this wave, straight from the values in global memory.
        if (far_any && __ballot(far_seen) != 0ull) {
            int m_far = m;
            asm volatile("" : "+s"(m_far));   // read again: its tables are not kept till here
            const MemberDev md = member(a, m_far);
            const int nx = md.nx, nq = md.nq;
            const V *const src = reinterpret_cast<const V *>(F32 ? md.vals32 : md.vals64);
            const int rs = a.raw ? nq : nq + 2;
            const size_t fs = a.raw ? (size_t)nx * nq : (size_t)(F32 ? md.slab32 : md.slab64);
            const size_t o0 = a.raw ? 0 : (size_t)rs + 1;
            for (int t = t_first; t < ntile; t += stride) {
                const int rel = t * 64 + lane;
                double v = spp[rel < npts ? rel : npts - 1];
                if (square)
                    v = v * v;
                if (rel >= npts || !is_far(v))
                    continue;
                double xv = xp[rel], qv = qp[rel];
                if (a.q_is_q)
                    qv = qv * qv;
                bool q_ok;
                const bool ok = admit(xv, qv, q_ok);
                const int flags = (ok ? 0 : 1) + (AS && !q_ok ? 1 : 0);
                if (flags)   // only some lanes are here
                    atomicAdd(a.dom_count, (unsigned long long)flags);
                const double lnx = ln(xv), lnq = ln(qv);
                V wx[4], wq[4];
                const int ix = far_weights<V>(md.ax, xv, lnx, wx);
                const int kq = far_weights<V>(md.aq, qv, lnq, wq);
                const int sx = window4(ix, nx, wx);
                const int sq = window4(kq, nq, wq);
                if constexpr (AS)
                    alphas(rel, true, q_ok, sq, wq);
                gptr<V> g0 = (gptr<V>)(src + o0 + (size_t)sx * rs + sq);
                for (int u = 0; u < n_u; ++u) {
                    gptr<V> g = g0 + (size_t)a.urow[u] * fs;
                    V acc = V(0);
#pragma unroll
                    for (int jx = 0; jx < 4; ++jx, g += rs) {
                        V r = V(0);
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            r = (k == 0) ? wq[0] * g[0] : fma(wq[k], g[k], r);
                        acc = (jx == 0) ? wx[0] * r : fma(wx[jx], r, acc);
                    }
                    out[(int64_t)rel * n_u + u] = ok ? acc : fwd::quiet_nan<V>();
                }
            }
        }
    }
}

// The cut of every member of a set, one workgroup each: a team evaluates many
// members in turn, and would make each one's cut anew (9 us a member).
template <int VS>
__global__ __launch_bounds__(kRouteBlock<double>) void route_cut_kernel(const RouteArgs a)
{
    extern __shared__ uint4 smem4[];
    char *sm = reinterpret_cast<char *>(smem4);
    const MemberDev md = member(a, blockIdx.x);
    const RoutePlan plan = route_plan(md.nx, md.nq, md.ax.nbuckets, md.aq.nbuckets, a.n_u, VS, 0);
    const int ns = plan.split ? md.nq : md.nx;
    if (plan.pieces < 2)
        return;
    RouteCut *rc = reinterpret_cast<RouteCut *>(sm);
    double *kn = reinterpret_cast<double *>(sm + route_round16(sizeof(RouteCut)));
    gptr<double> ks = (gptr<double>)(plan.split ? md.aq.knots : md.ax.knots);
    const double *sp = plan.split ? a.q : a.x;
    make_cut<kRouteBlock<double>>(rc, kn, reinterpret_cast<int *>(kn + ns), ns, plan.most,
                                  a.team_size, [&](int i) { return ks[i]; },
                                  [&](int k) { return sp[k * a.n / kRouteSamples]; });
    if (threadIdx.x < sizeof(RouteCut) / 4)
        reinterpret_cast<int *>(a.cuts + blockIdx.x)[threadIdx.x] =
            reinterpret_cast<const int *>(rc)[threadIdx.x];
}

template <typename V, bool AS>
hipError_t go(const RouteArgs &a, hipStream_t s)
{
    auto fn = xfx_route_kernel<V, AS>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kLdsLimit);
    if (e != hipSuccess)
        return e;
    if (a.cuts) {
        // ns doubles and ns ints of the longest axis, as loaded (4096 knots at most)
        const size_t lds = route_round16(sizeof(RouteCut)) + (size_t)a.longest * 12;
        hipLaunchKernelGGL((route_cut_kernel<(int)sizeof(V)>), dim3((unsigned)a.n_mem),
                           dim3(kRouteBlock<double>), lds, s, a);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)(a.teams * a.team_size)), dim3(kRouteBlock<V>), kLdsLimit,
                       s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_route(const RouteArgs &a, bool f32, hipStream_t s)
{
    if (a.as_out)
        return f32 ? go<float, true>(a, s) : go<double, true>(a, s);
    return f32 ? go<float, false>(a, s) : go<double, false>(a, s);
}

}  // namespace pdfx
