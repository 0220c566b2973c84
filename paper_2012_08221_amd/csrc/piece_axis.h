// Parts of the kernels that keep a piece of the grid in LDS: the search tables of a
// part of an axis, bins, folded weights, windows and stencils, and the cut of an
// axis into pieces.
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
template <bool F32>
__device__ __forceinline__ void load_axes(const PieceAxis (&p)[2], const AxisDev *const (&ax)[2],
                                          int block)
{
    const int most = max(max(p[0].cnt + 1, p[0].nb / 2), max(p[1].cnt + 1, p[1].nb / 2));
    for (int i = threadIdx.x; i < most; i += block) {
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

// The lane, recomputed where it is used: what is derived from it is then not
// kept in registers across the loops, which have none to spare.
__device__ __forceinline__ int fresh_lane()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// K values of V side by side in LDS.
template <typename V, int K>
__device__ __forceinline__ void lds_values(const char *p, V v[K])
{
    if constexpr (sizeof(V) * K == 16) {
        const uint4 d = *reinterpret_cast<const uint4 *>(p);
        __builtin_memcpy(v, &d, 16);
    } else if constexpr (sizeof(V) * K == 8) {
        const uint2 d = *reinterpret_cast<const uint2 *>(p);
        __builtin_memcpy(v, &d, 8);
    } else {
        v[0] = *reinterpret_cast<const V *>(p);
    }
}

// 16-tap stencil of the K rows of one plane at node address p (bytes), rows
// row_bytes apart.
template <typename V, int K>
__device__ __forceinline__ void plane_stencil(const char *p, int row_bytes, const V wx[4],
                                              const V wq[4], V acc[K])
{
    constexpr int NB = (int)sizeof(V) * K;
#pragma unroll
    for (int jx = 0; jx < 4; ++jx) {
        V r[K];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            V v[K];
            lds_values<V, K>(p + jx * row_bytes + k * NB, v);
#pragma unroll
            for (int g = 0; g < K; ++g)
                r[g] = (k == 0) ? wq[0] * v[g] : fma(wq[k], v[g], r[g]);
        }
#pragma unroll
        for (int g = 0; g < K; ++g)
            acc[g] = (jx == 0) ? wx[0] * r[g] : fma(wx[jx], r[g], acc[g]);
        // eight reads in flight a wave: with 16 waves that fills the LDS pipe, and
        // sixteen would not fit the 128 registers
        if (jx == 1)
            asm volatile("" ::: "memory");
    }
}

// The lane's register of another lane of its quad.
template <int CTRL>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, true);
}

// Exchanges between lanes l and l ^ D (D = 1, 2) the 16-byte pieces c0 of the
// lanes with that bit set against the c1 of the others.
template <int D>
__device__ __forceinline__ void swap_pieces(int lane, uint4 &c0, uint4 &c1)
{
    constexpr int CTRL = D == 1 ? 0xB1 : 0x4E;   // quad_perm [1,0,3,2], [2,3,0,1]
    const bool up = lane & D;
    auto one = [&](uint32_t &a, uint32_t &b) {
        const uint32_t fa = quad_lane<CTRL>(a), fb = quad_lane<CTRL>(b);
        a = up ? fb : a;
        b = up ? b : fa;
    };
    one(c0.x, c1.x);
    one(c0.y, c1.y);
    one(c0.z, c1.z);
    one(c0.w, c1.w);
}

// Shares team_size workgroups among the pieces by weight w (one lane per
// piece, pieces <= team_size): at least one each, the others to the piece with
// the largest weight per workgroup.  Returns the lane's number.
__device__ __forceinline__ int share_out(float w, int pieces, int team_size)
{
    const int lane = threadIdx.x & 63;
    float sum = lane < pieces ? w : 0.f;
    for (int d = 32; d; d >>= 1)
        sum += __shfl_xor(sum, d);
    int mine = lane < pieces ? (int)(w / sum * (float)team_size) : 0;
    if (lane < pieces && mine < 1)
        mine = 1;
    int total = mine;
    for (int d = 32; d; d >>= 1)
        total += __shfl_xor(total, d);
    // too many (pieces raised to one): from the lightest load; too few: to the heaviest
    while (total != team_size) {
        const bool more = total < team_size;
        float key = -1.f;
        if (lane < pieces)
            key = more ? w / (float)mine : (mine > 1 ? 1.f / (w / (float)(mine - 1) + 1e-30f) : -1.f);
        int at = lane;
        for (int d = 32; d; d >>= 1) {
            const float k2 = __shfl_xor(key, d);
            const int a2 = __shfl_xor(at, d);
            if (k2 > key || (k2 == key && a2 < at)) {
                key = k2;
                at = a2;
            }
        }
        if (lane == at)
            mine += more ? 1 : -1;
        total += more ? 1 : -1;
    }
    return mine;
}

constexpr int kRouteSamples = 1024;

// Makes the cut of an axis of ns knots for pieces of at most `most` intervals.
// knot(i): the i-th knot; sample(k): the k-th sampled point's coordinate, on the
// same scale.  kn, cum: LDS for ns doubles and ns ints.  Every workgroup of the
// team makes the same cut from the same samples.
template <int BLOCK, typename Knot, typename Sample>
__device__ __forceinline__ void make_cut(RouteCut *rc, double *kn, int *cum, int ns, int most,
                                         int team_size, Knot knot, Sample sample)
{
    constexpr int S = kRouteSamples, PER = (S + BLOCK - 1) / BLOCK;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // nothing of this is kept in registers beyond it
    const int lane = tid & 63;
    const int ni = ns - 1;
    double v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k)
        v[k] = sample(min(k * BLOCK + tid, S - 1));
    for (int i = tid; i < ns; i += BLOCK) {
        kn[i] = knot(i);
        cum[i] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (k * BLOCK + tid >= S)
            break;
        const double u = v[k];
        int lo = 0, hi = ni;              // interval in [lo, hi)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (u >= kn[mid])
                lo = mid;
            else
                hi = mid;
        }
        atomicAdd(&cum[lo], 1);
    }
    __syncthreads();
    if (tid < 64) {
        // running sums: cum[i] = samples in intervals [0, i]
        const int per = (ni + 63) / 64;
        int own = 0;
        for (int i = lane * per; i < (lane + 1) * per && i < ni; ++i) {
            own += cum[i];
            cum[i] = own;
        }
        int incl = own;
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(incl, d);
            incl += lane >= d ? o : 0;
        }
        for (int i = lane * per; i < (lane + 1) * per && i < ni; ++i)
            cum[i] += incl - own;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // first interval with more than c samples up to and in it, or ni
        auto reach = [&](int c) {
            int lo = 0, hi = ni;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (cum[mid] > c)
                    hi = mid;
                else
                    lo = mid + 1;
            }
            return lo;
        };
        int a = reach(0), b = reach(S - 1) + 1;
        const int pieces = (b - a + most - 1) / most;
        // room left in the pieces goes to the intervals beyond, half to either side
        int spare = pieces * most - (b - a);
        const int down = min(a, max(spare / 2, spare - (ni - b)));
        a -= down;
        spare -= down;
        b += min(ni - b, spare);
        const int below = a > 0 ? cum[a - 1] : 0, inside = cum[b - 1] - below;
        // equal shares of the samples, as far as `most` allows
        int want = reach(below + (int)((int64_t)inside * lane / pieces) - 1) + 1;
        int cut = a;
        for (int k = 1; k < pieces; ++k) {
            const int prev = __shfl(cut, k - 1), w = __shfl(want, k);
            int c = max(w, max(prev + 1, b - (pieces - k) * most));
            c = min(c, min(prev + most, b - (pieces - k)));
            if (lane == k)
                cut = c;
        }
        if (lane >= pieces)
            cut = b;
        const int next = __shfl(cut, lane < 63 ? lane + 1 : 63);
        // a scan costs about 1/32 of an evaluation per point and piece
        const int held = lane < pieces ? cum[next - 1] - (cut > 0 ? cum[cut - 1] : 0) : 0;
        const int width = share_out((float)held + (float)S * (1.f / 32.f), pieces, team_size);
        if (lane < pieces) {
            rc->cut[lane] = cut;
            rc->width[lane] = width;
        }
        if (lane == 0) {
            rc->pieces = pieces;
            rc->cut[pieces] = b;
        }
    }
    __syncthreads();
}

}  // namespace piece
}  // namespace pdfx
