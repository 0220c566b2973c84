// Conflict-free order for LDS scatters of 4 x 4 windows.
//
// The 16 adds of a point go to a window of 4 x 4 knots anywhere on the grid; lanes
// that make them in the same order hit random banks together.  Here the knots are
// laid out in 4 x 4 blocks of 16 words, so that every window holds each of the 16
// word positions of a block exactly once, and lane l makes its s-th add at the word
// position s ^ (l mod 16): any 16 neighbouring lanes then hit 16 different
// positions.  Integer sums do not depend on the order, so it may differ from lane
// to lane.  8-byte adds on MI355X: 3.5e12 a second at random windows in a common
// order, 5.8e12 in this one.
#pragma once

#include "xfx_fwd_impl.h"

namespace pdfx {

// Layout of an na x nb grid (axis a: x, or Q^2 if `swapped`): word of knot (a, b) =
// (a / 4) * strip + b * 4 + a mod 4.  The word positions of a window are all
// different if strip is a multiple of 16; where that takes too much room strip is
// 4 nb and windows across two strips meet other lanes' words at times.
struct BlockLayout {
    int na, nb, strip, words;
    bool swapped;
};

// The layout of an nx x nq grid in at most `room` words: padded to whole blocks if
// that fits, else with strips along the axis that takes less room.
inline BlockLayout block_layout(int nx, int nq, int room)
{
    auto up = [](int n) { return (n + 3) / 4 * 4; };
    if (up(nx) * up(nq) <= room)
        return BlockLayout{nx, nq, 4 * up(nq), up(nx) * up(nq), false};
    const bool swapped = nx * up(nq) < up(nx) * nq;
    const int na = swapped ? nq : nx, nb = swapped ? nx : nq;
    return BlockLayout{na, nb, 4 * nb, up(na) * nb, swapped};
}

__device__ __forceinline__ int block_word(const BlockLayout &y, int ix, int kq)
{
    const int a = y.swapped ? kq : ix, b = y.swapped ? ix : kq;
    return (a >> 2) * y.strip + b * 4 + (a & 3);
}

// c ? b : a, as the one conditional move a word that it is: written as an expression,
// chains of such selects over small arrays turn into indexed reads, several times
// as long.  mask: the lanes where c holds.
__device__ __forceinline__ double pick(double a, double b, unsigned long long mask)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    unsigned lo, hi;
    asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(lo) : "v"((unsigned)ua), "v"((unsigned)ub), "s"(mask));
    asm("v_cndmask_b32 %0, %1, %2, %3"
        : "=v"(hi)
        : "v"((unsigned)(ua >> 32)), "v"((unsigned)(ub >> 32)), "s"(mask));
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}

// First knot of the window of interval i on an axis of n >= 4 knots.
__device__ __forceinline__ int visit_start(int i, int n)
{
    return min(max(i - 1, 0), n - 4);
}

// The weights w of knots i-1 .. i+2 in the order in which a lane with key l visits the
// positions of interval i's window: o[s] is the weight of the knot at position s ^ l,
// w[((s ^ l) - (i - 1)) mod 4].  At either end of the axis the window starts a knot
// later or earlier; the knot it has instead is congruent to the one outside, whose
// weight is 0.
__device__ __forceinline__ void visit_weights(const double w[4], int i, int l, double o[4])
{
    const int r = i - 1;
    const unsigned long long odd = __ballot(r & 1), flip = __ballot(l & 1),
                             half = __ballot(((r >> 1) ^ (l >> 1)) & 1);
    double t[4], u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        t[k] = pick(w[k], w[(k + 3) & 3], odd);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        u[k] = pick(t[k], t[k ^ 1], flip);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        o[k] = pick(u[k], u[k ^ 2], half);
}

// Byte offsets of a window's rows (along axis a, from a0) and columns (from b0) in
// the order of lane key l, for words of UNIT bytes: the add at (i, j) goes to
// row[i] + col[j].
template <int UNIT>
__device__ __forceinline__ void visit_rows(int a0, int strip, int l, int row[4])
{
    const int far = strip * UNIT, base = (a0 >> 2) * far, r = a0 & 3;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int k = s ^ (l & 3);
        row[s] = base + k * UNIT + (k < r ? far : 0);
    }
}
template <int UNIT>
__device__ __forceinline__ void visit_cols(int b0, int l, int col[4])
{
    const int base = (b0 >> 2) * (16 * UNIT), r = b0 & 3;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int k = s ^ ((l >> 2) & 3);
        col[s] = base + k * (4 * UNIT) + (k < r ? 16 * UNIT : 0);
    }
}

// The 64-bit LDS word at byte offset row + col of base, its address kept in one
// register (it would be formed anew at every add).
typedef __attribute__((address_space(3))) unsigned long long LdsWord;
__device__ __forceinline__ LdsWord *visit_word(unsigned long long *base, int row, int col)
{
    LdsWord *w = reinterpret_cast<LdsWord *>(reinterpret_cast<__attribute__((address_space(3))) char *>(
                                                 (LdsWord *)base) +
                                             (row + col));
    asm volatile("" : "+v"(w));
    return w;
}

// The two constants of an interval that its folded weights need (the others follow:
// ql and qr are 1/2 inside the subgrid and 1 at its ends, where pl or pr is 0).
struct FoldPair {
    double pl, pr;
};
__device__ __forceinline__ void fold_pair(double t, const FoldPair &c, double w[4])
{
    const double ql = c.pl != 0.0 ? 0.5 : 1.0, qr = c.pr != 0.0 ? 0.5 : 1.0;
    fwd::fold<double>(t, c.pl, c.pl - ql, ql, qr, qr - c.pr, c.pr, w);
}

}  // namespace pdfx
