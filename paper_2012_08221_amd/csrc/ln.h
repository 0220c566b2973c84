// Natural logarithm of a coordinate inside its axis' range (positive and finite).
//
// The library's log takes 93 vector instructions in FP64, 44 of them additions that keep
// every step in two words, and a point needs two or three of them: half of alpha_s, two
// fifths of the luminosity at one Q^2, a fifth of the routed forward kernel.  Here (46)
// only what is as large as the result is kept exactly: with x = 2^k m, m in [sqrt(1/2),
// sqrt(2)), f = m - 1 and s = f / (2 + f),
//   ln x = k ln 2 + f - f^2/2 + s (f^2/2 + R),   R = 2 (s^2/3 + s^4/5 + s^6/7 + ...),
// the first three terms summed without error into two words and the last, below 1/20,
// rounded.  R / s^2 is a polynomial in s^2 that interpolates it at 8 Chebyshev points of
// [0, (3 - 2 sqrt 2)^2] (error 1e-19).  Against 80-bit arithmetic over [1e-9, 1e10]: at
// most 0.635 ulp, 1.1 % of the results near 1 not the nearest double (the library's:
// 0.640 ulp, 5.8 %).
#pragma once

#include <hip/hip_runtime.h>

namespace pdfx {

__device__ __forceinline__ double ln(double x)
{
#pragma clang fp contract(off)   // the sums in two words need the products rounded
    double m = __builtin_amdgcn_frexp_mant(x);   // [1/2, 1)
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0.70710678118654752440;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double k = (double)e, f = m - 1.0, d = m + 1.0;
    // s = f / d, to about an ulp
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    double s = f * r;
    s = fma(fma(-s, d, f), r, s);
    const double z = s * s;
    double p = 0.13086767009948175;
    p = fma(p, z, 0.13268759668560612);
    p = fma(p, z, 0.15386240205813478);
    p = fma(p, z, 0.18181795630884753);
    p = fma(p, z, 0.2222222239180047);
    p = fma(p, z, 0.28571428570803231);
    p = fma(p, z, 0.40000000000000879);
    p = fma(p, z, 0.66666666666666663);
    // ln 2 in two words, the first short enough for k ln2_hi to be exact
    const double ln2_hi = 0x1.62e42fefa38p-1, ln2_lo = 0x1.ef35793c7673p-45;
    const double h = 0.5 * f, q = h * f, ql = fma(h, f, -q);
    const double c = fma(s, fma(z, p, q), fma(k, ln2_lo, -ql));
    const double a = k * ln2_hi;
    const double t = a + f, tl = f - (t - a);   // |a| > |f| or a = 0
    const double u = t - q, ul = (t - u) - q;
    return u + (tl + (ul + c));
}

}  // namespace pdfx
