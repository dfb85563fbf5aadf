// Double-double arithmetic: unevaluated sums hi + lo with |lo| <= ulp(hi) / 2
// (about 32 digits).  Plain functions of their arguments, so a host compiler
// can build this header too (with __device__ and __forceinline__ defined and
// dd_rcp, an estimate of a reciprocal, given).
//
// Errors, in units of 2^-106 of the magnitudes that enter, over random
// operands against 113 bits (mean, largest); in brackets the same for the
// forms with every operation renormalised (accurate add, three quotients):
//   dvd    0.18, 1.4  (0.22, 1.8)      mac2   0.17, 2.9  (0.21, 2.7)
//   sub_q  0.16, 2.3  (0.17, 2.6)      32 terms by mac2  0.18, 2.9  (0.20, 3.3)
// Low words added in plain FP64 instead (two quotients, one normalisation per
// sum) cost 1.3 to 4.8 times the brackets' means and are not used.
#pragma once

#include <cmath>

#pragma clang fp contract(off)

#ifdef __HIPCC__
__device__ __forceinline__ double dd_rcp(double q) { return __builtin_amdgcn_rcp(q); }
#endif

struct dd {
    double hi, lo;
};

__device__ __forceinline__ dd mk(double a) { return {a, 0.0}; }
__device__ __forceinline__ dd quick_two_sum(double a, double b) {
    const double s = a + b;
    return {s, b - (s - a)};
}
__device__ __forceinline__ dd two_sum(double a, double b) {
    const double s = a + b;
    const double bb = s - a;
    return {s, (a - (s - bb)) + (b - bb)};
}
__device__ __forceinline__ dd two_prod(double a, double b) {
    const double p = a * b;
    return {p, __builtin_fma(a, b, -p)};
}
// The error-free sums do not depend on the order of their operands, so
// add(a, b) and add(b, a) are the same bits.
__device__ __forceinline__ dd add(dd a, dd b) {
    dd s = two_sum(a.hi, b.hi);
    const dd t = two_sum(a.lo, b.lo);
    s.lo += t.hi;
    s = quick_two_sum(s.hi, s.lo);
    s.lo += t.lo;
    return quick_two_sum(s.hi, s.lo);
}
__device__ __forceinline__ dd neg(dd a) { return {-a.hi, -a.lo}; }
__device__ __forceinline__ dd sub(dd a, dd b) { return add(a, neg(b)); }
__device__ __forceinline__ dd mul(dd a, dd b) {
    dd p = two_prod(a.hi, b.hi);
    const double c = a.hi * b.lo;
    const double d = a.lo * b.hi;
    p.lo += c + d;
    return quick_two_sum(p.hi, p.lo);
}
__device__ __forceinline__ dd mul_d(dd a, double b) {
    dd p = two_prod(a.hi, b);
    p.lo += a.lo * b;
    return quick_two_sum(p.hi, p.lo);
}
// 1 / q to the last place or so: hardware reciprocal, two Newton steps
__device__ __forceinline__ double recip1(double q) {
    double r = dd_rcp(q);
    r = __builtin_fma(r, __builtin_fma(-q, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-q, r, 1.0), r);
}
// a / b: the first quotient corrected to the last place, so that its remainder
// is exact in one FMA; the rest of the remainder as a two-sum, and a third
// quotient of what the second leaves.
__device__ __forceinline__ dd dvd(dd a, dd b) {
    const double r = recip1(b.hi);
    double q1 = a.hi * r;
    q1 = __builtin_fma(__builtin_fma(-q1, b.hi, a.hi), r, q1);
    const dd rem = two_sum(__builtin_fma(-q1, b.hi, a.hi), __builtin_fma(-q1, b.lo, a.lo));
    const double q2 = rem.hi * r;
    const double rem2 = __builtin_fma(-q2, b.hi, rem.hi) + __builtin_fma(-q2, b.lo, rem.lo);
    const dd q = quick_two_sum(q1, q2);
    return quick_two_sum(q.hi, __builtin_fma(rem2, r, q.lo));
}
__device__ __forceinline__ dd dsqrt(dd a) {
    if (!(a.hi > 0.0)) return mk(a.hi == 0.0 ? 0.0 : NAN);
    const double x = 1.0 / sqrt(a.hi);
    const double ax = a.hi * x;
    const dd e = sub(a, two_prod(ax, ax));
    return two_sum(ax, e.hi * (x * 0.5));
}
// s + a b + c d: the high words' sums and products are error-free, their low
// words go in first (they are the larger), then s.lo and the cross products,
// each group renormalised.  32 operations where two products and two accurate
// sums take 58.
__device__ __forceinline__ dd mac2(dd s, dd a, dd b, dd c, dd d) {
    const dd p = two_prod(a.hi, b.hi), q = two_prod(c.hi, d.hi);
    const dd t = two_sum(s.hi, p.hi), u = two_sum(t.hi, q.hi);
    const double cross = __builtin_fma(a.hi, b.lo, __builtin_fma(a.lo, b.hi, __builtin_fma(c.hi, d.lo, c.lo * d.hi)));
    const dd r = quick_two_sum(u.hi, (t.lo + u.lo) + (p.lo + q.lo));
    return quick_two_sum(r.hi, r.lo + (s.lo + cross));
}
// (d - x) - q for a double x
__device__ __forceinline__ dd sub_q(dd d, double x, dd q) {
    const dd t = two_sum(d.hi, -x), u = two_sum(t.hi, -q.hi);
    const dd r = quick_two_sum(u.hi, t.lo + u.lo);
    return quick_two_sum(r.hi, r.lo + (d.lo - q.lo));
}
__device__ __forceinline__ double to_d(dd a) { return a.hi + a.lo; }
