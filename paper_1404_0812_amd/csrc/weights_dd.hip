// Extended-precision (double-double) RBF-FD weights for target condition
// numbers beyond what FP64 resolves (Sec. 6.2 computes the weights for
// kappa_T up to 1e20 in quadruple precision and then steps in FP64).
//
// Same quantities as the FP64 path (Sec. 4, eq. surface_lap_P1: the first
// row of L_P = sum_d G^d G^d, formed as w = (A~^{-1} r)[:n] with
// r = sum_d (B^d)^T g_d, g_d = (A~^{-1} b_d)[:n]; Sec. 5: eps by bisection on
// kappa_2(A~) = max|lambda| / min|lambda|), for the paper's own local system:
// the constant border (a column of ones) and the multiquadric or inverse
// multiquadric kernel, with every quantity derived from the FP64 inputs
// carried as an unevaluated sum of two doubles (about 32 significant digits):
// coordinate differences (exact two-sums), squared distances, kernel values,
// unit normals, the Householder tridiagonalisation and Sturm counts behind
// kappa_2, and a pivoted LU factorisation for the solves.  Only the final
// weights, eps and kappa_2 are rounded to FP64.
//
// One wavefront per stencil.  While eps is searched the local matrix lives in
// registers, 32 FP64 words per lane for m = n + 1 <= 32: lane (c, h) holds the
// rows of parity h of column c, so that both halves of the wavefront work on
// every Householder step (m <= 48: lane c holds all of column c).  v and w of
// a step reach the rows through DPP row broadcasts.  The final LU works in
// LDS, in the space of the search's vectors.
//
// What bounds it: FP64 issue (two double-double products and their sum with a
// third value are 32 operations, see dd.h).  The matrix in 38 KB of LDS, every
// operation renormalised by itself, quotients of three divisions and 13
// eigenvalue passes per decision took 38.3 ms for 2562 stencils of 31 nodes to
// kappa_T = 1e18; now 6.3 ms (40962 stencils: 551 -> 84 ms; 1200 of 47 nodes:
// 33 -> 16 ms).  Low words summed in plain FP64 took 5.1 ms and were less
// accurate (MQ weights up to 1.09 times the former kernel's mean error); now,
// against 113-bit weights at the same eps, 28 sets of 642 stencils (11 to 47
// nodes, kappa 1e18 and 1e20) have 0.96 to 1.02 times its mean error, 0.99 over all.
#include "common.h"
#include "dd.h"
#include "weights_job.h"

#include <cmath>
#include <type_traits>

#pragma clang fp contract(off)

namespace {

constexpr int DD_MAX = 48;

template <int MM>
struct DDL {
    static constexpr int H = MM == 32 ? 2 : 1;    // lanes per column
    static constexpr int R = MM / H;              // rows per lane: H i + h, i = 0 .. R - 1
    static constexpr int BR = MM == 32 ? 4 : 16;  // rows per block of the reduction's code
    static constexpr int LDA = MM + 1;
};

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ dd dpp(dd v) {
    return {dpp<CTRL>(v.hi), dpp<CTRL>(v.lo)};
}
// v of lane I of the caller's row of 16 lanes
template <int I>
__device__ __forceinline__ double row_lane(double v) {
    double r = v;  // the builtin's type follows its operands
    r = __builtin_amdgcn_update_dpp(r, v, 0x150 + I, 0xf, 0xf, true);
    return r;
}
template <int I>
__device__ __forceinline__ dd row_lane(dd v) {
    return {row_lane<I>(v.hi), row_lane<I>(v.lo)};
}
__device__ __forceinline__ void swap16(double v, double& a, double& b) {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    a = __hiloint2double((int)h[0], (int)l[0]);
    b = __hiloint2double((int)h[1], (int)l[1]);
}
// a: the lower 32 lanes' value of v, b: the upper 32 lanes', in both halves
__device__ __forceinline__ void swap32(double v, double& a, double& b) {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    a = __hiloint2double((int)h[0], (int)l[0]);
    b = __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ void swap32(dd v, dd& a, dd& b) {
    swap32(v.hi, a.hi, b.hi);
    swap32(v.lo, a.lo, b.lo);
}
__device__ __forceinline__ dd halves_sum(dd v) {
    dd a, b;
    swap32(v, a, b);
    return add(a, b);
}
// Sum over the columns (each half of the wavefront holds all of them where
// H = 2), the same bits in every lane: two partners add the same two values,
// and add() does not depend on their order.
template <int MM>
__device__ __forceinline__ dd wsum(dd v) {
    v = add(v, dpp<0xB1>(v));   // quad_perm [1,0,3,2]
    v = add(v, dpp<0x4E>(v));   // quad_perm [2,3,0,1]
    v = add(v, dpp<0x141>(v));  // row_half_mirror
    v = add(v, dpp<0x140>(v));  // row_mirror
    dd a, b;
    swap16(v.hi, a.hi, b.hi);
    swap16(v.lo, a.lo, b.lo);
    if constexpr (DDL<MM>::H == 2) return add(a, b);
    else return halves_sum(add(a, b));
}

__device__ __forceinline__ void fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int MM>
struct DDShared {
    struct Search {
        double4 de[MM];  // d_i and e_{i-1}^2, high and low words
        double eh[MM];
        double ch[64], cl[64], vh[64], vl[64], wh[64], wl[64];  // pivot column, v, w
    };
    struct Factor {
        double ah[MM * DDL<MM>::LDA], al[MM * DDL<MM>::LDA];
    };
    union {
        Search f;
        Factor g;
    };
    double x[MM], y[MM], z[MM];
    double bh[4][MM], bl[4][MM];
    double n0h[3], n0l[3];  // the centre's unit normal
    int piv[MM];
};

__device__ __forceinline__ dd ld(const double* h, const double* l, int i) { return {h[i], l[i]}; }
__device__ __forceinline__ void st(double* h, double* l, int i, dd v) {
    h[i] = v.hi;
    l[i] = v.lo;
}
template <int MM>
__device__ __forceinline__ dd A(const DDShared<MM>& S, int r, int c) {
    return {S.g.ah[r * DDL<MM>::LDA + c], S.g.al[r * DDL<MM>::LDA + c]};
}
template <int MM>
__device__ __forceinline__ void setA(DDShared<MM>& S, int r, int c, dd v) {
    S.g.ah[r * DDL<MM>::LDA + c] = v.hi;
    S.g.al[r * DDL<MM>::LDA + c] = v.lo;
}

// x_i - x_j as an exact double-double, squared distance
template <int MM>
__device__ __forceinline__ void diff3(const DDShared<MM>& S, int i, int j, dd (&d)[3]) {
    d[0] = two_sum(S.x[i], -S.x[j]);
    d[1] = two_sum(S.y[i], -S.y[j]);
    d[2] = two_sum(S.z[i], -S.z[j]);
}
__device__ __forceinline__ dd norm2(const dd (&d)[3]) { return add(add(mul(d[0], d[0]), mul(d[1], d[1])), mul(d[2], d[2])); }

// phi and psi = phi'(r)/r from the squared distance (MQ: kernel 0, IMQ: 1)
template <int K>
__device__ __forceinline__ dd phi(dd e2, dd r2) {
    const dd t = add(mk(1.0), mul(e2, r2));
    const dd s = dsqrt(t);
    return K == RBFFD_KERNEL_MQ ? s : dvd(mk(1.0), s);
}
template <int K>
__device__ __forceinline__ dd psi(dd e2, dd r2) {
    const dd t = add(mk(1.0), mul(e2, r2));
    const dd s = dsqrt(t);
    return K == RBFFD_KERNEL_MQ ? dvd(e2, s) : neg(dvd(e2, mul(s, t)));
}

// Entry (r, c) of A~ = [[A, 1], [1^T, 0]] at eps^2 = e2
template <int K, int MM>
__device__ __forceinline__ dd entry(const DDShared<MM>& S, int n, int m, dd e2, int r, int c) {
    if (r < n && c < n) {
        dd d[3];
        diff3(S, r, c, d);
        return phi<K>(e2, norm2(d));
    }
    return mk(r < m && c < m && (r < n || c < n) ? 1.0 : 0.0);
}

// f(i) for the one constant i in [LO, HI) that equals the wave-uniform k
template <int LO, int HI, typename F>
__device__ __forceinline__ void at_row(int k, F&& f) {
    if constexpr (HI - LO == 1) {
        f(std::integral_constant<int, LO>{});
        // keeps the branches apart: merged, they would index the array dynamically
        asm volatile("; row %0" ::"n"(LO));
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (k < MID) at_row<LO, MID>(k, f);
        else at_row<MID, HI>(k, f);
    }
}
// f(i) for i = LO .. HI - 1 as constants
template <int LO, int HI, typename F>
__device__ __forceinline__ void each(F&& f) {
    if constexpr (LO < HI) {
        f(std::integral_constant<int, LO>{});
        each<LO + 1, HI>(f);
    }
}

// Row r of the register matrix at the lane's column, in every lane that has
// the column.
template <int MM>
__device__ __forceinline__ dd row_at(const dd (&a)[DDL<MM>::R], int r) {
    constexpr int H = DDL<MM>::H;
    dd v = mk(0.0);
    at_row<0, DDL<MM>::R>(r / H, [&](auto q) __attribute__((always_inline)) { v = a[decltype(q)::value]; });
    if constexpr (H == 2) {
        dd lo, hi;
        swap32(v, lo, hi);
        v = r & 1 ? hi : lo;
    }
    return v;
}

// Householder steps whose row k + 1 lies in block B of the lane's rows; the
// code holds only the rows from that block on.
template <int MM, int B>
__device__ __forceinline__ void tridiag_block(dd (&a)[DDL<MM>::R], DDShared<MM>& S, int m, int c, int h, int l15, dd& x) {
    constexpr int H = DDL<MM>::H, R = DDL<MM>::R, BR = DDL<MM>::BR;
    const int k0 = B == 0 ? 0 : H * BR * B - 1, kend = m - 2 < H * BR * (B + 1) - 1 ? m - 2 : H * BR * (B + 1) - 1;
#pragma unroll 1
    for (int k = k0; k < kend; ++k) {
        const dd alpha = ld(S.f.ch, S.f.cl, k + 1);
        const bool tail = c > k + 1 && c < m;
        const dd xn2 = wsum<MM>(tail ? mul(x, x) : mk(0.0));
        dd beta = alpha, tau = mk(0.0), scal = mk(0.0);
        if (xn2.hi > 0.0) {
            const dd nrm = dsqrt(add(mul(alpha, alpha), xn2));
            beta = alpha.hi >= 0.0 ? neg(nrm) : nrm;
            tau = dvd(sub(beta, alpha), beta);
            scal = dvd(mk(1.0), sub(alpha, beta));
        }
        const dd vj = (c == k + 1) ? mk(1.0) : (tail ? mul(x, scal) : mk(0.0));
        if (c == k && h == 0) {
            const dd e2 = mul(beta, beta);
            S.f.de[k].x = x.hi;
            S.f.de[k].y = x.lo;
            S.f.eh[k] = beta.hi;
            S.f.de[k + 1].z = e2.hi;
            S.f.de[k + 1].w = e2.lo;
        }
        st(S.f.vh, S.f.vl, c, vj);
        fence();
        // w = tau A v - (tau^2 / 2) (v^T A v) v over the rows from k + 1 on
        dd v[R / 16], w[R / 16];
#pragma unroll
        for (int g = 0; g < R / 16; ++g) v[g] = ld(S.f.vh, S.f.vl, H * (16 * g + l15) + h);
        dd p = mk(0.0), p2 = mk(0.0);  // two chains, two terms at a time
        each<BR * B / 2, R / 2>([&](auto q) __attribute__((always_inline)) {
            constexpr int i = 2 * decltype(q)::value;
            dd& s = (i / 2) % 2 ? p2 : p;
            s = mac2(s, a[i], row_lane<i % 16>(v[i / 16]), a[i + 1], row_lane<(i + 1) % 16>(v[(i + 1) / 16]));
        });
        p = add(p, p2);
        if constexpr (H == 2) p = halves_sum(p);
        dd wj = (c > k && c < m) ? mul(tau, p) : mk(0.0);
        const dd s = wsum<MM>(mul(wj, vj));
        wj = sub(wj, mul(mul_d(mul(tau, s), 0.5), vj));
        st(S.f.wh, S.f.wl, c, wj);
        fence();
#pragma unroll
        for (int g = 0; g < R / 16; ++g) w[g] = ld(S.f.wh, S.f.wl, H * (16 * g + l15) + h);
        const dd nv = neg(vj), nw = neg(wj);
        each<BR * B, R>([&](auto q) __attribute__((always_inline)) {
            constexpr int i = decltype(q)::value;
            a[i] = mac2(a[i], row_lane<i % 16>(v[i / 16]), nw, row_lane<i % 16>(w[i / 16]), nv);
        });
        x = row_at<MM>(a, k + 1);
        st(S.f.ch, S.f.cl, c, x);
        fence();
    }
    if constexpr (BR * (B + 1) < R) tridiag_block<MM, B + 1>(a, S, m, c, h, l15, x);
}

// S.f.de and S.f.eh: the tridiagonal form of A~(eps).
template <int K, int MM>
__device__ __forceinline__ void tridiag_dd(DDShared<MM>& S, int n, int m, double eps, int c, int h, int l15) {
    constexpr int H = DDL<MM>::H, R = DDL<MM>::R;
    const dd e2 = two_prod(eps, eps);
    dd a[R];
    each<0, R>([&](auto q) __attribute__((always_inline)) {
        constexpr int i = decltype(q)::value;
        a[i] = entry<K, MM>(S, n, m, e2, H * i + h, c);
    });
    dd x = row_at<MM>(a, 0);
    fence();
    st(S.f.ch, S.f.cl, c, x);
    fence();
    tridiag_block<MM, 0>(a, S, m, c, h, l15, x);
    // trailing 2 x 2 block: x is row m - 2
    const dd y = row_at<MM>(a, m - 1);
    if (h == 0) {
        if (c == m - 2) {
            S.f.de[m - 2].x = x.hi;
            S.f.de[m - 2].y = x.lo;
        }
        if (c == m - 1) {
            const dd q = mul(x, x);
            S.f.eh[m - 2] = x.hi;
            S.f.de[m - 1].z = q.hi;
            S.f.de[m - 1].w = q.lo;
            S.f.de[m - 1].x = y.hi;
            S.f.de[m - 1].y = y.lo;
        }
    }
    fence();
}

// #eigenvalues of T below sigma (double-double recurrence, FP64 shift)
template <int MM>
__device__ __forceinline__ int sturm_dd(const DDShared<MM>& S, int m, double sigma, double pivmin) {
    int cnt = 0;
    dd q = mk(1.0);
#pragma unroll 2
    for (int i = 0; i < m; ++i) {
        const double4 de = S.f.de[i];
        dd t = dvd({de.z, de.w}, q);
        if (i == 0) t = mk(0.0);
        q = sub_q({de.x, de.y}, sigma, t);
        if (fabs(q.hi) < pivmin) q = mk(-pivmin);
        cnt += q.hi < 0.0 ? 1 : 0;
    }
    return cnt;
}

// Brackets of lambda_1 and lambda_m; max |lambda| = max(-lambda_1, lambda_m).
struct SpecDD {
    double lo1, hi1, lo2, hi2, pivmin;
    bool finite;
    __device__ double alo() const { return fmax(-hi1, lo2); }
    __device__ double ahi() const { return fmax(-lo1, hi2); }
    __device__ double amax() const { return 0.5 * (alo() + ahi()); }
};

// Multisection rounds on max |lambda| until its bracket is a few ulps wide, at
// most `rounds`: while both ends can be the larger, half the lanes split each
// bracket 33 ways; then all split one 65 ways.
template <int MM>
__device__ __forceinline__ void refine_dd(const DDShared<MM>& S, int m, int lane, SpecDD& sp, int rounds) {
    for (int rd = 0; rd < rounds && sp.ahi() - sp.alo() > 4e-16 * sp.ahi(); ++rd) {
        const bool need1 = !(sp.lo2 > -sp.lo1), need2 = !(-sp.hi1 > sp.hi2), both = need1 && need2;
        const int parts = both ? 32 : 64, tt = lane & (parts - 1);
        const bool top = both ? lane >= 32 : need2;  // lambda_m's bracket
        const double lo = top ? sp.lo2 : sp.lo1, hi = top ? sp.hi2 : sp.hi1;
        const double sig = lo + (hi - lo) * (double)(tt + 1) / (double)(parts + 1);
        const uint64_t bal = __ballot(sturm_dd(S, m, sig, sp.pivmin) < (top ? m : 1));
        auto cut = [&](double& l, double& u, int nb) {
            const double w = (u - l) / (double)(parts + 1), l0 = l;
            if (nb < parts) u = l0 + w * (double)(nb + 1);
            if (nb > 0) l = l0 + w * (double)nb;
        };
        if (both) {
            cut(sp.lo1, sp.hi1, __popcll(bal & 0xffffffffull));
            cut(sp.lo2, sp.hi2, __popcll(bal >> 32));
        } else if (need2) {
            cut(sp.lo2, sp.hi2, __popcll(bal));
        } else {
            cut(sp.lo1, sp.hi1, __popcll(bal));
        }
    }
}

// Gershgorin interval (and the extreme diagonal entries, Rayleigh quotients:
// lambda_1 <= min d, lambda_m >= max d), then `rounds` rounds.
template <int MM>
__device__ __forceinline__ SpecDD spectrum_dd(const DDShared<MM>& S, int m, int lane, int rounds) {
    double ngl = -INFINITY, gu = -INFINITY, emax2 = 0.0, dmx = -INFINITY, ndm = -INFINITY;
    bool fin = true;
    if (lane < m) {
        const double d = S.f.de[lane].x, e = lane < m - 1 ? S.f.eh[lane] : 0.0;
        const double off = (lane > 0 ? fabs(S.f.eh[lane - 1]) : 0.0) + fabs(e);
        ngl = off - d;
        gu = off + d;
        dmx = d;
        ndm = -d;
        emax2 = lane < m - 1 ? S.f.de[lane + 1].z : 0.0;
        fin = isfinite(d) && isfinite(e);
    }
    for (int o = 1; o < 64; o <<= 1) {
        ngl = fmax(ngl, __shfl_xor(ngl, o, 64));
        gu = fmax(gu, __shfl_xor(gu, o, 64));
        dmx = fmax(dmx, __shfl_xor(dmx, o, 64));
        ndm = fmax(ndm, __shfl_xor(ndm, o, 64));
        emax2 = fmax(emax2, __shfl_xor(emax2, o, 64));
    }
    SpecDD sp;
    sp.finite = __ballot(!fin) == 0;
    sp.pivmin = 1e-290 * fmax(1.0, emax2);
    const double pad = 4.0 * (gu + ngl) * 2.3e-16 + 2.0 * sp.pivmin;
    sp.lo1 = -ngl - pad;
    sp.hi2 = gu + pad;
    sp.hi1 = fmin(sp.hi2, -ndm + pad);
    sp.lo2 = fmax(sp.lo1, dmx - pad);
    if (sp.finite) refine_dd(S, m, lane, sp, rounds);
    return sp;
}

// kappa_2 > target: some |lambda| < max |lambda| / target.  The counts at both
// ends of max |lambda|'s bracket decide, and only where they differ the
// bracket is refined.
template <int MM>
__device__ __forceinline__ bool above_dd(const DDShared<MM>& S, int m, SpecDD& sp, double target, int lane) {
    if (!sp.finite || !(sp.amax() > 0.0)) return true;
    for (int it = 0;; ++it) {
        const double mid = sp.amax() / target;
        double sig = 0.0;
        if (lane == 0) sig = -sp.alo() / target;
        if (lane == 1) sig = sp.alo() / target;
        if (lane == 2) sig = -sp.ahi() / target;
        if (lane == 3) sig = sp.ahi() / target;
        if (lane == 4) sig = -mid;
        if (lane == 5) sig = mid;
        const int c = lane < 6 ? sturm_dd(S, m, sig, sp.pivmin) : 0;
        if (__shfl(c, 1, 64) > __shfl(c, 0, 64)) return true;
        if (__shfl(c, 3, 64) == __shfl(c, 2, 64)) return false;
        if (it == 8 || sp.ahi() - sp.alo() <= 4e-16 * sp.ahi()) return __shfl(c, 5, 64) > __shfl(c, 4, 64);
        refine_dd(S, m, lane, sp, 2);
    }
}

// smallest |lambda| by geometric multisection on both sides of zero
template <int MM>
__device__ __forceinline__ double min_abs_dd(const DDShared<MM>& S, int m, const SpecDD& sp, int lane) {
    const int nu = sturm_dd(S, m, 0.0, sp.pivmin);
    const double L = sp.amax() * 1e-40 + sp.pivmin, Hh = sp.amax() * (1.0 + 1e-14);
    double lp = log(L), hp = log(Hh), ln_ = log(L), hn = log(Hh);
    const int g = lane >> 5, tt = lane & 31;
    for (int rd = 0; rd < 16 && fmax(hp - lp, hn - ln_) > 1e-14; ++rd) {
        const double lo = g ? ln_ : lp, hi = g ? hn : hp;
        const double sig = exp(lo + (hi - lo) * (double)(tt + 1) / 33.0);
        const int cnt = sturm_dd(S, m, g ? -sig : sig, sp.pivmin);
        const uint64_t bal = __ballot(g ? cnt >= nu : cnt <= nu);
        const int nb1 = __popcll(bal & 0xffffffffull), nb2 = __popcll(bal >> 32);
        const double a1 = lp + (hp - lp) * (double)nb1 / 33.0, b1 = lp + (hp - lp) * (double)(nb1 + 1) / 33.0;
        const double a2 = ln_ + (hn - ln_) * (double)nb2 / 33.0, b2 = ln_ + (hn - ln_) * (double)(nb2 + 1) / 33.0;
        if (nb1 > 0) lp = a1;
        if (nb1 < 32) hp = b1;
        if (nb2 > 0) ln_ = a2;
        if (nb2 < 32) hn = b2;
    }
    const double pos = nu < m ? exp(0.5 * (lp + hp)) : INFINITY;
    const double ng = nu > 0 ? exp(0.5 * (ln_ + hn)) : INFINITY;
    return fmin(pos, ng);
}

// LU with partial pivoting of A~ in place (lane (c, h): column c, rows of
// parity h); false on a zero pivot
template <int MM>
__device__ bool lu_dd(DDShared<MM>& S, int m, int c, int h) {
    constexpr int H = DDL<MM>::H, LDA = DDL<MM>::LDA;
    const int lane = threadIdx.x;
    for (int k = 0; k < m; ++k) {
        const double v = (lane >= k && lane < m) ? fabs(S.g.ah[lane * LDA + k]) : -1.0;
        double mx = v;
        for (int o = 1; o < 64; o <<= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
        const uint64_t hit = __ballot(v == mx && v >= 0.0);
        const int p = hit ? __ffsll((long long)hit) - 1 : k;
        if (!(mx > 0.0)) return false;
        if (lane == 0) S.piv[k] = p;
        if (p != k && lane < m) {
            const dd a = A(S, k, lane), b = A(S, p, lane);
            setA(S, k, lane, b);
            setA(S, p, lane, a);
        }
        fence();
        const dd piv = A(S, k, k);
        if (lane > k && lane < m) setA(S, lane, k, dvd(A(S, lane, k), piv));
        fence();
        if (c > k && c < m) {
            const dd ukj = A(S, k, c);
            for (int r = k + 1 + ((k + 1 + h) & (H - 1)); r < m; r += H) setA(S, r, c, sub(A(S, r, c), mul(A(S, r, k), ukj)));
        }
        fence();
    }
    return true;
}

// b_v <- A~^{-1} b_v for the first nb right-hand sides in S.bh/bl
template <int MM>
__device__ void lu_solve_dd(DDShared<MM>& S, int m, int nb, int lane) {
    if (lane < nb)
        for (int k = 0; k < m; ++k) {
            const int p = S.piv[k];
            if (p != k) {
                const dd a = ld(S.bh[lane], S.bl[lane], k), b = ld(S.bh[lane], S.bl[lane], p);
                st(S.bh[lane], S.bl[lane], k, b);
                st(S.bh[lane], S.bl[lane], p, a);
            }
        }
    fence();
    for (int k = 0; k < m; ++k) {  // L (unit diagonal)
        if (lane > k && lane < m) {
            const dd l = A(S, lane, k);
            for (int v = 0; v < nb; ++v)
                st(S.bh[v], S.bl[v], lane, sub(ld(S.bh[v], S.bl[v], lane), mul(l, ld(S.bh[v], S.bl[v], k))));
        }
        fence();
    }
    for (int k = m - 1; k >= 0; --k) {  // U
        if (lane < nb) st(S.bh[lane], S.bl[lane], k, dvd(ld(S.bh[lane], S.bl[lane], k), A(S, k, k)));
        fence();
        if (lane < k) {
            const dd u = A(S, lane, k);
            for (int v = 0; v < nb; ++v)
                st(S.bh[v], S.bl[v], lane, sub(ld(S.bh[v], S.bl[v], lane), mul(u, ld(S.bh[v], S.bl[v], k))));
        }
        fence();
    }
}

template <int K, int MM>
__global__ __launch_bounds__(64, 2) void k_weights_dd(rbw::Job J) {
    constexpr int H = DDL<MM>::H, R = DDL<MM>::R;
    __shared__ DDShared<MM> S;
    const int64_t s = blockIdx.x;
    if (s >= J.N) return;
    const rbw::WOpts& o = J.o;
    const int n = o.n, m = n + 1, lane = threadIdx.x;
    const int c = H == 2 ? lane & 31 : lane, h = H == 2 ? lane >> 5 : 0, l15 = lane & 15;
    // gather: coordinates; unit normals in double-double (lanes of the first half)
    bool bad = false, badn = false;
    dd nu[3] = {mk(0.0), mk(0.0), mk(0.0)};
    if (lane < n) {
        int64_t node = J.idx[s * n + lane];
        bad = node < 0 || node >= J.N;
        if (bad) node = 0;
        S.x[lane] = J.xyz[3 * node];
        S.y[lane] = J.xyz[3 * node + 1];
        S.z[lane] = J.xyz[3 * node + 2];
        const dd nx = mk(J.nrm[3 * node]), ny = mk(J.nrm[3 * node + 1]), nz = mk(J.nrm[3 * node + 2]);
        const dd nn = dsqrt(add(add(mul(nx, nx), mul(ny, ny)), mul(nz, nz)));
        badn = !(nn.hi > 0.0 && isfinite(nn.hi));
        const dd inv = badn ? mk(0.0) : dvd(mk(1.0), nn);
        nu[0] = mul(nx, inv);
        nu[1] = mul(ny, inv);
        nu[2] = mul(nz, inv);
        if (lane == 0)
            for (int q = 0; q < 3; ++q) st(S.n0h, S.n0l, q, nu[q]);
    }
    fence();
    bool dup = false;
    double r20 = 0.0;
    if (lane < n) {
        dd d[3];
        diff3(S, lane, 0, d);
        const dd r2 = norm2(d);
        r20 = r2.hi;
        dup = lane > 0 && r2.hi == 0.0;
    }
    if (__ballot(bad) || __ballot(badn)) {
        const bool any_bad = __ballot(bad) != 0;
        if (lane == 0) {
            if (J.eps) J.eps[s] = NAN;
            if (J.kappa) J.kappa[s] = NAN;
            if (J.nevals) J.nevals[s] = 0;
            if (J.status) J.status[s] = any_bad ? RBFFD_ST_BAD_INDEX : RBFFD_ST_BAD_NORMAL;
        }
        if (lane < n) J.w[s * n + lane] = NAN;
        return;
    }
    int status = __ballot(dup) ? RBFFD_ST_DUPLICATE : RBFFD_ST_OK;
    double rmax = r20;
    for (int o2 = 1; o2 < 64; o2 <<= 1) rmax = fmax(rmax, __shfl_xor(rmax, o2, 64));
    const double rho = sqrt(rmax);
    // shape parameter: one evaluation per turn, so that its code is there once
    enum Phase { LOW, HIGH, MID, FINAL };
    int evals = 0, ph = FINAL, q = 0;
    double eps, lo = 0.0, hi = 0.0;
    if (o.mode == RBFFD_EPS_FIXED) {
        eps = o.eps_fixed;
    } else if (o.mode == RBFFD_EPS_GIVEN) {
        eps = J.eps_in[s];
    } else {
        lo = o.br_lo / rho;
        hi = o.br_hi / rho;
        eps = lo;
        ph = LOW;
    }
    SpecDD sp;
    for (;;) {
        tridiag_dd<K, MM>(S, n, m, eps, c, h, l15);
        sp = spectrum_dd(S, m, lane, ph == FINAL ? 24 : 2);
        ++evals;
        if (ph == FINAL) break;
        const bool above = above_dd(S, m, sp, o.kappa_target, lane);
        if (ph == LOW) {
            if (!above && q < o.max_expand) {
                ++q;
                lo *= 0.5;
                eps = lo;
                continue;
            }
            if (!above && status == RBFFD_ST_OK) status = RBFFD_ST_NO_BRACKET;
            q = 0;
            eps = hi;
            ph = HIGH;
            continue;
        }
        if (ph == HIGH) {
            if (above && q < o.max_expand) {
                ++q;
                hi *= 2.0;
                eps = hi;
                continue;
            }
            if (above && status == RBFFD_ST_OK) status = RBFFD_ST_NO_BRACKET;
        } else if (above) {
            lo = eps;
        } else {
            hi = eps;
        }
        ph = hi - lo > o.eps_tol ? MID : FINAL;
        eps = 0.5 * (lo + hi);
    }
    double kappa = NAN;
    if (sp.finite && sp.amax() > 0.0) kappa = sp.amax() / min_abs_dd(S, m, sp, lane);
    else if (status == RBFFD_ST_OK) status = RBFFD_ST_NONFINITE;
    if (lane == 0) {
        if (J.eps) J.eps[s] = eps;
        if (J.kappa) J.kappa[s] = kappa;
        if (J.nevals) J.nevals[s] = evals;
    }
    // weights: LU of A~(eps), g_d = (A~^{-1} b_d)[:n], r = sum_d (B^d)^T g_d, w = (A~^{-1} r)[:n]
    const dd e2 = two_prod(eps, eps);
    fence();
    if (c < m)
        for (int r = h; r < m; r += H) setA(S, r, c, entry<K, MM>(S, n, m, e2, r, c));
    if (lane < m) {
        dd b[3] = {mk(0.0), mk(0.0), mk(0.0)};
        if (lane < n) {  // row 1 of B^d: psi(r_1j) [Pi_1 (x_1 - x_j)]_d; the ones border has zero gradient
            dd d[3];
            diff3(S, 0, lane, d);
            const dd ps = psi<K>(e2, norm2(d));
            const dd n0[3] = {ld(S.n0h, S.n0l, 0), ld(S.n0h, S.n0l, 1), ld(S.n0h, S.n0l, 2)};
            const dd dn = add(add(mul(n0[0], d[0]), mul(n0[1], d[1])), mul(n0[2], d[2]));
            for (int t = 0; t < 3; ++t) b[t] = mul(ps, sub(d[t], mul(n0[t], dn)));
        }
        for (int t = 0; t < 3; ++t) st(S.bh[t], S.bl[t], lane, b[t]);
    }
    fence();
    if (!lu_dd(S, m, c, h)) {
        if (status == RBFFD_ST_OK) status = RBFFD_ST_SINGULAR;
        if (lane == 0 && J.status) J.status[s] = status;
        if (lane < n) J.w[s * n + lane] = NAN;
        return;
    }
    lu_solve_dd(S, m, 3, lane);
    // h_i = Pi_i g_i, in place
    if (lane < n) {
        dd g[3];
        for (int t = 0; t < 3; ++t) g[t] = ld(S.bh[t], S.bl[t], lane);
        const dd dn = add(add(mul(nu[0], g[0]), mul(nu[1], g[1])), mul(nu[2], g[2]));
        for (int t = 0; t < 3; ++t) st(S.bh[t], S.bl[t], lane, sub(g[t], mul(nu[t], dn)));
    }
    fence();
    // r_j = sum_i psi(r_ij) (x_i - x_j) . h_i, r_n = 0
    dd rj = mk(0.0);
    if (c < n)
        for (int i = h; i < n; i += H) {
            dd d[3];
            diff3(S, i, c, d);
            const dd ps = psi<K>(e2, norm2(d));
            dd dot = mul(d[0], ld(S.bh[0], S.bl[0], i));
            for (int t = 1; t < 3; ++t) dot = add(dot, mul(d[t], ld(S.bh[t], S.bl[t], i)));
            rj = add(rj, mul(ps, dot));
        }
    if (H == 2) rj = halves_sum(rj);
    fence();
    if (lane < m) st(S.bh[0], S.bl[0], lane, rj);
    fence();
    lu_solve_dd(S, m, 1, lane);
    if (lane < n) J.w[s * n + lane] = to_d(ld(S.bh[0], S.bl[0], lane));
    if (lane == 0 && J.status) J.status[s] = status;
}

template <int MM>
void launch_dd(hipStream_t st, const rbw::Job& J) {
    const dim3 g((unsigned)J.N), b(64);
    if (J.o.kernel == RBFFD_KERNEL_MQ) hipLaunchKernelGGL((k_weights_dd<RBFFD_KERNEL_MQ, MM>), g, b, 0, st, J);
    else hipLaunchKernelGGL((k_weights_dd<RBFFD_KERNEL_IMQ, MM>), g, b, 0, st, J);
}

}  // namespace

int weights_check_opts(rbffd_ctx ctx, int64_t N, const rbffd_weight_opts* opts, rbw::WOpts& o);

extern "C" int rbffd_build_weights_dd(rbffd_ctx ctx, int64_t N, const double* xyz, const double* nrm,
                                      const rbffd_weight_opts* opts, const int32_t* idx_in, const double* eps_in,
                                      int32_t* idx_out, double* w, double* eps, double* kappa, int32_t* status,
                                      int32_t* nevals) {
    if (!ctx) return RBFFD_E_ARG;
    rbw::Job J;
    int rc = weights_check_opts(ctx, N, opts, J.o);
    if (rc) return rc;
    if (J.o.kernel != RBFFD_KERNEL_MQ && J.o.kernel != RBFFD_KERNEL_IMQ)
        return set_error(ctx, RBFFD_E_UNSUPPORTED, "extended-precision weights: MQ or IMQ kernel only");
    if (J.o.degree != 0)
        return set_error(ctx, RBFFD_E_UNSUPPORTED, "extended-precision weights: constant border (degree 0) only");
    if (J.o.n + 1 > DD_MAX)
        return set_error(ctx, RBFFD_E_UNSUPPORTED, "extended-precision weights: n + 1 = %d exceeds %d", J.o.n + 1,
                         DD_MAX);
    if (J.o.mode == RBFFD_EPS_LEARNED)
        return set_error(ctx, RBFFD_E_UNSUPPORTED, "extended-precision weights: fixed, given or bisection eps only");
    if (N == 0) return RBFFD_OK;
    if (!xyz || !nrm || !w) return set_error(ctx, RBFFD_E_ARG, "null pointer");
    if (J.o.mode == RBFFD_EPS_GIVEN && !eps_in) return set_error(ctx, RBFFD_E_ARG, "eps_in required for this eps_mode");
    const int32_t* idx = idx_in;
    if (!idx) {
        if (!idx_out) return set_error(ctx, RBFFD_E_ARG, "idx_out required when idx_in is NULL");
        rc = knn_internal(ctx, N, xyz, J.o.n, idx_out, nullptr);
        if (rc) return rc;
        idx = idx_out;
    } else if (idx_out && idx_out != idx_in) {
        HIP_TRY(ctx, hipMemcpyAsync(idx_out, idx_in, N * J.o.n * sizeof(int32_t), hipMemcpyDeviceToDevice, ctx->stream));
    }
    J.N = N;
    J.xyz = xyz;
    J.nrm = nrm;
    J.idx = idx;
    J.eps_in = eps_in;
    J.w = w;
    J.eps = eps;
    J.kappa = kappa;
    J.status = status;
    J.nevals = nevals;
    J.kappa_only = 0;
    // two lanes per column as long as they fit; past that one lane holds a column
    if (J.o.n + 1 <= 32) launch_dd<32>(ctx->stream, J);
    else launch_dd<DD_MAX>(ctx->stream, J);
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}
