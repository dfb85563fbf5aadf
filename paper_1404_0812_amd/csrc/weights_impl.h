// Device routines of the per-stencil weights computation (see weights.hip).
#pragma once

#include "common.h"
#include "weights_job.h"

#include <cmath>
#include <type_traits>

namespace rbw {

constexpr int RMAX = RBW_RMAX;  // border columns (degree-2 monomials in R^3)

// Tilings, named by the largest m they hold: 32 (two stencils per wavefront,
// one in each half, lane of the half = column), 48 and 64 (one wavefront per
// stencil, lane = column) and 128 (four wavefronts, wave (rb, cb) holding
// rows 64 rb .. 64 rb + 63 of columns 64 cb + lane).  The same operations in
// the same order whatever the tiling: lanes and rows past m hold zeros, and a
// sum over 32 lanes equals the sum over 64 whose upper half is zero.
//
// The two halves of a wavefront run different stencils, so whatever depends
// on the stencil (brackets, counts, the phase of the search) may diverge
// between them; nothing below moves data across the halves, and m is made
// wave-uniform before it bounds a loop (see process_stencil).
//
// Why these lines: at m = 32 (the paper's n = 31 with the constant border) one
// stencil per wavefront leaves half the lanes idle (10242 stencils by
// bisection: 6.35 ms; two per wavefront: 3.27 ms); 48 rows instead of 64 let
// three wavefronts share a SIMD (2500 stencils of 31 nodes, degree 2, one
// eps: 462 -> 408 us).  Past 64 the matrix needs more than one wavefront's
// registers.
template <int MM>
struct Lay {
    static constexpr int NB = MM == 128 ? 2 : 1;   // row and column blocks
    static constexpr int R = MM < 64 ? MM : 64;    // matrix rows held by a thread
    static constexpr int SPW = MM == 32 ? 2 : 1;   // stencils per wavefront
    static constexpr int LW = 64 / SPW;            // lanes of a stencil in a wavefront
    static constexpr int LA = MM > LW ? MM : LW;   // entries of a lane-indexed array
    static constexpr int OCC = MM <= 48 ? 3 : 2;   // wavefronts per SIMD
    // border basis entries: n + M <= MM with M = 1, 4 or 10 columns
    static constexpr int UN = MM == 32 ? 220 : 10 * (MM - 10);
    static constexpr int WAVES = NB * NB;          // wavefronts per stencil
};

// ------------------------------------------------------------ reductions ----
// Wavefront reductions with DPP (within rows of 16 lanes) and the row swaps
// (across the four rows).  Every lane must be active; the result is the same,
// bit for bit, in every lane.
// With every row and bank enabled and a permutation inside full rows, every
// lane reads a valid source lane, so no "old" value is needed (mov_dpp leaves
// it undefined and spares the two moves that would initialise it).
template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum16(double v) {
    v += dpp64<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp64<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp64<0x141>(v);  // row_half_mirror
    v += dpp64<0x140>(v);  // row_mirror
    return v;
}
// Cross-row step with the gfx950 row swaps, staying in vector registers: with
// both operands the same value, permlane16_swap gives every lane of rows
// (0, 1) the pair (r0, r1) and of rows (2, 3) the pair (r2, r3);
// permlane32_swap then pairs the two halves.  Every lane ends with
// (r0 + r1) + (r2 + r3) (op = max: the same association with fmax).
__device__ __forceinline__ void swap16(double v, double& a, double& b) {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    a = __hiloint2double((int)h[0], (int)l[0]);
    b = __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ void swap32(double v, double& a, double& b) {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    a = __hiloint2double((int)h[0], (int)l[0]);
    b = __hiloint2double((int)h[1], (int)l[1]);
}
template <int MM>
__device__ __forceinline__ double rows_total(double v) {
    double a, b;
    swap16(v, a, b);
    if constexpr (MM == 32) return a + b;
    swap32(a + b, a, b);
    return a + b;
}
template <int MM>
__device__ __forceinline__ double wave_sum(double v) {
    return rows_total<MM>(row_sum16(v));
}
// Sum of the products x y: the first step pairs one lane's rounded product
// with the other lane's through an FMA, so the two lanes of a pair differ in
// the last bit and only one lane's total (lane 0, or the caller's own) counts.
template <int MM>
__device__ __forceinline__ double wave_dot(double x, double y) {
    double v = fma(x, y, dpp64<0xB1>(x * y));
    v += dpp64<0x4E>(v);
    v += dpp64<0x141>(v);
    v += dpp64<0x140>(v);
    return rows_total<MM>(v);
}
// wave_dot(x0, y0) + wave_dot(x1, y1), whole wavefront, the same in every
// lane: the row totals of the two products share the cross-row steps (row 0
// and 2 finish the first, row 1 and 3 the second), and the lanes 0 of the two
// hand over the totals.
__device__ __forceinline__ double wave_dot_pair(double x0, double y0, double x1, double y1);
// The same swaps with two different operands x (vdst) and y (vsrc):
// permlane32_swap leaves x = [x lanes 0-31, y lanes 0-31] and
// y = [x lanes 32-63, y lanes 32-63], so their sum folds x into lanes 0-31
// and y into lanes 32-63; permlane16_swap leaves x = [x row 0, y row 0, x row 2,
// y row 2] and y = [x row 1, y row 1, x row 3, y row 3] (rows of 16 lanes).
__device__ __forceinline__ double fold32(double x, double y) {
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false,
                                                    false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false,
                                                    false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ double fold16(double x, double y) {
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false,
                                                    false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false,
                                                    false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ double readlane64(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
__device__ __forceinline__ double wave_dot_pair(double x0, double y0, double x1, double y1) {
    double u = fma(x0, y0, dpp64<0xB1>(x0 * y0));
    double v = fma(x1, y1, dpp64<0xB1>(x1 * y1));
    u += dpp64<0x4E>(u);
    v += dpp64<0x4E>(v);
    u += dpp64<0x141>(u);
    v += dpp64<0x141>(v);
    u += dpp64<0x140>(u);
    v += dpp64<0x140>(v);
    double a, b;
    swap32(fold16(u, v), a, b);
    a += b;
    return readlane64(a, 0) + readlane64(a, 16);
}
// Four wavefront sums at once: the folds put a, c, b, d in rows 0..3 (two
// stencils per wavefront: a, b and c, d in the two rows of each half).
template <int MM>
__device__ __forceinline__ void wave_sum4(double& a, double& b, double& c, double& d) {
    if constexpr (MM == 32) {
        const double s = row_sum16(fold16(a, b));
        const double t = row_sum16(fold16(c, d));
        swap16(s, a, b);
        swap16(t, c, d);
        return;
    }
    const double s = fold32(a, b);
    const double t = fold32(c, d);
    const double u = row_sum16(fold16(s, t));
    a = readlane64(u, 0);
    c = readlane64(u, 16);
    b = readlane64(u, 32);
    d = readlane64(u, 48);
}
// Three wavefront sums at once: a and b share the first fold (a in lanes 0-31,
// b in 32-63), c is folded with itself, the second fold puts a, c, b, c in
// rows 0..3, one row sum finishes all three, and lanes 0, 32, 16 hand them
// to every lane.  About a third of the instructions of three wave_sum calls.
__device__ __forceinline__ void wave_sum3(double& a, double& b, double& c) {  // whole wavefront
    const double s = fold32(a, b);
    const double t = fold32(c, c);
    const double u = row_sum16(fold16(s, t));
    a = readlane64(u, 0);
    c = readlane64(u, 16);
    b = readlane64(u, 32);
}
template <int MM>
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp64<0xB1>(v));
    v = fmax(v, dpp64<0x4E>(v));
    v = fmax(v, dpp64<0x141>(v));
    v = fmax(v, dpp64<0x140>(v));
    double a, b;
    swap16(v, a, b);
    if constexpr (MM == 32) return fmax(a, b);
    swap32(fmax(a, b), a, b);
    return fmax(a, b);
}
// 1/q: hardware reciprocal and one Newton step (the step squares the hardware
// estimate's relative error).  Used by the Sturm recurrence, whose count only
// needs the sign of each pivot (which the recurrence gets backward-stably),
// by the tridiagonal factorisation, where an error of an ulp or two in a
// multiplier is a backward perturbation of T of the size GEPP itself leaves,
// and by the Householder reduction (tau and the scale of v).
__device__ __forceinline__ double recip(double q) {
    const double r = __builtin_amdgcn_rcp(q);
    return fma(r, fma(-q, r, 1.0), r);
}

// ---------------------------------------------------------- radial kernels ----
// sqrt(x) for x >= 1: the hardware reciprocal square root y ~ 1/sqrt(x),
// then g = x y, h = y / 2 refined by one coupled Newton step and two
// residual corrections g += (x - g^2) h, the last of which rounds correctly.
// The general square root adds a rescaling for tiny arguments and a class
// check (seven more instructions); the radial kernels' argument 1 + eps^2 r^2
// never needs them (for x >= 1 the two give the same bits; a non-finite x
// gives a non-finite result either way).
__device__ __forceinline__ double sqrt_ge1(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    double d = fma(-g, g, x);
    g = fma(d, h, g);
    d = fma(-g, g, x);
    return fma(d, h, g);
}
template <int K>
__device__ __forceinline__ double rbf_phi(double e2, double r2) {
    double e = e2 * r2;
    if (K == RBFFD_KERNEL_MQ) return sqrt_ge1(1.0 + e);
    if (K == RBFFD_KERNEL_IMQ) return 1.0 / sqrt_ge1(1.0 + e);
    return exp(-e);
}
// phi'(r)/r
template <int K>
__device__ __forceinline__ double rbf_psi(double e2, double r2) {
    double e = e2 * r2;
    if (K == RBFFD_KERNEL_MQ) return e2 / sqrt_ge1(1.0 + e);
    if (K == RBFFD_KERNEL_IMQ) return -e2 / (sqrt_ge1(1.0 + e) * (1.0 + e));
    return -2.0 * e2 * exp(-e);
}

// LDS of one stencil.  The arrays of the eigenvalue search and those of the
// solves are never live together and share their space.
template <int MM>
struct Shared {
    static constexpr bool ONE = MM <= 64;
    static constexpr int LA = Lay<MM>::LA, LW = Lay<MM>::LW;
    struct Search {
        double2 de[MM];  // (d_i, e_{i-1}^2): one 16-byte read per Sturm step
        double col[LA];  // next pivot column
        double ww[LA];
        double vr[Lay<MM>::WAVES][LW], wr[Lay<MM>::WAVES][LW];  // v and w of a wave's row block
        double pp[ONE ? 1 : 2][ONE ? 1 : MM];                   // matvec partial sums per row block
        double nrm2[ONE ? 1 : 2];                               // squared norm of the pivot column's tail
    };
    struct Solve {
        double fd[MM], fdu[MM], fdl[MM], ffact[MM];  // pivoted tridiagonal factors (fd: 1/pivot)
        double rhs[3][LA];
        double zb[LA];
        double hx[ONE ? 1 : MM], hy[ONE ? 1 : MM], hz[ONE ? 1 : MM];
        double vb[ONE ? 1 : MM];
        double G[ONE ? 6 * (Lay<MM>::R / 4) : 1];  // Gram entries of the reflectors in blocks of four
        int fswap[MM];
    };
    union {
        Search f;
        Solve g;
    };
    double x[MM], y[MM], z[MM];  // stencil node coordinates
    double U[Lay<MM>::UN];       // border basis values U[j * us + k], us = border_cols(degree)
    double T[RMAX * RMAX];       // monomial coefficients of the border basis T[l*RMAX + k]
    double red[ONE ? 1 : 16];    // cross-wave partial sums, two sets of 8
    double d[MM], e[MM], tau[MM];
    double nrm0[3];
    double eps;  // the next evaluation's, and whether there is none (four waves)
    int done;
    int m, r, n, fact_ok;
    // h = Pi g: its three components take the place of the solved right-hand sides (one wave)
    __device__ double* h(int i) {
        if constexpr (ONE) return g.rhs[i];
        else return i == 0 ? g.hx : (i == 1 ? g.hy : g.hz);
    }
};

// m and n as scalars (the same for the whole stencil, so for the wavefront).
template <int MM>
__device__ __forceinline__ int stencil_m(const Shared<MM>& S) {
    return __builtin_amdgcn_readfirstlane(S.m);
}
template <int MM>
__device__ __forceinline__ int stencil_n(const Shared<MM>& S) {
    return __builtin_amdgcn_readfirstlane(S.n);
}

// Position of a thread in the stencil's work group.
struct Tid {
    int lane;  // 0..63
    int rb;    // row block (rows 64 rb + jj held in registers)
    int cb;    // column block
    int c;     // column index 64 cb + lane
    int tid;   // 0 .. 63 (255 with four waves) within the stencil's threads
    int l15;   // lane within its row of 16
    mutable int rot = 0;  // reductions done so far (selects the slot set)
};

// One wavefront: order LDS accesses and keep the compiler from moving them.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <int MM>
__device__ __forceinline__ void bsync() {
    if constexpr (MM <= 64) {
        wave_order();
    } else {
        __syncthreads();
    }
}

// Cross-wave partial sums (four waves) go through one of two slot sets, taken in
// turn by successive reductions; every reduction has one barrier between its
// writes and its reads, so by the time a set is written again every thread
// has read it, and no second barrier is needed.
__device__ __forceinline__ double* red_set(double* red, const Tid& t) { return red + 8 * (t.rot++ & 1); }

// Sum over the columns (lane-distributed; each column is held by Lay::NB threads).
template <int MM>
__device__ __forceinline__ double sum_cols(double v, Shared<MM>& S, const Tid& t) {
    const double w = wave_sum<MM>(v);
    if constexpr (MM <= 64) {
        return w;
    } else {
        double* red = red_set(S.red, t);
        if (t.rb == 0 && t.lane == 0) red[t.cb] = w;
        bsync<MM>();
        return red[0] + red[1];
    }
}
template <int MM>
__device__ __forceinline__ void sum_cols3(double& a, double& b, double& c, Shared<MM>& S, const Tid& t) {
    wave_sum3(a, b, c);
    if constexpr (MM == 128) {
        double* red = red_set(S.red, t);
        if (t.rb == 0 && t.lane == 0) {
            red[t.cb] = a;
            red[2 + t.cb] = b;
            red[4 + t.cb] = c;
        }
        bsync<MM>();
        a = red[0] + red[1];
        b = red[2] + red[3];
        c = red[4] + red[5];
    }
}
// Sum over the rows held by lanes (row 64 rb + lane; cb == 0 waves count).
template <int MM>
__device__ __forceinline__ double sum_rows(double v, Shared<MM>& S, const Tid& t) {
    const double w = wave_sum<MM>(v);
    if constexpr (MM <= 64) {
        return w;
    } else {
        double* red = red_set(S.red, t);
        if (t.cb == 0 && t.lane == 0) red[6 + t.rb] = w;
        bsync<MM>();
        return red[6] + red[7];
    }
}
// Four sums over the rows held by lanes at once (see sum_rows).
template <int MM>
__device__ __forceinline__ void sum_rows4(double& a, double& b, double& c, double& d, Shared<MM>& S, const Tid& t) {
    wave_sum4<MM>(a, b, c, d);
    if constexpr (MM == 128) {
        double* red = red_set(S.red, t);
        if (t.cb == 0 && t.lane == 0) {
            red[4 * t.rb] = a;
            red[4 * t.rb + 1] = b;
            red[4 * t.rb + 2] = c;
            red[4 * t.rb + 3] = d;
        }
        bsync<MM>();
        a = red[0] + red[4];
        b = red[1] + red[5];
        c = red[2] + red[6];
        d = red[3] + red[7];
    }
}
template <int MM>
__device__ __forceinline__ double max_cols(double v, Shared<MM>& S, const Tid& t) {
    const double w = wave_max<MM>(v);
    if constexpr (MM <= 64) {
        return w;
    } else {
        double* red = red_set(S.red, t);
        if (t.rb == 0 && t.lane == 0) red[t.cb] = w;
        bsync<MM>();
        return fmax(red[0], red[1]);
    }
}

// ----------------------------------------------------------- local matrix ----
// Column t.c, rows 64 rb .. 64 rb + 63 of A~(eps).
template <int K, int MM>
__device__ __forceinline__ void build_matrix(double (&a)[Lay<MM>::R], const Shared<MM>& S, const Tid& t, double e2, int us) {
    const int n = stencil_n<MM>(S), m = stencil_m<MM>(S), c = t.c;
    const int cc = c < n ? c : 0;
    const double xi = S.x[cc], yi = S.y[cc], zi = S.z[cc];
    const int r0 = 64 * t.rb;
#pragma unroll
    for (int jj = 0; jj < Lay<MM>::R; ++jj) {
        const int j = r0 + jj;
        double v = 0.0;
        if (j < n) {
            if (c < n) {
                const double dx = xi - S.x[j], dy = yi - S.y[j], dz = zi - S.z[j];
                const double r2 = (dx * dx + dy * dy) + dz * dz;
                v = rbf_phi<K>(e2, r2);
            } else if (c < m) {
                v = S.U[j * us + (c - n)];
            }
        } else if (j < m) {
            if (c < n) v = S.U[c * us + (j - n)];
        }
        a[jj] = v;
    }
}

// Row broadcasts.  v holds 16 consecutive entries of a vector, the same 16 in
// each of the wavefront's four rows of lanes (lane l: entry l % 16), and
// entry O + i multiplies the registers of matrix row i through the DPP row
// broadcast of v_fmac_f64 -- no LDS read and no extra instruction per row.
// s_nop: two wait states between a vector write of v and its DPP read (the
// compiler does not look for that hazard inside an asm block).  Reading v and
// w per row from LDS instead (a broadcast read of two rows at a time) kept the
// LDS busy 44% and the waves waiting 47% of the time; bisection of 250k
// 50-node stencils went from 48% to 65% VALU issue, the learned pass over
// them from 28.9 to 24.0 ms, 16 surfaces of 31 to 101 nodes from 189 to
// 133 ms (28 to 12.6 ms in the one-wave tiling, 157 to 117 in the four-wave).
//   dot8:  p0 += sum over even i of v_i a_i, p1 over odd i, in row order
//   rank2: a_i = fma(-v_i, wi, fma(-w_i, vi, a_i)) with nv = -vi, nw = -wi
#define RBW_BC(i) " row_newbcast:%" #i " row_mask:0xf bank_mask:0xf\n\t"
template <int O>
__device__ __forceinline__ void dot8(double& p0, double& p1, double v, double a0, double a1, double a2, double a3,
                                     double a4, double a5, double a6, double a7) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %3" RBW_BC(11) "v_fmac_f64_dpp %1, %2, %4" RBW_BC(12)
        "v_fmac_f64_dpp %0, %2, %5" RBW_BC(13) "v_fmac_f64_dpp %1, %2, %6" RBW_BC(14)
        "v_fmac_f64_dpp %0, %2, %7" RBW_BC(15) "v_fmac_f64_dpp %1, %2, %8" RBW_BC(16)
        "v_fmac_f64_dpp %0, %2, %9" RBW_BC(17) "v_fmac_f64_dpp %1, %2, %10" RBW_BC(18)
        : "+&v"(p0), "+&v"(p1)
        : "v"(v), "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(a4), "v"(a5), "v"(a6), "v"(a7), "n"(O), "n"(O + 1),
          "n"(O + 2), "n"(O + 3), "n"(O + 4), "n"(O + 5), "n"(O + 6), "n"(O + 7));
}
template <int O>
__device__ __forceinline__ void rank2(double v, double w, double nv, double nw, double& a0, double& a1, double& a2,
                                      double& a3, double& a4, double& a5, double& a6, double& a7) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %9, %10" RBW_BC(12) "v_fmac_f64_dpp %1, %9, %10" RBW_BC(13)
        "v_fmac_f64_dpp %2, %9, %10" RBW_BC(14) "v_fmac_f64_dpp %3, %9, %10" RBW_BC(15)
        "v_fmac_f64_dpp %4, %9, %10" RBW_BC(16) "v_fmac_f64_dpp %5, %9, %10" RBW_BC(17)
        "v_fmac_f64_dpp %6, %9, %10" RBW_BC(18) "v_fmac_f64_dpp %7, %9, %10" RBW_BC(19)
        "v_fmac_f64_dpp %0, %8, %11" RBW_BC(12) "v_fmac_f64_dpp %1, %8, %11" RBW_BC(13)
        "v_fmac_f64_dpp %2, %8, %11" RBW_BC(14) "v_fmac_f64_dpp %3, %8, %11" RBW_BC(15)
        "v_fmac_f64_dpp %4, %8, %11" RBW_BC(16) "v_fmac_f64_dpp %5, %8, %11" RBW_BC(17)
        "v_fmac_f64_dpp %6, %8, %11" RBW_BC(18) "v_fmac_f64_dpp %7, %8, %11" RBW_BC(19)
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3), "+&v"(a4), "+&v"(a5), "+&v"(a6), "+&v"(a7)
        : "v"(v), "v"(w), "v"(nv), "v"(nw), "n"(O), "n"(O + 1), "n"(O + 2), "n"(O + 3), "n"(O + 4), "n"(O + 5),
          "n"(O + 6), "n"(O + 7));
}
#undef RBW_BC
// Rows 8 j .. 8 j + 7 (j a constant after unrolling); v, w: the 16-entry groups.
template <int R>
__device__ __forceinline__ void dot_rows(const double (&a)[R], int j, const double* v, double& p0, double& p1) {
    if (j & 1)
        dot8<8>(p0, p1, v[j >> 1], a[8 * j], a[8 * j + 1], a[8 * j + 2], a[8 * j + 3], a[8 * j + 4], a[8 * j + 5],
                a[8 * j + 6], a[8 * j + 7]);
    else
        dot8<0>(p0, p1, v[j >> 1], a[8 * j], a[8 * j + 1], a[8 * j + 2], a[8 * j + 3], a[8 * j + 4], a[8 * j + 5],
                a[8 * j + 6], a[8 * j + 7]);
}
template <int R>
__device__ __forceinline__ void rank2_rows(double (&a)[R], int j, const double* v, const double* w, double nv,
                                           double nw) {
    if (j & 1)
        rank2<8>(v[j >> 1], w[j >> 1], nv, nw, a[8 * j], a[8 * j + 1], a[8 * j + 2], a[8 * j + 3], a[8 * j + 4],
                 a[8 * j + 5], a[8 * j + 6], a[8 * j + 7]);
    else
        rank2<0>(v[j >> 1], w[j >> 1], nv, nw, a[8 * j], a[8 * j + 1], a[8 * j + 2], a[8 * j + 3], a[8 * j + 4],
                 a[8 * j + 5], a[8 * j + 6], a[8 * j + 7]);
}

// f(i) for the one constant i in [LO, HI) that equals the wave-uniform k: a
// binary tree of scalar branches.
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

// Scalars of one reflector H = I - tau v v^T that maps the pivot column's
// tail (squared norm xnorm2 below alpha) to beta e_1; v = (1, scal * tail).
struct Reflector {
    double tau, beta, scal;
};
__device__ __forceinline__ Reflector reflector(double alpha, double xnorm2) {
    Reflector h{0.0, alpha, 0.0};
    if (xnorm2 > 0.0) {
        h.beta = -copysign(sqrt(alpha * alpha + xnorm2), alpha);
        // reciprocals instead of divisions: an ulp or so in tau and in the
        // scale of v, a perturbation of each reflector's orthogonality of
        // the size its own rounding already leaves
        h.tau = (h.beta - alpha) * recip(h.beta);
        h.scal = recip(alpha - h.beta);
    }
    return h;
}

// Householder tridiagonalisation of the m x m leading block (lane = column).
// On return: S.d[0..m-1], S.e[0..m-2], S.de, S.tau[0..m-3], and row k of
// the register matrix holds the reflector v_k (v_k[k+1] = 1).
//
// One wave: steps k = 8 B .. 8 B + 7 run the code of block B, which holds only
// the rows from 8 B on.  xi: the pivot column (row k of the symmetric matrix).
template <int MM, int B>
__device__ __forceinline__ void tridiag_block(double (&a)[Lay<MM>::R], Shared<MM>& S, const Tid& t, int m, int cl,
                                              double& xi) {
    constexpr int R = Lay<MM>::R;
    const int c = t.c;
    const int kend = m - 2 < 8 * B + 8 ? m - 2 : 8 * B + 8;
#pragma unroll 1
    for (int k = 8 * B; k < kend; ++k) {
        const double alpha = S.f.col[k + 1], dk = S.f.col[k];
        const bool tail = cl > k + 1;
        const double xnorm2 = wave_sum<MM>(tail ? xi * xi : 0.0);
        const Reflector h = reflector(alpha, xnorm2);
        const double vi = (c == k + 1) ? 1.0 : (tail ? xi * h.scal : 0.0);
        S.f.vr[0][c] = vi;
        if (t.tid == 0) {
            S.d[k] = dk;
            S.e[k] = h.beta;
            S.f.de[k].x = dk;
            S.f.de[k + 1].y = h.beta * h.beta;
            S.tau[k] = h.tau;
        }
        bsync<MM>();
        double v[R / 16], w[R / 16];
#pragma unroll
        for (int g = 0; g < R / 16; ++g) v[g] = g >= B / 2 ? S.f.vr[0][16 * g + t.l15] : 0.0;
        // p = A v (entries of v up to row k are zero)
        double p0 = 0.0, p1 = 0.0;
#pragma unroll
        for (int j = 0; j < R / 8; ++j)
            if (j >= B && (j <= B + 1 || 8 * j < m)) dot_rows<R>(a, j, v, p0, p1);
        double wi = cl > k ? h.tau * (p0 + p1) : 0.0;
        const double s = wave_dot<MM>(wi, vi);
        wi = fma(-0.5 * h.tau * s, vi, wi);
        S.f.wr[0][c] = wi;
        bsync<MM>();
#pragma unroll
        for (int g = 0; g < R / 16; ++g) w[g] = g >= B / 2 ? S.f.wr[0][16 * g + t.l15] : 0.0;
        // A -= v w^T + w v^T
        const double nv = -vi, nw = -wi;
#pragma unroll
        for (int j = 0; j < R / 8; ++j)
            if (j >= B && (j <= B + 1 || 8 * j < m)) rank2_rows<R>(a, j, v, w, nv, nw);
        // row k keeps v, row k + 1 is the next pivot column
        at_row<0, 8>(k - 8 * B, [&](auto q) __attribute__((always_inline)) {
            constexpr int row = 8 * B + decltype(q)::value;
            a[row] = vi;
            if constexpr (row + 1 < R) xi = a[row + 1];
        });
        S.f.col[c] = xi;
        bsync<MM>();
    }
    if constexpr (B + 1 < R / 8) tridiag_block<MM, B + 1>(a, S, t, m, cl, xi);
}

template <int MM>
__device__ __forceinline__ void tridiag_one(double (&a)[Lay<MM>::R], Shared<MM>& S, const Tid& t, int m) {
    double xi = a[0];
    S.f.col[t.c] = xi;
    bsync<MM>();
    tridiag_block<MM, 0>(a, S, t, m, t.c < m ? t.c : -1, xi);
    // trailing 2 x 2 block: row m - 1
    at_row<0, Lay<MM>::R>(m - 1, [&](auto q) __attribute__((always_inline)) {
        S.f.ww[t.c] = a[decltype(q)::value];
    });
}

// Four waves.  The two waves that hold row k + 1 publish it with the sums of
// its squares; every wave then forms the reflector and both halves of p and w
// itself (the sums over a column block are the same bits wherever they are
// formed), so a step needs two barriers: after the row-block partial sums of
// p and after the next pivot column.
template <int MM>
__device__ __forceinline__ void tridiag_four(double (&a)[Lay<MM>::R], Shared<MM>& S, const Tid& t, int m) {
    constexpr int R = Lay<MM>::R;
    const int c = t.c, o = c ^ 64, r0 = 64 * t.rb, wv = 2 * t.rb + t.cb;
    const bool own = t.rb == t.cb;  // this wave's rows are its columns' block
    const int cl = c < m ? c : -1, ol = o < m ? o : -1;
    // row k (held by this wave) as pivot column k: its entries and their tail's squared norm
    auto publish = [&](double x, int k) {
        S.f.col[c] = x;
        const double n2 = wave_sum<MM>(cl > k + 1 ? x * x : 0.0);
        if (t.lane == 0) S.f.nrm2[t.cb] = n2;
    };
    if (t.rb == 0) publish(a[0], 0);
    bsync<MM>();
#pragma unroll 1
    for (int k = 0; k < m - 2; ++k) {
        const double xc = S.f.col[c], xo = S.f.col[o];
        const double alpha = S.f.col[k + 1], dk = S.f.col[k];
        const bool tc = cl > k + 1, to = ol > k + 1;
        // columns up to k are done with: past k = 62 the whole first block
        const bool live = t.cb == 1 || k < 63;
        const double xnorm2 = S.f.nrm2[0] + S.f.nrm2[1];
        const Reflector h = reflector(alpha, xnorm2);
        const double vc = (c == k + 1) ? 1.0 : (tc ? xc * h.scal : 0.0);
        const double vo = (o == k + 1) ? 1.0 : (to ? xo * h.scal : 0.0);
        S.f.vr[wv][t.lane] = own ? vc : vo;
        if (t.tid == 0) {
            S.d[k] = dk;
            S.e[k] = h.beta;
            S.f.de[k].x = dk;
            S.f.de[k + 1].y = h.beta * h.beta;
            S.tau[k] = h.tau;
        }
        wave_order();
        double v[R / 16], w[R / 16];
#pragma unroll
        for (int g = 0; g < R / 16; ++g) v[g] = S.f.vr[wv][16 * g + t.l15];
        double p0 = 0.0, p1 = 0.0;
#pragma unroll
        for (int j = 0; j < R / 8; ++j)
            if (r0 + 8 * j + 8 > k + 1 && r0 + 8 * j < m && live) dot_rows<R>(a, j, v, p0, p1);
        S.f.pp[t.rb][c] = p0 + p1;
        bsync<MM>();
        const double pc = S.f.pp[0][c] + S.f.pp[1][c], po = S.f.pp[0][o] + S.f.pp[1][o];
        double wc = cl > k ? h.tau * pc : 0.0, wo = ol > k ? h.tau * po : 0.0;
        const double s = wave_dot_pair(wc, vc, wo, vo);
        wc = fma(-0.5 * h.tau * s, vc, wc);
        wo = fma(-0.5 * h.tau * s, vo, wo);
        S.f.wr[wv][t.lane] = own ? wc : wo;
        wave_order();
#pragma unroll
        for (int g = 0; g < R / 16; ++g) w[g] = S.f.wr[wv][16 * g + t.l15];
        const double nv = -vc, nw = -wc;
#pragma unroll
        for (int j = 0; j < R / 8; ++j)
            if (r0 + 8 * j + 8 > k + 1 && r0 + 8 * j < m && live) rank2_rows<R>(a, j, v, w, nv, nw);
        if (t.rb == k >> 6)
            at_row<0, R>(k & 63, [&](auto q) __attribute__((always_inline)) {
                    a[decltype(q)::value] = vc;
            });
        if (t.rb == (k + 1) >> 6) {
            double x = 0.0;
            at_row<0, R>((k + 1) & 63, [&](auto q) __attribute__((always_inline)) { x = a[decltype(q)::value]; });
            publish(x, k + 1);
        }
        bsync<MM>();
    }
    if (t.rb == (m - 1) >> 6)
        at_row<0, R>((m - 1) & 63, [&](auto q) __attribute__((always_inline)) {
            S.f.ww[c] = a[decltype(q)::value];
        });
}

template <int MM>
__device__ __forceinline__ void tridiagonalise(double (&a)[Lay<MM>::R], Shared<MM>& S, const Tid& t, int m) {
    if constexpr (MM <= 64) tridiag_one<MM>(a, S, t, m);
    else tridiag_four<MM>(a, S, t, m);
    bsync<MM>();
    if (t.tid == 0) {
        if (m >= 2) {
            S.d[m - 2] = S.f.de[m - 2].x = S.f.col[m - 2];
            S.e[m - 2] = S.f.col[m - 1];
            S.f.de[m - 1].y = S.f.col[m - 1] * S.f.col[m - 1];
        }
        S.d[m - 1] = S.f.de[m - 1].x = S.f.ww[m - 1];
    }
    bsync<MM>();
}

// ------------------------------------------------------------ Sturm counts ----
// Number of eigenvalues of T below sigma (wave-local).
template <int MM>
__device__ __forceinline__ int sturm(const Shared<MM>& S, int m, double sigma, double pivmin) {
    double q = S.d[0] - sigma;
    if (fabs(q) < pivmin) q = -pivmin;
    int c = q < 0.0 ? 1 : 0;
#pragma unroll 4
    for (int i = 1; i < m; ++i) {
        const double2 de = S.f.de[i];
        q = fma(-de.y, recip(q), de.x - sigma);
        if (fabs(q) < pivmin) q = -pivmin;
        c += q < 0.0 ? 1 : 0;
    }
    return c;
}

// Two shifts per lane.
template <int MM>
__device__ __forceinline__ void sturm2(const Shared<MM>& S, int m, double sa, double sb, double pivmin, int& ca,
                                       int& cb) {
    const double d0 = S.d[0];
    double qa = d0 - sa, qb = d0 - sb;
    if (fabs(qa) < pivmin) qa = -pivmin;
    if (fabs(qb) < pivmin) qb = -pivmin;
    ca = qa < 0.0 ? 1 : 0;
    cb = qb < 0.0 ? 1 : 0;
#pragma unroll 2
    for (int i = 1; i < m; ++i) {
        const double2 de = S.f.de[i];
        qa = fma(-de.y, recip(qa), de.x - sa);
        qb = fma(-de.y, recip(qb), de.x - sb);
        if (fabs(qa) < pivmin) qa = -pivmin;
        if (fabs(qb) < pivmin) qb = -pivmin;
        ca += qa < 0.0 ? 1 : 0;
        cb += qb < 0.0 ? 1 : 0;
    }
}

// One multisection round: shift sig(l) and its test pass(l, count) for
// l = 0..63; bit l of the result is the test's.  Each lane takes one l, or
// two (lane and lane + 32) where a stencil has half a wavefront.
template <int MM, typename F, typename P>
__device__ __forceinline__ uint64_t sturm64(const Shared<MM>& S, int m, int lane, double pivmin, F&& sig, P&& pass) {
    if constexpr (Lay<MM>::SPW == 1) {
        return __ballot(pass(lane, sturm<MM>(S, m, sig(lane), pivmin)));
    } else {
        int c0, c1;
        sturm2<MM>(S, m, sig(lane), sig(lane + 32), pivmin, c0, c1);
        const int half = threadIdx.x & 32;
        const uint64_t b0 = __ballot(pass(lane, c0)) >> half, b1 = __ballot(pass(lane + 32, c1)) >> half;
        return (b0 & 0xffffffffull) | (b1 << 32);
    }
}
// Lanes of the stencil for which p holds.
template <int MM>
__device__ __forceinline__ uint64_t stencil_ballot(bool p) {
    const uint64_t b = __ballot(p);
    return MM == 32 ? (b >> (threadIdx.x & 32)) & 0xffffffffull : b;
}
// Value of lane `l` (< 32) of the stencil's lanes in this wavefront.
template <int MM>
__device__ __forceinline__ int from_lane(int v, int l) {
    return __shfl(v, l, Lay<MM>::LW);
}

struct Spectrum {
    double amax;  // max |lambda| (midpoint estimate)
    bool finite;
    double pivmin;
    // multisection brackets: lambda_1 in [lo1, hi1], lambda_m in [lo2, hi2]
    double lo1, hi1, lo2, hi2;
};

// max |lambda| = max(-lambda_1, lambda_m) lies in [alo, ahi].
__device__ __forceinline__ void amax_bounds(const Spectrum& sp, double& alo, double& ahi) {
    alo = fmax(-sp.hi1, sp.lo2);
    ahi = fmax(-sp.lo1, sp.hi2);
}

// Up to `rounds` more multisection rounds on the brackets of lambda_1 and
// lambda_m.  While both can still be max |lambda| = max(-lambda_1, lambda_m),
// lanes 0..31 split lambda_1's bracket and lanes 32..63 lambda_m's 33 ways;
// once one of them is ruled out (its magnitude bound lies below the other's),
// all 64 lanes split the other's bracket 65 ways.  With rel > 0 the rounds
// stop as soon as the bracket of max |lambda| is within 2 rel of its midpoint
// (midpoint error <= rel relative).  sp.amax is that midpoint.
template <int MM>
__device__ __forceinline__ void spectrum_refine(const Shared<MM>& S, int lane, Spectrum& sp, int rounds,
                                                double rel = 0.0) {
    const int m = stencil_m<MM>(S);
    double lo1 = sp.lo1, hi1 = sp.hi1, lo2 = sp.lo2, hi2 = sp.hi2;
    for (int rd = 0; rd < rounds; ++rd) {
        // all conditions below are wave-uniform: the brackets are
        const double alo = fmax(-hi1, lo2), ahi = fmax(-lo1, hi2);
        if (rel > 0.0 && ahi - alo <= rel * (alo + ahi)) break;
        const bool need1 = !(lo2 > -lo1);  // lambda_1 can still be the largest in magnitude
        const bool need2 = !(-hi1 > hi2);  // lambda_m can
        if (need1 && need2) {
            const uint64_t bal = sturm64<MM>(
                S, m, lane, sp.pivmin,
                [&](int l) {
                    const double lo = l >> 5 ? lo2 : lo1, hi = l >> 5 ? hi2 : hi1;
                    return lo + (hi - lo) * (double)((l & 31) + 1) / 33.0;
                },
                [&](int l, int cnt) { return cnt < (l >> 5 ? m : 1); });  // the eigenvalue lies above the shift
            const int nb1 = __popcll(bal & 0xffffffffull);
            const int nb2 = __popcll(bal >> 32);
            const double n_lo1 = nb1 > 0 ? lo1 + (hi1 - lo1) * (double)nb1 / 33.0 : lo1;
            const double n_hi1 = nb1 < 32 ? lo1 + (hi1 - lo1) * (double)(nb1 + 1) / 33.0 : hi1;
            const double n_lo2 = nb2 > 0 ? lo2 + (hi2 - lo2) * (double)nb2 / 33.0 : lo2;
            const double n_hi2 = nb2 < 32 ? lo2 + (hi2 - lo2) * (double)(nb2 + 1) / 33.0 : hi2;
            lo1 = n_lo1; hi1 = n_hi1; lo2 = n_lo2; hi2 = n_hi2;
        } else {
            const double lo = need2 ? lo2 : lo1, hi = need2 ? hi2 : hi1;
            const int nb = __popcll(sturm64<MM>(
                S, m, lane, sp.pivmin, [&](int l) { return lo + (hi - lo) * (double)(l + 1) / 65.0; },
                [&](int, int cnt) { return cnt < (need2 ? m : 1); }));
            const double n_lo = nb > 0 ? lo + (hi - lo) * (double)nb / 65.0 : lo;
            const double n_hi = nb < 64 ? lo + (hi - lo) * (double)(nb + 1) / 65.0 : hi;
            if (need2) {
                lo2 = n_lo;
                hi2 = n_hi;
            } else {
                lo1 = n_lo;
                hi1 = n_hi;
            }
        }
    }
    sp.lo1 = lo1; sp.hi1 = hi1; sp.lo2 = lo2; sp.hi2 = hi2;
    sp.amax = 0.5 * (fmax(-hi1, lo2) + fmax(-lo1, hi2));
}

// Largest |lambda| of T to ~33^-rounds of the Gershgorin width (see
// spectrum_refine for rel).
template <int MM>
__device__ __forceinline__ Spectrum spectrum_max(const Shared<MM>& S, int lane, int rounds, double rel = 0.0) {
    const int m = stencil_m<MM>(S);
    Spectrum sp;
    // Gershgorin interval of T: each lane takes rows lane, lane + 64, then
    // wavefront min/max (exact, so the same bits as a serial scan)
    // and the extreme diagonal entries, Rayleigh quotients of unit vectors:
    // lambda_1 <= min d_i and lambda_m >= max d_i
    double ngl = -INFINITY, gu = -INFINITY, emax2 = 0.0, dmax = -INFINITY, ndmin = -INFINITY;
    bool fin = true;
    for (int i = lane; i < m; i += Lay<MM>::LW) {
        const double off = (i > 0 ? fabs(S.e[i - 1]) : 0.0) + (i < m - 1 ? fabs(S.e[i]) : 0.0);
        ngl = fmax(ngl, off - S.d[i]);
        gu = fmax(gu, S.d[i] + off);
        dmax = fmax(dmax, S.d[i]);
        ndmin = fmax(ndmin, -S.d[i]);
        if (i < m - 1) emax2 = fmax(emax2, S.f.de[i + 1].y);
        fin = fin && isfinite(S.d[i]) && (i == m - 1 || isfinite(S.e[i]));
    }
    double gl = -wave_max<MM>(ngl);
    gu = wave_max<MM>(gu);
    dmax = wave_max<MM>(dmax);
    const double dmin = -wave_max<MM>(ndmin);
    emax2 = wave_max<MM>(emax2);
    fin = stencil_ballot<MM>(!fin) == 0;
    sp.finite = fin;
    sp.pivmin = 2.2250738585072014e-308 * fmax(1.0, emax2);
    const double w = gu - gl;
    gl -= 2.0 * w * 2.2e-16 + 2.0 * sp.pivmin;
    gu += 2.0 * w * 2.2e-16 + 2.0 * sp.pivmin;
    sp.lo1 = gl;
    sp.hi2 = gu;
    // widened like the Gershgorin ends, for the counts' own rounding
    sp.hi1 = fmin(gu, dmin + 2.0 * w * 2.2e-16 + 2.0 * sp.pivmin);
    sp.lo2 = fmax(gl, dmax - 2.0 * w * 2.2e-16 - 2.0 * sp.pivmin);
    if (!fin) {
        sp.amax = NAN;
        return sp;
    }
    spectrum_refine<MM>(S, lane, sp, rounds, rel);
    return sp;
}

// #eigenvalues with |lambda| < tau for two thresholds (lanes 0-1 and 2-3)
template <int MM>
__device__ __forceinline__ void small_counts(const Shared<MM>& S, int lane, const Spectrum& sp, double tau_a,
                                             double tau_b, int& ca, int& cb) {
    const int m = stencil_m<MM>(S);
    double sig = 0.0;
    if (lane == 0) sig = -tau_a;
    if (lane == 1) sig = tau_a;
    if (lane == 2) sig = -tau_b;
    if (lane == 3) sig = tau_b;
    const int c = lane < 4 ? sturm<MM>(S, m, sig, sp.pivmin) : 0;
    const int c0 = from_lane<MM>(c, 0), c1 = from_lane<MM>(c, 1), c2 = from_lane<MM>(c, 2), c3 = from_lane<MM>(c, 3);
    ca = c1 - c0;
    cb = c3 - c2;
}

// Smallest |lambda| (geometric multisection on both sides of zero) within
// [L, H]; nu = #eigenvalues below zero.  The candidates are lambda_{nu+1} > 0
// and -lambda_nu > 0: while both can be the smaller, lanes 0..31 and 32..63
// split their log brackets 33 ways; once one is ruled out (or does not
// exist), all 64 lanes split the other's 65 ways.  Rounds continue until the
// log bracket of min |lambda| is 2 rel wide (midpoint error <= rel relative),
// at most `rounds`.
template <int MM>
__device__ __forceinline__ double min_abs_refine(const Shared<MM>& S, int lane, const Spectrum& sp, int nu, double lp,
                                                 double hp, double ln_, double hn, int rounds, double rel) {
    const int m = stencil_m<MM>(S);
    const bool has_pos = nu < m, has_neg = nu > 0;
    for (int rd = 0; rd < rounds; ++rd) {
        // wave-uniform: the brackets are
        const bool need_p = has_pos && !(has_neg && lp > hn);
        const bool need_n = has_neg && !(has_pos && ln_ > hp);
        const double blo = need_p ? (need_n ? fmin(lp, ln_) : lp) : ln_;
        const double bhi = need_p ? (need_n ? fmin(hp, hn) : hp) : hn;
        if (!(bhi - blo > 2.0 * rel)) break;
        if (need_p && need_n) {
            const uint64_t bal = sturm64<MM>(
                S, m, lane, sp.pivmin,
                [&](int l) {
                    const double lo = l >> 5 ? ln_ : lp, hi = l >> 5 ? hn : hp;
                    const double sig = exp(lo + (hi - lo) * (double)((l & 31) + 1) / 33.0);
                    return l >> 5 ? -sig : sig;
                },
                // the target's magnitude lies above: lambda_{nu+1} > sig, or lambda_nu < -sig
                [&](int l, int cnt) { return l >> 5 ? cnt >= nu : cnt <= nu; });
            const int nb1 = __popcll(bal & 0xffffffffull);
            const int nb2 = __popcll(bal >> 32);
            const double a1 = lp + (hp - lp) * (double)nb1 / 33.0, b1 = lp + (hp - lp) * (double)(nb1 + 1) / 33.0;
            const double a2 = ln_ + (hn - ln_) * (double)nb2 / 33.0, b2 = ln_ + (hn - ln_) * (double)(nb2 + 1) / 33.0;
            if (nb1 > 0) lp = a1;
            if (nb1 < 32) hp = b1;
            if (nb2 > 0) ln_ = a2;
            if (nb2 < 32) hn = b2;
        } else {
            const double lo = need_p ? lp : ln_, hi = need_p ? hp : hn;
            const int nb = __popcll(sturm64<MM>(
                S, m, lane, sp.pivmin,
                [&](int l) {
                    const double sig = exp(lo + (hi - lo) * (double)(l + 1) / 65.0);
                    return need_p ? sig : -sig;
                },
                [&](int, int cnt) { return need_p ? cnt <= nu : cnt >= nu; }));
            const double a1 = lo + (hi - lo) * (double)nb / 65.0, b1 = lo + (hi - lo) * (double)(nb + 1) / 65.0;
            const double n_lo = nb > 0 ? a1 : lo, n_hi = nb < 64 ? b1 : hi;
            if (need_p) {
                lp = n_lo;
                hp = n_hi;
            } else {
                ln_ = n_lo;
                hn = n_hi;
            }
        }
    }
    const double pos = has_pos ? exp(0.5 * (lp + hp)) : INFINITY;
    const double neg = has_neg ? exp(0.5 * (ln_ + hn)) : INFINITY;
    return fmin(pos, neg);
}

template <int MM>
__device__ __forceinline__ double spectrum_min_abs_in(const Shared<MM>& S, int lane, const Spectrum& sp, int nu,
                                                      double L, double H, int rounds, double rel) {
    return min_abs_refine<MM>(S, lane, sp, nu, log(L), log(H), log(L), log(H), rounds, rel);
}

// The band test of a learned proposal and the first round of its min |lambda|
// search in one Sturm pass: lanes 0-3 count the eigenvalues with
// |lambda| < tau_a and < tau_b, lane 4 those below zero (nu), and lanes 8-35
// / 36-63 split [tau_b, tau_a] (log scale) 29 ways on the positive / negative
// side.  If the proposal is kept (ca > 0, cb == 0), min |lambda| lies in
// [tau_b, tau_a), and the returned log brackets (lp, hp) and (ln_, hn) are
// those after that first round.
template <int MM>
__device__ __forceinline__ void band_counts_min(const Shared<MM>& S, int lane, const Spectrum& sp, double tau_a,
                                                double tau_b, int& ca, int& cb, int& nu, double& lp, double& hp,
                                                double& ln_, double& hn) {
    const int m = stencil_m<MM>(S);
    const double l0 = log(tau_b), l1 = log(tau_a);
    auto shift = [&](int l) {
        double sig = 0.0;
        if (l == 0) sig = -tau_a;
        if (l == 1) sig = tau_a;
        if (l == 2) sig = -tau_b;
        if (l == 3) sig = tau_b;
        if (l >= 8 && l < 36) sig = exp(l0 + (l1 - l0) * (double)(l - 8 + 1) / 29.0);
        if (l >= 36) sig = -exp(l0 + (l1 - l0) * (double)(l - 36 + 1) / 29.0);
        return sig;
    };
    int c_lane = 0;  // the count of this lane's first shift
    const uint64_t bal = sturm64<MM>(S, m, lane, sp.pivmin, shift, [&](int l, int cnt) {
        if (l < 32) c_lane = cnt;
        if (l < Lay<MM>::LW) nu = from_lane<MM>(cnt, 4);
        // lambda_{nu+1} > sig (positive shifts), lambda_nu < sig (negative ones)
        return l < 8 ? false : (l < 36 ? cnt <= nu : cnt >= nu);
    });
    const int c0 = from_lane<MM>(c_lane, 0), c1 = from_lane<MM>(c_lane, 1);
    const int c2 = from_lane<MM>(c_lane, 2), c3 = from_lane<MM>(c_lane, 3);
    ca = c1 - c0;
    cb = c3 - c2;
    const int nb1 = __popcll((bal >> 8) & 0xfffffffull);
    const int nb2 = __popcll(bal >> 36);
    lp = l0; hp = l1; ln_ = l0; hn = l1;
    if (nb1 > 0) lp = l0 + (l1 - l0) * (double)nb1 / 29.0;
    if (nb1 < 28) hp = l0 + (l1 - l0) * (double)(nb1 + 1) / 29.0;
    if (nb2 > 0) ln_ = l0 + (l1 - l0) * (double)nb2 / 29.0;
    if (nb2 < 28) hn = l0 + (l1 - l0) * (double)(nb2 + 1) / 29.0;
}

// Smallest |lambda| with no prior bracket: [1e-30, 1] x max |lambda|, 7 rounds.
template <int MM>
__device__ __forceinline__ double spectrum_min_abs(const Shared<MM>& S, int lane, const Spectrum& sp) {
    const int nu = sturm<MM>(S, stencil_m<MM>(S), 0.0, sp.pivmin);  // eigenvalues below zero (uniform)
    return spectrum_min_abs_in<MM>(S, lane, sp, nu, sp.amax * 1e-30 + sp.pivmin,
                                   sp.amax * (1.0 + 1e-12) + sp.pivmin, 7, 0.0);
}

// ------------------------------------------------------- tridiagonal solve ----
// Gaussian elimination with partial pivoting of T (one thread); false on a
// zero pivot.  The diagonal and super-diagonal of the row being eliminated are
// carried in registers, so each step reads LDS only for inputs that do not
// depend on the previous step.
template <int MM>
__device__ __forceinline__ bool tri_factor(Shared<MM>& S) {
    const int m = stencil_m<MM>(S);
    double dcur = S.d[0];                      // pivot-row diagonal (after earlier steps)
    double ucur = m > 1 ? S.e[0] : 0.0;        // its super-diagonal
    for (int i = 0; i < m - 1; ++i) {
        const double sub = S.e[i];             // sub-diagonal entry below the pivot
        const double dnext = S.d[i + 1];
        const double unext = i < m - 2 ? S.e[i + 1] : 0.0;
        // The pivot's reciprocal (hardware reciprocal + one Newton step) gives
        // the multiplier too, which keeps a full division off the serial chain.
        if (fabs(dcur) >= fabs(sub)) {
            if (dcur == 0.0) return false;
            const double rp = recip(dcur);
            const double f = sub * rp;
            S.g.fd[i] = rp;                      // reciprocal of the pivot
            S.g.fdu[i] = ucur;
            S.g.fdl[i] = 0.0;
            S.g.ffact[i] = f;
            S.g.fswap[i] = 0;
            dcur = dnext - f * ucur;
            ucur = unext;
        } else {                               // swap rows i and i + 1
            const double rp = recip(sub);
            const double f = dcur * rp;
            S.g.fd[i] = rp;
            S.g.fdu[i] = dnext;
            S.g.fdl[i] = i < m - 2 ? unext : 0.0;  // second super-diagonal
            S.g.ffact[i] = f;
            S.g.fswap[i] = 1;
            dcur = ucur - f * dnext;
            ucur = i < m - 2 ? -f * unext : unext;
        }
    }
    if (dcur == 0.0) return false;
    S.g.fd[m - 1] = recip(dcur);
    S.g.fdu[m - 1] = 0.0;
    S.g.fdl[m - 1] = 0.0;
    return true;
}

// b <- T^{-1} b with the factors of tri_factor (one thread); the running
// entries of b are carried in registers.
template <int MM>
__device__ __forceinline__ void tri_solve(const Shared<MM>& S, double* b) {
    const int m = stencil_m<MM>(S);
    double bi = b[0];
    for (int i = 0; i < m - 1; ++i) {
        const double f = S.g.ffact[i];
        const double bn = b[i + 1];
        if (!S.g.fswap[i]) {
            b[i] = bi;
            bi = bn - f * bi;
        } else {
            b[i] = bn;
            bi = bi - f * bn;
        }
    }
    double x1 = bi * S.g.fd[m - 1];  // x_{i+1}
    b[m - 1] = x1;
    if (m < 2) return;
    double x2 = x1;                // x_{i+2}
    x1 = (b[m - 2] - S.g.fdu[m - 2] * x2) * S.g.fd[m - 2];
    b[m - 2] = x1;
    for (int i = m - 3; i >= 0; --i) {
        const double x = (b[i] - S.g.fdu[i] * x1 - S.g.fdl[i] * x2) * S.g.fd[i];
        b[i] = x;
        x2 = x1;
        x1 = x;
    }
}

// Four waves: y <- Q^T y (FWD) or y <- Q y, for NV = 1 or 3 vectors (thread holds
// component t.c).  The reflector v_k is published through LDS by the row block
// that holds row k.
template <int MM, int NV, bool FWD>
__device__ __forceinline__ void apply_q(const double (&a)[Lay<MM>::R], Shared<MM>& S, const Tid& t, double (&y)[3]) {
    static_assert(MM > 64, "four-wave tiling only");
    const int m = stencil_m<MM>(S);
    #pragma unroll
    for (int kk = 0; kk < MM - 2; ++kk) {
        const int k = FWD ? kk : MM - 3 - kk;  // a compile-time constant after unrolling
        if (k < m - 2) {
            if (t.rb == k / 64) S.g.vb[t.c] = a[k % 64];
            bsync<MM>();
            const double v = S.g.vb[t.c];
            if constexpr (NV == 3) {
                double s0 = v * y[0], s1 = v * y[1], s2 = v * y[2];
                sum_cols3<MM>(s0, s1, s2, S, t);  // ends with a barrier
                const double ta = S.tau[k];
                y[0] = fma(-ta * s0, v, y[0]);
                y[1] = fma(-ta * s1, v, y[1]);
                y[2] = fma(-ta * s2, v, y[2]);
            } else {
                const double s0 = sum_cols<MM>(v * y[0], S, t);
                y[0] = fma(-S.tau[k] * s0, v, y[0]);
            }
        }
    }
}

// One wave, NV vectors: Q^T y (FWD) or Q y four reflectors at a time.
// For a block H_{k0} .. H_{k0+3} the four products d_i = v_i . y of a vector
// are reduced together, and the coupling of successive reflectors inside the
// block comes from their Gram entries G_ij = v_i . v_j (S.G, six per block,
// from reflector_gram): applying H_{k0} first, s_i = d_i - sum_{j<i} tau_j s_j G_ij
// and y -= sum_i tau_i s_i v_i (the reverse order for Q y).  Rows past the last
// reflector enter with v = 0 and tau = 0.
template <int MM, int NV, bool FWD>
__device__ __forceinline__ void apply_q_blocked(const double (&a)[Lay<MM>::R], Shared<MM>& S, double (&y)[3]) {
    static_assert(MM <= 64, "one-wave tiling only");
    const int p = stencil_m<MM>(S) - 2;
#pragma unroll
    for (int bb = 0; bb < Lay<MM>::R / 4; ++bb) {
        const int b = FWD ? bb : Lay<MM>::R / 4 - 1 - bb;
        const int k0 = 4 * b;
        if (k0 < p) {
            const double v0 = a[k0], v1 = k0 + 1 < p ? a[k0 + 1] : 0.0;
            const double v2 = k0 + 2 < p ? a[k0 + 2] : 0.0, v3 = k0 + 3 < p ? a[k0 + 3] : 0.0;
            const double t0 = S.tau[k0], t1 = k0 + 1 < p ? S.tau[k0 + 1] : 0.0;
            const double t2 = k0 + 2 < p ? S.tau[k0 + 2] : 0.0, t3 = k0 + 3 < p ? S.tau[k0 + 3] : 0.0;
            double d[NV][4];
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                d[q][0] = v0 * y[q];
                d[q][1] = v1 * y[q];
                d[q][2] = v2 * y[q];
                d[q][3] = v3 * y[q];
            }
#pragma unroll
            for (int q = 0; q < NV; ++q) wave_sum4<MM>(d[q][0], d[q][1], d[q][2], d[q][3]);
            const double* G = S.g.G + 6 * b;  // G01 G02 G03 G12 G13 G23
            const double g01 = G[0], g02 = G[1], g03 = G[2], g12 = G[3], g13 = G[4], g23 = G[5];
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                double s0, s1, s2, s3;
                if (FWD) {
                    s0 = d[q][0];
                    s1 = fma(-t0 * s0, g01, d[q][1]);
                    s2 = fma(-t1 * s1, g12, fma(-t0 * s0, g02, d[q][2]));
                    s3 = fma(-t2 * s2, g23, fma(-t1 * s1, g13, fma(-t0 * s0, g03, d[q][3])));
                } else {
                    s3 = d[q][3];
                    s2 = fma(-t3 * s3, g23, d[q][2]);
                    s1 = fma(-t2 * s2, g12, fma(-t3 * s3, g13, d[q][1]));
                    s0 = fma(-t1 * s1, g01, fma(-t2 * s2, g02, fma(-t3 * s3, g03, d[q][0])));
                }
                y[q] = fma(-t3 * s3, v3, fma(-t2 * s2, v2, fma(-t1 * s1, v1, fma(-t0 * s0, v0, y[q]))));
            }
        }
    }
}

// S.G for apply_q_blocked (one wave, after the final tridiagonalisation).
template <int MM>
__device__ __forceinline__ void reflector_gram(const double (&a)[Lay<MM>::R], Shared<MM>& S, const Tid& t) {
    static_assert(MM <= 64, "one-wave tiling only");
    const int p = stencil_m<MM>(S) - 2;
#pragma unroll
    for (int b = 0; b < Lay<MM>::R / 4; ++b) {
        const int k0 = 4 * b;
        if (k0 < p) {
            const double v0 = a[k0], v1 = k0 + 1 < p ? a[k0 + 1] : 0.0;
            const double v2 = k0 + 2 < p ? a[k0 + 2] : 0.0, v3 = k0 + 3 < p ? a[k0 + 3] : 0.0;
            double g01 = v0 * v1, g02 = v0 * v2, g03 = v0 * v3, g12 = v1 * v2;
            double g13 = v1 * v3, g23 = v2 * v3, z0 = 0.0, z1 = 0.0;
            wave_sum4<MM>(g01, g02, g03, g12);
            wave_sum4<MM>(g13, g23, z0, z1);
            if (t.tid == 0) {
                double* G = S.g.G + 6 * b;
                G[0] = g01; G[1] = g02; G[2] = g03; G[3] = g12; G[4] = g13; G[5] = g23;
            }
        }
    }
    bsync<MM>();
}

// y <- A~^{-1} y via Q T^{-1} Q^T
template <int MM, int NV>
__device__ __forceinline__ void solve(const double (&a)[Lay<MM>::R], Shared<MM>& S, const Tid& t, double (&y)[3]) {
    const int m = stencil_m<MM>(S);
    if constexpr (MM <= 64) apply_q_blocked<MM, NV, true>(a, S, y);
    else apply_q<MM, NV, true>(a, S, t, y);
    if (t.rb == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) S.g.rhs[v][t.c] = y[v];
    }
    bsync<MM>();
    if (t.tid < NV) tri_solve<MM>(S, S.g.rhs[t.tid]);
    bsync<MM>();
#pragma unroll
    for (int v = 0; v < NV; ++v) y[v] = t.c < m ? S.g.rhs[v][t.c] : 0.0;
    bsync<MM>();
    if constexpr (MM <= 64) apply_q_blocked<MM, NV, false>(a, S, y);
    else apply_q<MM, NV, false>(a, S, t, y);
}

// (A~ z) row t.c for NV vectors read from S.zb; A~ re-evaluated from the nodes
template <int K, int MM, int NV>
__device__ __forceinline__ void matvec_lds(const Shared<MM>& S, const Tid& t, double e2, int us, double (&out)[3]) {
    const int n = stencil_n<MM>(S), m = stencil_m<MM>(S), r = S.r, c = t.c;
    out[0] = out[1] = out[2] = 0.0;
    if (c < n) {
        const double xi = S.x[c], yi = S.y[c], zi = S.z[c];
        for (int j = 0; j < n; ++j) {
            const double dx = xi - S.x[j], dy = yi - S.y[j], dz = zi - S.z[j];
            const double av = rbf_phi<K>(e2, (dx * dx + dy * dy) + dz * dz);
#pragma unroll
            for (int v = 0; v < NV; ++v) out[v] = fma(av, S.g.zb[j], out[v]);
        }
        for (int k = 0; k < r; ++k) {
            const double u = S.U[c * us + k];
#pragma unroll
            for (int v = 0; v < NV; ++v) out[v] = fma(u, S.g.zb[n + k], out[v]);
        }
    } else if (c < m) {
        const int k = c - n;
        for (int j = 0; j < n; ++j) {
            const double u = S.U[j * us + k];
#pragma unroll
            for (int v = 0; v < NV; ++v) out[v] = fma(u, S.g.zb[j], out[v]);
        }
    }
}

// Solve with one step of iterative refinement: z = A~^{-1} b, z += A~^{-1}(b - A~ z).
// The Householder route alone leaves an error several times that of LU with
// partial pivoting on these ill-conditioned saddle systems; one step brings it
// to that level.
template <int K, int MM, int NV>
__device__ __forceinline__ void solve_refined(const double (&a)[Lay<MM>::R], Shared<MM>& S, const Tid& t, double e2, int us,
                                              double (&y)[3]) {
    const double b[3] = {y[0], y[1], y[2]};
    solve<MM, NV>(a, S, t, y);
    if (t.rb == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) S.g.zb[t.c] = y[v];
    }
    bsync<MM>();
    double az[3];
    matvec_lds<K, MM, NV>(S, t, e2, us, az);
    bsync<MM>();
    double r[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int v = 0; v < NV; ++v) r[v] = t.c < stencil_m<MM>(S) ? b[v] - az[v] : 0.0;
    solve<MM, NV>(a, S, t, r);
#pragma unroll
    for (int v = 0; v < NV; ++v) y[v] += r[v];
}

// --------------------------------------------------------------- border ----
// Monomials in xi (order: 1, x, y, z, x^2, y^2, z^2, xy, xz, yz) at row
// jr = 64 rb + lane, orthonormalised by classical Gram-Schmidt applied twice
// (the projections on all earlier kept columns formed together, four sums at
// a time, then subtracted; once more on the result); kept
// columns go to S.U and their monomial coefficients to S.T.  A column is
// dropped when its residual norm is at most rank_tol times the largest column
// norm, that of the ones column (sqrt n; every |xi| <= 1), the analogue of a
// singular value cut relative to the largest one.  (Relative to the column's
// own norm would miss an exact dependency among small columns: at the poles
// of a fine sphere the z^2 column, of norm ~1e-4 sqrt n, keeps a rounding
// residual of 4e-10 of its norm.)  Degree 0 is the plain column of ones.
template <int MM>
__device__ __forceinline__ void build_border(Shared<MM>& S, const Tid& t, int degree, double rank_tol, double xr, double yr,
                             double zr) {
    const int n = stencil_n<MM>(S);
    const int jr = 64 * t.rb + t.lane;
    if (degree == 0) {
        if (t.cb == 0 && jr < n) S.U[jr] = 1.0;
        if (t.tid < RMAX) S.T[t.tid * RMAX] = t.tid == 0 ? 1.0 : 0.0;
        if (t.tid == 0) S.r = 1;
        bsync<MM>();
        return;
    }
    const int M = degree == 1 ? 4 : 10;
    const bool act = jr < n;
    double u[RMAX];
    u[0] = 1.0; u[1] = xr; u[2] = yr; u[3] = zr;
    u[4] = xr * xr; u[5] = yr * yr; u[6] = zr * zr; u[7] = xr * yr; u[8] = xr * zr; u[9] = yr * zr;
#pragma unroll
    for (int l = 0; l < RMAX; ++l)
        if (!act) u[l] = 0.0;
    // thread l (< M) of the stencil holds row l of the coefficient matrix
    double tc[RMAX];
#pragma unroll
    for (int q = 0; q < RMAX; ++q) tc[q] = (t.tid == q) ? 1.0 : 0.0;
    bool keep[RMAX];
    int r = 0;
#pragma unroll
    for (int l = 0; l < RMAX; ++l) {
        keep[l] = false;
        if (l < M) {
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
                double cq[RMAX];
#pragma unroll
                for (int q0 = 0; q0 < l; q0 += 4) {  // constant trip counts: u, tc, keep stay in registers
                    double g[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) g[i] = (q0 + i < l && keep[q0 + i]) ? u[q0 + i] * u[l] : 0.0;
                    sum_rows4<MM>(g[0], g[1], g[2], g[3], S, t);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (q0 + i < l) cq[q0 + i] = g[i];
                }
#pragma unroll
                for (int q = 0; q < l; ++q) {
                    u[l] = fma(-cq[q], u[q], u[l]);
                    tc[l] = fma(-cq[q], tc[q], tc[l]);
                }
            }
            const double n2 = sum_rows<MM>(u[l] * u[l], S, t);
            if (n2 > rank_tol * rank_tol * (double)n && n2 > 0.0) {
                const double inv = 1.0 / sqrt(n2);
                u[l] *= inv;
                tc[l] *= inv;
                keep[l] = true;
                if (act && t.cb == 0) S.U[jr * M + r] = u[l];
                if (t.tid < RMAX) S.T[t.tid * RMAX + r] = tc[l];
                ++r;
            }
        }
    }
    if (t.tid == 0) S.r = r;
    bsync<MM>();
}

// ------------------------------------------------------ kappa evaluations ----
// kappa_2(T) > target ?  (non-finite counts as above, like an infinite kappa)
// kappa > target exactly when some |lambda| < max|lambda| / target.  With
// max |lambda| known to lie in [alo, ahi], an eigenvalue below alo / target
// decides "above" and none below ahi / target decides "not above"; only when
// the two counts differ is max |lambda| refined (two multisection rounds at a
// time), so every decision is the one the Sturm counts of T give at the exact
// max |lambda|, up to a bracket of a few ulps.  sp's brackets are refined in place.
template <int MM>
__device__ __forceinline__ bool kappa_above(const Shared<MM>& S, int lane, Spectrum& sp, double target) {
    if (!sp.finite || !(sp.amax > 0.0)) return true;
    for (int it = 0; it < 12; ++it) {
        double alo, ahi;
        amax_bounds(sp, alo, ahi);
        int ca, cb;
        small_counts<MM>(S, lane, sp, alo / target, ahi / target, ca, cb);
        if (ca > 0) return true;
        if (cb == 0) return false;
        if (ahi - alo <= 8.0 * 2.2e-16 * ahi) break;  // bracket at FP64 resolution
        spectrum_refine<MM>(S, lane, sp, 2);
    }
    int ca, cb;
    small_counts<MM>(S, lane, sp, sp.amax / target, sp.amax / target, ca, cb);
    return ca > 0;
}

// --------------------------------------------------------------- stencil ----
// What process_stencil found before the search: the thread's node, its unit
// normal and scaled offset, the stencil radius, and whether nodes coincide.
struct Gathered {
    double px, py, pz, nx, ny, nz, xi, yi, zi, rho, irho, dupf;
};

// Shape parameter, kappa_2 and weights of stencil s (see process_stencil).
template <int K, int MM>
__device__ __forceinline__ void solve_stencil(const Job& J, int64_t s, Shared<MM>& S, const Tid& t,
                                              const Gathered& G0) {
    const WOpts& o = J.o;
    const int n = o.n, c = t.c, us = border_cols(o.degree);
    const double px = G0.px, py = G0.py, pz = G0.pz, nx = G0.nx, ny = G0.ny, nz = G0.nz;
    const double xi = G0.xi, yi = G0.yi, zi = G0.zi, rho = G0.rho, irho = G0.irho, dupf = G0.dupf;
    int status = RBFFD_ST_OK;
    int evals = 0;
    double a[Lay<MM>::R];
    double eps;
    if (dupf > 0.0) status = RBFFD_ST_DUPLICATE;

    // ---- shape parameter: one evaluation (matrix, tridiagonal form, max |lambda|)
    // per turn of the loop, so that its code is in the kernel once
    enum Phase { LEARN, LOW, HIGH, MID, FINAL };
    double amin_known = 0.0;  // min |lambda| if already found
    double lo = 0.0, hi = 0.0;
    int ph = FINAL, q = 0;
    if (o.mode == RBFFD_EPS_FIXED) {
        eps = o.eps_fixed;
    } else if (o.mode == RBFFD_EPS_GIVEN) {
        eps = J.eps_in[s];
    } else {
        lo = o.br_lo / rho;
        hi = o.br_hi / rho;
        eps = lo;
        ph = LOW;
        if (o.mode == RBFFD_EPS_LEARNED) {
            const double e = J.eps_in[s];
            if (isfinite(e) && e > 0.0) {
                eps = e;
                ph = LEARN;
            } else if (status == RBFFD_ST_OK) {
                status = RBFFD_ST_FALLBACK;
            }
        }
    }
    Spectrum sp{};
    // What follows an evaluation: the next eps (false) or the end (true).
    auto advance = [&]() __attribute__((always_inline)) {
        // max |lambda| of a proposal to band_rel: also the reported kappa's if kept
        sp = spectrum_max<MM>(S, t.lane, ph == FINAL || ph == LEARN ? 8 : 2, ph == LEARN ? o.band_rel : 0.0);
        ++evals;
        if (ph == FINAL) return true;
        const bool good = sp.finite && sp.amax > 0.0;
        if (ph == LEARN) {
            if (good) {
                int c_lo, c_hi, nu;  // |lambda| below amax/band_lo and below amax/band_hi
                const double tau_lo = sp.amax / o.band_lo, tau_hi = sp.amax / o.band_hi;
                double lp, hp, ln_, hn;
                band_counts_min<MM>(S, t.lane, sp, tau_lo, tau_hi, c_lo, c_hi, nu, lp, hp, ln_, hn);
                if (c_lo > 0 && c_hi == 0) {  // band_lo < kappa <= band_hi
                    // min |lambda| lies in [tau_hi, tau_lo): its first round is done
                    amin_known = min_abs_refine<MM>(S, t.lane, sp, nu, lp, hp, ln_, hn, 6, o.band_rel);
                    return true;
                }
            }
            if (status == RBFFD_ST_OK) status = RBFFD_ST_FALLBACK;
            eps = lo;
            ph = LOW;
            return false;
        }
        if (ph == MID && o.band_stop && good) {
            int c_lo, c_hi;
            small_counts<MM>(S, t.lane, sp, sp.amax / o.band_lo, sp.amax / o.band_hi, c_lo, c_hi);
            if (c_lo > 0 && c_hi == 0) {
                // six more rounds: the same brackets as eight from the start,
                // full precision for the reported kappa
                spectrum_refine<MM>(S, t.lane, sp, 6);
                return true;
            }
        }
        const bool above = kappa_above<MM>(S, t.lane, sp, o.kappa_target);
        if (ph == LOW) {
            if (!above && q < o.max_expand) {
                ++q;
                lo *= 0.5;
                eps = lo;
                return false;
            }
            if (!above && status == RBFFD_ST_OK) status = RBFFD_ST_NO_BRACKET;
            q = 0;
            eps = hi;
            ph = HIGH;
            return false;
        }
        if (ph == HIGH) {
            if (above && q < o.max_expand) {
                ++q;
                hi *= 2.0;
                eps = hi;
                return false;
            }
            if (above && status == RBFFD_ST_OK) status = RBFFD_ST_NO_BRACKET;
        } else if (above) {
            lo = eps;
        } else {
            hi = eps;
        }
        ph = hi - lo > o.eps_tol ? MID : FINAL;
        eps = 0.5 * (lo + hi);
        return false;
    };
    // With four waves the first one searches alone (the other three would
    // only repeat it) and hands over eps.
    const bool lead = MM <= 64 || t.rb + t.cb == 0;
    for (;;) {
        build_matrix<K, MM>(a, S, t, eps * eps, us);
        tridiagonalise<MM>(a, S, t, stencil_m<MM>(S));
        bool done = false;
        if (lead) done = advance();
        if constexpr (MM == 128) {
            if (t.tid == 0) {
                S.eps = eps;
                S.done = done;
            }
            bsync<MM>();
            eps = S.eps;
            done = __builtin_amdgcn_readfirstlane(S.done);
        }
        if (done) break;
    }
    // ---- kappa_2 at the final eps
    double kappa = NAN;
    if (!lead) {
        // outputs and the status are the first wave's
    } else if (sp.finite && sp.amax > 0.0) {
        const double amin = amin_known > 0.0 ? amin_known : spectrum_min_abs<MM>(S, t.lane, sp);
        kappa = sp.amax / amin;
    } else if (status == RBFFD_ST_OK) {
        status = RBFFD_ST_NONFINITE;
    }
    if (lead && !sp.finite && status == RBFFD_ST_OK) status = RBFFD_ST_NONFINITE;
    if (t.tid == 0) {
        if (J.eps) J.eps[s] = eps;
        if (J.kappa) J.kappa[s] = kappa;
        if (J.nevals) J.nevals[s] = evals;
    }
    if (J.kappa_only) {
        if (t.tid == 0 && J.status) J.status[s] = status;
        bsync<MM>();
        return;
    }

    // ---- weights: w = (A~^{-1} r)[:n], r = sum_d (B^d)^T g_d, g_d = (A~^{-1} b_d)[:n]
    if (t.tid == 0) S.fact_ok = sp.finite ? (int)tri_factor<MM>(S) : 0;
    bsync<MM>();
    const int m = stencil_m<MM>(S);
    if (!S.fact_ok) {
        if (status == RBFFD_ST_OK) status = sp.finite ? RBFFD_ST_SINGULAR : RBFFD_ST_NONFINITE;
        if (t.tid == 0 && J.status) J.status[s] = status;
        if (c < n && t.rb == 0) J.w[s * n + c] = NAN;
        bsync<MM>();
        return;
    }
    const double e2 = eps * eps;
    const double n0x = S.nrm0[0], n0y = S.nrm0[1], n0z = S.nrm0[2];
    // b_d (row 1 of B^d) as an m-vector, component c
    double b[3] = {0.0, 0.0, 0.0};
    if (c < n) {
        const double dx = S.x[0] - px, dy = S.y[0] - py, dz = S.z[0] - pz;  // x_1 - x_j
        const double r2 = (dx * dx + dy * dy) + dz * dz;
        const double ps = rbf_psi<K>(e2, r2);
        const double dn = n0x * dx + n0y * dy + n0z * dz;
        b[0] = ps * (dx - n0x * dn);
        b[1] = ps * (dy - n0y * dn);
        b[2] = ps * (dz - n0z * dn);
    } else if (c < m && o.degree > 0) {
        const int k = c - n;  // grad q_k at the centre (xi = 0): linear coefficients / rho
        const double gx = S.T[1 * RMAX + k] * irho, gy = S.T[2 * RMAX + k] * irho, gz = S.T[3 * RMAX + k] * irho;
        const double dn = n0x * gx + n0y * gy + n0z * gz;
        b[0] = gx - n0x * dn;
        b[1] = gy - n0y * dn;
        b[2] = gz - n0z * dn;
    }
    if constexpr (MM <= 64) reflector_gram<MM>(a, S, t);
    // g_d: plain solve.  Refining this solve as well as the final one does not
    // lower the error of w (measured against 60-digit weights: both ways
    // 0.02-0.07 kappa u at kappa_T = 1e10 and 1e12; without any refinement
    // 0.1-0.28 kappa u), so only the final solve is refined.
    solve<MM, 3>(a, S, t, b);
    // h_i = Pi_i g_i
    double hx = 0, hy = 0, hz = 0;
    if (c < n) {
        const double dn = nx * b[0] + ny * b[1] + nz * b[2];
        hx = b[0] - nx * dn;
        hy = b[1] - ny * dn;
        hz = b[2] - nz * dn;
    }
    if (t.rb == 0) {
        S.h(0)[c] = hx;
        S.h(1)[c] = hy;
        S.h(2)[c] = hz;
    }
    bsync<MM>();
    // r_j = sum_i psi(r_ij) (x_i - x_j) . h_i   (j = c < n)
    double rj = 0.0;
    const double *hs0 = S.h(0), *hs1 = S.h(1), *hs2 = S.h(2);
    if (c < n) {
#pragma unroll 4
        for (int i = 0; i < n; ++i) {
            const double dx = S.x[i] - px, dy = S.y[i] - py, dz = S.z[i] - pz;
            const double r2 = (dx * dx + dy * dy) + dz * dz;
            const double ps = rbf_psi<K>(e2, r2);
            rj = fma(ps, dx * hs0[i] + dy * hs1[i] + dz * hs2[i], rj);
        }
    }
    // r_{n+k} = sum_i grad q_k(x_i) . h_i
    if (o.degree > 0) {
        const int r = S.r;
        for (int k = 0; k < r; ++k) {
            double cv = 0.0;
            if (c < n) {
                const double* T = S.T;
                double gx = T[1 * RMAX + k], gy = T[2 * RMAX + k], gz = T[3 * RMAX + k];
                if (o.degree == 2) {
                    const double t4 = T[4 * RMAX + k], t5 = T[5 * RMAX + k], t6 = T[6 * RMAX + k];
                    const double t7 = T[7 * RMAX + k], t8 = T[8 * RMAX + k], t9 = T[9 * RMAX + k];
                    gx += 2.0 * t4 * xi + t7 * yi + t8 * zi;
                    gy += 2.0 * t5 * yi + t7 * xi + t9 * zi;
                    gz += 2.0 * t6 * zi + t8 * xi + t9 * yi;
                }
                cv = (gx * hx + gy * hy + gz * hz) * irho;
            }
            cv = sum_cols<MM>(cv, S, t);
            if (c == n + k) rj = cv;
        }
    }
    double wv[3] = {rj, 0.0, 0.0};
    solve_refined<K, MM, 1>(a, S, t, e2, us, wv);
    if (c < n && t.rb == 0) J.w[s * n + c] = wv[0];
    if (t.tid == 0 && J.status) J.status[s] = status;
    bsync<MM>();
}

// The whole computation for stencil s of job J by the waves of one stencil.
template <int K, int MM>
__device__ __forceinline__ void process_stencil(const Job& J, int64_t s, Shared<MM>& S, const Tid& t) {
    const WOpts& o = J.o;
    const int n = o.n;
    const int c = t.c;
    // ---- gather the stencil (thread's column node; rb == 0 threads fill LDS)
    double px = 0, py = 0, pz = 0, nx = 0, ny = 0, nz = 0;
    bool bad = false;   // stencil index outside [0, N): read node 0 instead, flag the stencil
    bool badn = false;  // zero or non-finite normal: Pi_i undefined, flag the stencil
    if (c < n) {
        int64_t node = J.idx[s * n + c];
        bad = node < 0 || node >= J.N;
        if (bad) node = 0;
        px = J.xyz[3 * node];
        py = J.xyz[3 * node + 1];
        pz = J.xyz[3 * node + 2];
        if (J.nrm) {
            nx = J.nrm[3 * node];
            ny = J.nrm[3 * node + 1];
            nz = J.nrm[3 * node + 2];
            const double nn = sqrt(nx * nx + ny * ny + nz * nz);
            badn = !(nn > 0.0 && nn <= 1.79e308);
            const double dn = badn ? 1.0 : nn;
            nx /= dn; ny /= dn; nz /= dn;
        }
        if (t.rb == 0) {
            S.x[c] = px;
            S.y[c] = py;
            S.z[c] = pz;
        }
    }
    if (t.tid == 0) {
        S.nrm0[0] = nx; S.nrm0[1] = ny; S.nrm0[2] = nz;
        S.n = n;
    }
    bsync<MM>();
    // ---- stencil radius, scaled offsets of the thread's column node and row node
    const double dx0 = px - S.x[0], dy0 = py - S.y[0], dz0 = pz - S.z[0];
    const double r20 = c < n ? (dx0 * dx0 + dy0 * dy0) + dz0 * dz0 : 0.0;
    // 3: an index out of range somewhere in the stencil; 2: a zero or
    // non-finite normal; 1: two nodes coincide
    const double flagf =
        max_cols<MM>(bad ? 3.0 : (badn ? 2.0 : ((c > 0 && c < n && r20 == 0.0) ? 1.0 : 0.0)), S, t);
    if (flagf >= 2.0) {
        if (t.tid == 0) {
            if (J.eps) J.eps[s] = NAN;
            if (J.kappa) J.kappa[s] = NAN;
            if (J.nevals) J.nevals[s] = 0;
            if (J.status) J.status[s] = flagf >= 3.0 ? RBFFD_ST_BAD_INDEX : RBFFD_ST_BAD_NORMAL;
        }
        if (!J.kappa_only && c < n && t.rb == 0) J.w[s * n + c] = NAN;
        bsync<MM>();
        return;
    }
    const double dupf = flagf;
    const double rho = sqrt(max_cols<MM>(r20, S, t));
    const double irho = 1.0 / rho;
    const double xi = dx0 / rho, yi = dy0 / rho, zi = dz0 / rho;
    const int jr = 64 * t.rb + t.lane;
    double xr = 0, yr = 0, zr = 0;
    if (jr < n) {
        xr = (S.x[jr] - S.x[0]) / rho;
        yr = (S.y[jr] - S.y[0]) / rho;
        zr = (S.z[jr] - S.z[0]) / rho;
    }
    build_border<MM>(S, t, o.degree, o.rank_tol, xr, yr, zr);
    if (t.tid == 0) S.m = n + S.r;
    bsync<MM>();
    const Gathered G{px, py, pz, nx, ny, nz, xi, yi, zi, rho, irho, dupf};
    if constexpr (Lay<MM>::SPW == 1) {
        solve_stencil<K, MM>(J, s, S, t, G);
    } else {
        // m differs between the halves only where one of them dropped a border
        // column: then they run one after the other, so that m bounds the
        // loops as a scalar.  What is left and whose turn it is are scalar
        // masks, formed before the first pass: a loop on a lane's own flag
        // gets merged into one pass, and a value kept in a vector register
        // across the passes may come back wrong (the compiler reloads such a
        // spilled value where the branches meet, before it restores the mask
        // of active lanes, and with none active nothing is read).
        const int m = S.m;
        uint64_t left = __ballot(true);
        const uint64_t first = __ballot(m == __builtin_amdgcn_readlane(m, __builtin_ctzll(left)));
        for (uint64_t turn = first; left; turn = left) {
            if (__builtin_amdgcn_inverse_ballot_w64(turn)) solve_stencil<K, MM>(J, s, S, t, G);
            left &= ~turn;
        }
    }
}

}  // namespace rbw
