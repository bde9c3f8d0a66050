// Device helpers of the double-precision kernels: the cell operator of the f(R) equation
// in the variable u (f~_R = -exp(u)), eq. discrete_fR times c~^2 (= eq. bc_modified_fR_op
// for a cell with no ghost neighbour) and its diagonal derivative (eq. bc_modified_fR_dop).
#pragma once

#include "mgfr_impl.h"

namespace mgfr {
namespace dev {

struct OpVal {
    double L, dL;
};

// exp(x) to within one unit in the last place: x = k ln 2 + r with |r| <= ln 2 / 2 (Cody and
// Waite, ln 2 in two parts), exp(r) = 1 + r + r^2 / 2 + r^3 s(r), s of degree 9 with the least
// largest relative error of the sum (Remez' exchange; 7.9e-19 with its coefficients rounded).  Over
// 16 million arguments in each of [-700, 0], [-40, 0] and [0, 40] at most 0.867 units off, the library
// function 0.875, and 0.301 and 0.302 in the mean square (one degree less 0.883 and 0.302, for 0.3% of
// a 512^3 solve and 1% of a masked one).  Overflows to infinity, is zero below -746 (the smallest
// denormal is exp(-745.13...)) and NaN at NaN, always with the sign clear: k is capped so that r
// stays positive above the range.  The polynomial is written out with its coefficients in
// scalar registers because the compiler turns such a chain into v_fmac, whose addend is its
// destination, and copies each constant into vector registers first.  22 instructions against
// the library function's 31; the sweeps evaluate three per thread and step.
__device__ __forceinline__ double exp_(double x)
{
    const double k = __builtin_fmin(__builtin_rint(x * 1.4426950408889634), 1100.0);
    double r = __builtin_fma(k, -0x1.62e42fefa39efp-1, x);
    r = __builtin_fma(k, -0x1.abc9e3b39803fp-56, r);
    double q;
    asm("v_fma_f64 %0, %1, %2, %3\n\t"
        "v_fma_f64 %0, %0, %1, %4\n\t"
        "v_fma_f64 %0, %0, %1, %5\n\t"
        "v_fma_f64 %0, %0, %1, %6\n\t"
        "v_fma_f64 %0, %0, %1, %7\n\t"
        "v_fma_f64 %0, %0, %1, %8\n\t"
        "v_fma_f64 %0, %0, %1, %9\n\t"
        "v_fma_f64 %0, %0, %1, %10\n\t"
        "v_fma_f64 %0, %0, %1, %11\n\t"
        "v_fma_f64 %0, %0, %1, 0.5\n\t"
        "v_fma_f64 %0, %0, %1, 1.0\n\t"
        "v_fma_f64 %0, %0, %1, 1.0"
        : "=&v"(q)
        : "v"(r), "v"(0x1.1e67095a238dcp-29), "s"(0x1.af68a1ed6659ap-26), "s"(0x1.27e58d2d3339ap-22),
          "s"(0x1.71ddf24c3ce9ap-19), "s"(0x1.a01a015246db3p-16), "s"(0x1.a01a01b276d13p-13),
          "s"(0x1.6c16c16c270dfp-10), "s"(0x1.111111110efa1p-7), "s"(0x1.5555555555530p-5),
          "s"(0x1.555555555555ap-3));
    q = __builtin_amdgcn_ldexp(__builtin_fabs(q), (int)k);
    return x < -746.0 ? 0.0 : q;
}

// Curvature term S = A exp(-u/(n+1)).  For n = 1 it is A / sqrt(b) with b = exp(u) already
// at hand: the hardware reciprocal square root refined by two Newton steps (each doubles
// the correct bits), instead of a second double-precision exponential.
__device__ __forceinline__ double curvature(const Grid& g, double ui, double bi)
{
    if (g.half_power) {
        double y = __builtin_amdgcn_rsq(bi);
        double e = fma(-bi * y, y, 1.0);
        y = fma(0.5 * y, e, y);
        e = fma(-bi * y, y, 1.0);
        y = fma(0.5 * y, e, y);
        return g.A * y;
    }
    return g.A * exp_(-ui * g.inv_np1);
}

// L_i - f_i and dL_i/du_i from the cell value, its six neighbours and their b = exp(u).
__device__ __forceinline__ OpVal cell_op_b(const Grid& g, double ui, double bi, const double (&un)[6],
                                           const double (&bn)[6], double f)
{
    // the sums start from the first neighbour: an addition of zero is not folded away
    double su = un[0] - ui, sb = bn[0], sbu = bn[0] * su;
#pragma unroll
    for (int q = 1; q < 6; ++q) {
        const double du = un[q] - ui;
        su += du;
        sb += bn[q];
        sbu = fma(bn[q], du, sbu);
    }
    const double S = curvature(g, ui, bi);
    OpVal r;
    // sum_nb (b_nb + b_i)(u_nb - u_i) = sum b_nb du + b_i sum du
    r.L = g.C * fma(bi, su, sbu) + S - f;
    // sum_nb [b_i (u_nb - u_i) - b_nb - b_i]
    r.dL = g.C * (fma(bi, su, -sb) - 6.0 * bi) - S * g.inv_np1;
    return r;
}

__device__ __forceinline__ OpVal cell_op(const Grid& g, double ui, const double (&un)[6], double f)
{
    double bn[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) bn[q] = exp_(un[q]);
    return cell_op_b(g, ui, exp_(ui), un, bn, f);
}

__device__ __forceinline__ double rhs_value(const Grid& g, double src)
{
    return fma(g.fscale, src - g.sref, g.fshift);
}

__device__ __forceinline__ long long at(const Grid& g, int i, int j, int k)
{
    return ((((long long)i << g.lg) + j) << g.lg) + k;
}

// Newton step, bounded to [-ms, ms] when ms > 0; comparisons (not fmin/fmax) keep a NaN step NaN.
__device__ __forceinline__ double bounded(double step, double ms)
{
    if (ms > 0.0) {
        if (step > ms) step = ms;
        if (step < -ms) step = -ms;
    }
    return step;
}

}  // namespace dev
}  // namespace mgfr
