// Device-side cos and sin of integer multiples of an angle.
#pragma once

#include <hip/hip_runtime.h>

namespace zp {

// cos and sin of alpha theta for many alpha at one theta.  theta in quarter
// turns, theta 2/pi, is kept as an unevaluated sum hi + lo, formed once per
// point; alpha (hi + lo) less its nearest integer is then good to rounding
// (the product alpha hi is exact inside the fused multiply-add), and the
// Taylor polynomials of sin (to x^15) and cos (to x^16) on [-pi/4, pi/4] are
// within a rounding of the functions.  About 40 instructions, where a general
// sincos takes about 150.  Whole turns are taken off first, so that any finite
// theta gives values in range; the sum carries 106 bits, so the angle is good
// to rounding for |theta| up to about 2^50 / alpha.
struct Turn {
    double hi, lo;
    __device__ __forceinline__ explicit Turn(double theta)
    {
        constexpr double k2pi_hi = 0x1.45f306dc9c883p-1, k2pi_lo = -0x1.6b01ec5417056p-55; // 2/pi
        const double h = theta * k2pi_hi;
        const double l = __builtin_fma(theta, k2pi_lo, __builtin_fma(theta, k2pi_hi, -h));
        const double h4 = __builtin_fma(-4.0, __builtin_rint(0.25 * h), h);
        const double l4 = __builtin_fma(-4.0, __builtin_rint(0.25 * l), l);
        hi = h4 + l4;
        lo = l4 - (hi - h4);
    }
    __device__ __forceinline__ Turn() {}
    __device__ __forceinline__ void angle(double fa, double &cs, double &sn) const
    {
        const double n = __builtin_rint(fa * hi);
        const double f = __builtin_fma(fa, lo, __builtin_fma(fa, hi, -n));
        constexpr double pio2_hi = 0x1.921fb54442d18p+0, pio2_lo = 0x1.1a62633145c07p-54; // pi/2
        const double x = __builtin_fma(f, pio2_hi, f * pio2_lo);
        const double z = x * x;
        double ps = -1.0 / 1307674368000.0, pc = 1.0 / 20922789888000.0; // 1/15!, 1/16!
        ps = __builtin_fma(ps, z, 1.0 / 6227020800.0);
        pc = __builtin_fma(pc, z, -1.0 / 87178291200.0);
        ps = __builtin_fma(ps, z, -1.0 / 39916800.0);
        pc = __builtin_fma(pc, z, 1.0 / 479001600.0);
        ps = __builtin_fma(ps, z, 1.0 / 362880.0);
        pc = __builtin_fma(pc, z, -1.0 / 3628800.0);
        ps = __builtin_fma(ps, z, -1.0 / 5040.0);
        pc = __builtin_fma(pc, z, 1.0 / 40320.0);
        ps = __builtin_fma(ps, z, 1.0 / 120.0);
        pc = __builtin_fma(pc, z, -1.0 / 720.0);
        ps = __builtin_fma(ps, z, -1.0 / 6.0);
        pc = __builtin_fma(pc, z, 1.0 / 24.0);
        const double s = __builtin_fma(x * z, ps, x);
        const double c = __builtin_fma(z, __builtin_fma(pc, z, -0.5), 1.0);
        const int q = (int)n;
        const double a = q & 1 ? c : s, b = q & 1 ? s : c;
        sn = q & 2 ? -a : a;
        cs = (q + 1) & 2 ? -b : b;
    }
};

} // namespace zp
