// zmc_trig.hpp -- FP64 sine and cosine for the sampling kernels, shared by
// the precompiled integrands and the run-time compiled ones.
//
// For |t| <= kTrigMax: t = n pi/2 + (r + rl) with n = rint(2 t / pi), r in
// [-pi/4, pi/4] and |rl| far below r's last place or, beside a multiple of
// pi/2, far below r, and the quadrant n mod 4 picks +-sin(r + rl) or
// +-cos(r + rl).  The reduction is Cody and Waite's (pi/2 in three parts), in
// fused operations:
//   - r1 = t - n hi is exact: a multiple of 2^-53 below one in magnitude;
//   - n mid is exact (16 bits by 37) and r = r1 - n mid is rounded once.  What
//     that rounding lost, (r1 - r) - n mid, is formed exactly: where n mid is
//     the larger, r1 is a multiple of 2^-53 below 2^-38 and the difference of
//     two multiples of 2^-90 is exact; where it cancels against r1, r is exact
//     and r1 - r is n mid; else r1 - r is exact, r1 being the larger operand;
//   - rl takes that and n lo; what is left of pi/2, 2^-147, is below 1e-39 and
//     no double up to kTrigMax is nearer than 1e-19 to a multiple of pi/2.
// The values are a truncated series with the reduction's tail (the cosine's
// leading 1 - r^2/2 rounded, and what that lost added back, as in the classic
// kernel functions of Ng):
//     sin(r + rl) = r + (r^3 (-1/6 + r^2 P(r^2)) + rl w),   w = 1 - r^2/2,
//     cos(r + rl) = w + (r^4 Q(r^2) + ((1 - w) - r^2/2 - r rl)),
// -1/6 + r^2 P and Q the interpolating polynomials of (sin(r)/r - 1)/r^2 and
// (cos(r) - 1 + r^2/2)/r^4 at the Chebyshev nodes of r^2 in [0, (pi/4)^2].
// No branch and no table: 36 FP64 and integer instructions a value, where
// the library's functions take about 50 around a branch to their reduction
// of huge arguments.  Error against values of 113 bits, a million arguments up
// to 0.8 .. 65000: at most 0.78 ulp, 0.2906 rms (the library: 0.78 and
// 0.2932); at the doubles nearest the multiples of pi/2: at most 0.50 ulp.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zmc {

// Beyond it the library's functions take over: n has 16 bits here, so that its
// product with the middle part of pi/2 is exact.
constexpr double kTrigMax = 65536.0;

// QUARTERS = 0: sin(t); 1: cos(t) = sin(t + pi/2).
template <int QUARTERS>
__device__ __forceinline__ double trig_reduced(double t)
{
    // pi/2 = hi + mid + lo: 53, 37 and 53 bits
    constexpr double kHalfPiHi = 0x1.921fb54442d18p+0, kHalfPiMid = 0x1.1a6263314p-54,
                     kHalfPiLo = 0x1.701b839a25205p-92;
    constexpr double kRound = 6755399441055744.0; // 1.5 * 2^52: n lands in the low word
    const double y = fma(t, 0.6366197723675814, kRound);
    const double n = y - kRound;
    const uint32_t k = (uint32_t)__double2loint(y) + (uint32_t)QUARTERS;
    const double r1 = fma(-n, kHalfPiHi, t);
    const double r = fma(-n, kHalfPiMid, r1);
    const double rl = fma(-n, kHalfPiLo, fma(-n, kHalfPiMid, r1 - r));
    const double z = r * r;
    double p = 1.5917988979397432e-10;
    p = fma(p, z, -2.5051129896450185e-08);
    p = fma(p, z, 2.7557316093198404e-06);
    p = fma(p, z, -0.00019841269836740532);
    p = fma(p, z, 0.008333333333330936);
    double q = -1.138254464534925e-11;
    q = fma(q, z, 2.087614504941318e-09);
    q = fma(q, z, -2.755731726587808e-07);
    q = fma(q, z, 2.48015872987544e-05);
    q = fma(q, z, -0.0013888888888887389);
    q = fma(q, z, 0.041666666666666664);
    const double hr = -0.5 * r, rz = r * z;
    const double w = fma(hr, r, 1.0);
    const double e = fma(hr, r, 1.0 - w); // what rounding w lost
    const double s = r + fma(rz, -0.16666666666666666, fma(rz, z * p, rl * w));
    const double c = w + fma(z * z, q, fma(-r, rl, e));
    // odd quadrants take the cosine, quadrants 2 and 3 the negated value
    const uint32_t odd = (uint32_t)((int32_t)(k << 31) >> 31);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_bitop3_b32(odd, (uint32_t)__double2loint(c), (uint32_t)__double2loint(s), 0xCA);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_bitop3_b32(odd, (uint32_t)__double2hiint(c), (uint32_t)__double2hiint(s), 0xCA);
    return __hiloint2double((int)(hi ^ ((k << 30) & 0x80000000u)), (int)lo);
}

// The check is on the upper word without its sign: zero and what is below
// 2^-1042 go to the library too, which keeps the sign of a zero (the reduced
// form gives +0 for -0).
__device__ __forceinline__ double sin_f64(double t)
{
    constexpr uint32_t kTop = 0x40F00000u; // of kTrigMax
    if (__builtin_expect(((uint32_t)__double2hiint(t) << 1) - 2u < (kTop << 1) - 2u, 1)) return trig_reduced<0>(t);
    return ::sin(t);
}

__device__ __forceinline__ double cos_f64(double t)
{
    if (__builtin_expect(fabs(t) <= kTrigMax, 1)) return trig_reduced<1>(t);
    return ::cos(t);
}

} // namespace zmc
