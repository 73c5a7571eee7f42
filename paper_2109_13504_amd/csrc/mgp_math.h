// mgp_math.h -- the fp64 functions of the SIR model (stage 1), for the
// arguments that occur there.
//
// Stage 1 is bound by fp64 VALU issue, and the general library functions
// spend much of it on arguments that cannot occur: a sincos that reduces any
// double modulo 2 pi, a log and an exp with subnormal and overflow paths, a
// division scaled against overflow. Here the angle comes as a fraction of a
// turn in 32 bits, whose quadrant is two bits of it; the logarithm's argument
// is a count over 2^32; the exponent is negative; the divisor is at least 1.
// Instructions per particle of a predict/update step: 138 instead of 186.
//
// Accuracy: worst error over 2^24 arguments of each, in units in the last
// place against 64-bit-mantissa arithmetic, and the library function's on the
// same arguments:
//   neg_log_fraction  0.68, a little more than log's 0.65 (mean 0.251, 0.252)
//   exp_negative      0.84 (exp 0.86)    sqrt_positive 0.50 (sqrt 0.50)
//   sincos_turn       1.84; absolute 2.2e-16, against 6.9e-16 of sincos on
//                     the angle 2 pi b 2^-32 rounded to fp64, whose relative
//                     error has no bound near its zeros
// What the model takes from them, the normal draw sqrt(-2 ln u1) cos or sin of
// 2 pi u2, is off by 1.3e-15 at most and 6.0e-17 on average over 2^25 draws,
// with the library's functions by 3.0e-15 and 1.5e-16: the angle's rounding
// outweighs the logarithm's 0.03 units.
// ratio() equals IEEE division on all of them. twentieth() rounds correctly.
// Methods: the logarithm's reduction to [sqrt(1/2), sqrt(2)) by the high word,
// its form f - s (f - R) and the split of ln 2 are those of fdlibm's log (Sun
// Microsystems, 1993; FreeBSD's and musl's); the exponential reduces by k ln 2 in
// the same two parts (Cody and Waite); the square root is the coupled Newton
// iteration for sqrt(x) and 1 / (2 sqrt(x)) (Goldschmidt). The polynomials are
// this file's own: Chebyshev interpolants of the functions named beside them,
// computed in 60 digits; each term is the next power of the argument.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace mgp {

template <int N>
__device__ __forceinline__ double horner(const double (&c)[N], double x)
{
    double r = c[N - 1];
#pragma unroll
    for (int k = N - 2; k >= 0; --k) r = fma(r, x, c[k]);
    return r;
}

// 1/d to about 2^-47 for a normal d: the hardware estimate (2^-24) and one
// Newton step. The callers' last step corrects the quotient itself.
__device__ __forceinline__ double rough_reciprocal(double d)
{
    const double r = __builtin_amdgcn_rcp(d);
    return fma(r, fma(-d, r, 1.0), r);
}

// a / d for |d| between 1 and 1e300 and a of a magnitude that keeps the
// quotient normal or zero; NaN when either is NaN or both are infinite.
__device__ __forceinline__ double ratio(double a, double d)
{
    const double r = rough_reciprocal(d);
    const double q = a * r;
    return fma(fma(-q, d, a), r, q);
}

// a / 20 for a finite a.
__device__ __forceinline__ double twentieth(double a)
{
    const double q = a * 0x1.999999999999ap-5;
    return fma(fma(-q, 20.0, a), 0x1.999999999999ap-5, q);
}

// -ln((a + 1) 2^-32) >= 0. With (a + 1) = 2^k m, m in [sqrt(1/2), sqrt(2)),
// f = m - 1 and s = f / (2 + f): ln m = 2 atanh(s) = f - s (f - z Q(z)),
// z = s^2, Q(z) = 2 (atanh(s) / s - 1) / z on [0, 0.0295] (relative error of
// ln m below 2^-57). f is exact, so the rounding errors of s weigh at most a
// fifth.
__device__ __forceinline__ double neg_log_fraction(uint32_t a)
{
    constexpr double Q[7] = {0x1.5555555555558p-1, 0x1.99999999952d7p-2, 0x1.2492492df281ap-2, 0x1.c71c62e3f11e6p-3,
                             0x1.7462b51cb66b1p-3, 0x1.39fe51a7c18f9p-3, 0x1.2b5900de53b32p-3};
    constexpr double kLn2Hi = 0x1.62e42feep-1, kLn2Lo = 0x1.a39ef35793c76p-33;  // 32 leading bits, the rest
    const double x = (double)a + 1.0;
    // high words: 0x3FF00000 is 1.0, 0x3FE6A09E just below sqrt(1/2)
    const int t = __double2hiint(x) + (0x3FF00000 - 0x3FE6A09E);
    const double k = (double)((t >> 20) - 0x3FF - 32);
    const double m = __hiloint2double((t & 0xFFFFF) + 0x3FE6A09E, __double2loint(x));
    const double f = m - 1.0;
    const double d = 2.0 + f;
    const double r = rough_reciprocal(d);
    const double q = f * r;
    const double rest = fma(-q, d, f);
    const double s = fma(rest, r, q);
    const double s_lo = fma(rest, r, q - s);  // what s lost
    const double z = s * s;
    // s (z Q - f), the product with f exact inside the multiply-add
    const double small = fma(-s, f, fma(-s_lo, f, fma(k, kLn2Lo, s * (z * horner(Q, z)))));
    // k kLn2Hi (exact) + f with the rounding error kept: |k ln 2| >= |f| or k = 0
    const double big = k * kLn2Hi;
    const double hi = big + f;
    return -(hi + ((f - (hi - big)) + small));
}

// sqrt(x) for x = 0 or x in [2^-40, 2^40]: the hardware estimate of
// 1 / sqrt(x) (2^-24), one coupled Newton step for sqrt(x) and
// 1 / (2 sqrt(x)), and a correction of the root by its own residual.
__device__ __forceinline__ double sqrt_positive(double x)
{
    x = fmax(x, 0x1p-1000);  // 0: a root of 2^-500, which vanishes in any sum with a normal fp32 result
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, x), h, g);
}

// sin and cos of 2 pi b 2^-32: the nearest quarter turn by the top bits of b,
// then x = 2 pi r 2^-32 in [-pi/4, pi/4] for the exact rest r;
// sin x = x + x z S(z), cos x = 1 - z/2 + z^2 C(z), z = x^2 (relative errors
// below 2^-55 and 2^-59).
__device__ __forceinline__ void sincos_turn(uint32_t b, double& sn, double& cs)
{
    constexpr double S[6] = {-0x1.5555555555555p-3, 0x1.1111111110bb2p-7, -0x1.a01a019e83816p-13,
                             0x1.71de379654304p-19, -0x1.ae600aca92c64p-26, 0x1.5e0b05bff20f2p-33};
    constexpr double C[6] = {0x1.5555555555555p-5, -0x1.6c16c16c16967p-10, 0x1.a01a019f4e9b4p-16,
                             -0x1.27e4fa17bf139p-22, 0x1.1eeb68cd22f56p-29, -0x1.907d8f29fe831p-37};
    const uint32_t q = (b + 0x20000000u) >> 30;
    const double x = (double)(int32_t)(b - (q << 30)) * 0x1.921fb54442d18p-30;  // 2 pi 2^-32
    const double z = x * x;
    const double s = fma(x * z, horner(S, z), x);
    const double c = fma(z * z, horner(C, z), fma(-0.5, z, 1.0));
    const bool odd = (q & 1u) != 0;
    const double a = odd ? c : s, d = odd ? s : c;
    // sin changes sign in quarters 2 and 3, cos in 1 and 2
    sn = __hiloint2double(__double2hiint(a) ^ (int)((q & 2u) << 30), __double2loint(a));
    cs = __hiloint2double(__double2hiint(d) ^ (int)(((q + 1u) & 2u) << 30), __double2loint(d));
}

// exp(y) for y <= 0 as an fp32 result needs it: below -200 (e^-200 is 0 in
// fp32) it may return any value that rounds to 0. NaN for NaN.
// y = k ln 2 + r, exp(r) = 1 + r + r^2 P(r) on [-0.347, 0.347] (relative error
// below 2^-61).
__device__ __forceinline__ double exp_negative(double y)
{
    constexpr double P[11] = {0.5, 0x1.5555555555557p-3, 0x1.5555555555556p-5, 0x1.11111111100dcp-7,
                              0x1.6c16c16c162d4p-10, 0x1.a01a01abe7fe1p-13, 0x1.a01a01a6d889cp-16,
                              0x1.71de0231960ebp-19, 0x1.27e4db646b17ep-22, 0x1.af4de97ca4194p-26,
                              0x1.1f730349868cep-29};
    constexpr double kLn2Hi = 0x1.62e42feep-1, kLn2Lo = 0x1.a39ef35793c76p-33;
    y = y < -200.0 ? -200.0 : y;
    const double k = rint(y * 0x1.71547652b82fep+0);
    const double t = fma(-k, kLn2Hi, y);  // exact
    const double r = fma(-k, kLn2Lo, t);
    const double rest = fma(-k, kLn2Lo, t - r);  // what r lost
    return ldexp(1.0 + (r + fma(r * r, horner(P, r), rest)), (int)k);
}

}  // namespace mgp
