// Numbers m 2^k of the fp64 lattice sweep, and their way from and to natural logarithms.  (Read by a host compiler, too.)
//
// Every function is good to the last place or two of fp64: an error of one sign per step would stay in a sweep of T + U steps and grow with it.
#pragma once

#include <cmath>

#ifdef __HIPCC__
#define RNNT_SCALED __device__ __forceinline__
#else
#define RNNT_SCALED inline
#endif

namespace rnnt {

struct Scaled {
    double m, k;
};
constexpr double LOG2E_D = 1.4426950408889634074, LN2_D = 0.69314718055994530942;

// 2^x, |x| <= 1/2: the polynomial of degree 10 that meets 2^x at the zeros of the Chebyshev polynomial T_11 (coefficients from a solution of those eleven
// equations in 60 digits).  Relative error up to 3.1e-16 ahead of its roundings, of either sign, on average 5e-19; the Taylor series of the same length is
// off by 2.2e-13.
RNNT_SCALED double exp2_half(double x) {
    constexpr double c[11] = {1.0, 0.69314718055995, 0.24022650695910097, 0.05550410866444772, 0.009618129107606888, 0.0013333558230164974,
                              1.540353044173605e-4, 1.5252657260200837e-5, 1.321544258792169e-6, 1.0208690299958306e-7, 7.072585949269223e-9};
    double r = c[10];
#pragma unroll
    for (int i = 9; i >= 0; --i) r = fma(r, x, c[i]);
    return r;
}
// e^x
RNNT_SCALED Scaled scaled_exp(double x) {
#ifdef __clang__
#pragma clang fp contract(off)      // (y - k is at most 1/2, and 0 for an emission of EMISSION_FLOOR, only with y rounded)
#endif
    const double y = x * LOG2E_D, k = rint(y);
    return {exp2_half(y - k), k};
}
RNNT_SCALED Scaled times(const Scaled& a, const Scaled& b) { return {a.m * b.m, a.k + b.k}; }
// m 2^d, d <= 0 a whole number (far below the exponents of fp64: 0)
RNNT_SCALED double scale_down(double m, double d) { return ldexp(m, (int)fmax(d, -4000.0)); }
RNNT_SCALED Scaled plus(const Scaled& a, const Scaled& b) {
    const double k = fmax(a.k, b.k);
    return {scale_down(a.m, a.k - k) + scale_down(b.m, b.k - k), k};
}
// m = f 2^e, f in [1/2, 1)
RNNT_SCALED double mantissa(double m, int& e) {
#ifdef __HIP_DEVICE_COMPILE__
    e = __builtin_amdgcn_frexp_exp(m);
    return __builtin_amdgcn_frexp_mant(m);
#else
    return std::frexp(m, &e);
#endif
}
// ln(m 2^k), m > 0: an fp32 logarithm, and what it leaves over: the logarithm of 1 + d, |d| below 1e-6, by two terms
RNNT_SCALED double scaled_log(const Scaled& a) {
    int e;
    const double f = mantissa(a.m, e) * 1.41421356237309504880;      // [0.71, 1.42)
#ifdef __HIP_DEVICE_COMPILE__
    const double l = (double)__builtin_amdgcn_logf((float)f);
#else
    const double l = (double)std::log2((float)f);
#endif
    const double d = fma(f, exp2_half(-l), -1.0);
    return fma(l + (a.k + (e - 0.5)), LN2_D, fma(-0.5 * d, d, d));
}

}  // namespace rnnt
