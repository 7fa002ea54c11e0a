// FP64 sine and cosine of phases given in half turns (units of pi).
#pragma once

#include "common.hpp"

namespace chaff {

constexpr double PI_H = 3.14159265358979323846;

// All arguments are kept in half turns (units of pi), so that the range reduction
// is one exact subtraction of a whole number instead of the library's reduction by
// multiples of pi/2, and the quadrant is a sign.

// a t + c with the coefficient in a scalar register pair: left to itself the
// compiler moves every coefficient into vector registers first, one move per
// step of the series.
__device__ __forceinline__ double horner(double a, double t, double c) {
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(t), "s"(c));
    return d;
}
// sr = sin(pi x) / (pi x), c = cos(pi x): Taylor series in x^2; for |x| <= 1/4 the
// first omitted terms are 6e-17 and 2e-18
__device__ __forceinline__ void sinccospi_small(double x, double& sr, double& c) {
    const double t = (PI_H * x) * (PI_H * x);
    double p = horner(t, -1.0 / 1307674368000.0, 1.0 / 6227020800.0);
    p = horner(p, t, -1.0 / 39916800.0);
    p = horner(p, t, 1.0 / 362880.0);
    p = horner(p, t, -1.0 / 5040.0);
    p = horner(p, t, 1.0 / 120.0);
    p = horner(p, t, -1.0 / 6.0);
    sr = fma(p, t, 1.0);
    double q = horner(t, 1.0 / 20922789888000.0, -1.0 / 87178291200.0);
    q = horner(q, t, 1.0 / 479001600.0);
    q = horner(q, t, -1.0 / 3628800.0);
    q = horner(q, t, 1.0 / 40320.0);
    q = horner(q, t, -1.0 / 720.0);
    q = horner(q, t, 1.0 / 24.0);
    q = fma(q, t, -0.5);
    c = fma(q, t, 1.0);
}
// sine and cosine of pi (n / 2 + y), n whole, |y| at most a quarter and a little
__device__ __forceinline__ void sincospi_quarter(double n, double y, double& s, double& c) {
    double sn, cs;
    sinccospi_small(y, sn, cs);
    sn *= PI_H * y;
    const int k = (int)(n - 4.0 * floor(0.25 * n));   // quadrant, exact below 2^53
    const double a = (k & 1) ? cs : sn, b = (k & 1) ? sn : cs;
    s = (k & 2) ? -a : a;
    c = ((k + 1) & 2) ? -b : b;
}
// sin(pi x), cos(pi x) for any finite x (exact quadrant: 2 x - rint(2 x) is exact)
__device__ __forceinline__ void sincospi_any(double x, double& s, double& c) {
    const double n = rint(2.0 * x);
    sincospi_quarter(n, fma(-0.5, n, x), s, c);
}
// the same of x + lo: a phase and, far below a quarter, the part that its rounding left
__device__ __forceinline__ void sincospi_sum(double x, double lo, double& s, double& c) {
    const double n = rint(2.0 * x);
    sincospi_quarter(n, fma(-0.5, n, x) + lo, s, c);
}

}  // namespace chaff
