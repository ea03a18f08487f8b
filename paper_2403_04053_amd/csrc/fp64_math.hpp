// FP64 functions of the projection sums: reciprocal distance and sincos of a
// phase of bounded size, in a third of the instructions of the general
// library functions (no scaling of extreme operands, no reduction of huge
// angles) and to the same accuracy (about one unit in the last place).
#pragma once

#include <hip/hip_runtime.h>

namespace pstd {

// r = sqrt(x) and inv = 1 / r for positive normal x: the hardware's reciprocal
// square root (about 2^-27) after one step of Goldschmidt's coupled iteration of
// both, and one residual correction of each.
__device__ __forceinline__ void sqrt_rsqrt(double x, double* r, double* inv) {
    double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    e = fma(-h, g, 0.5);
    h = fma(h, e, h);
    g = fma(fma(-g, g, x), h, g);      // sqrt, residual exact
    y = h + h;
    *inv = fma(fma(-g, y, 1.0), y, y);  // 1 / g
    *r = g;
}

// Largest |x| fast_sincos takes: n = x 2 / pi then has at most 28 bits, the first
// fused product of the reduction below is exact, and the second rounds r once more:
// r is off by at most 2^-54.
constexpr double kFastSincosLimit = 2.0e8;

// sin and cos of |x| <= kFastSincosLimit: x = n pi/2 + r with pi/2 in three
// parts (Cody and Waite's reduction with fused products), then the Taylor
// series of both on |r| <= pi/4, whose first dropped terms are 6e-17 of sin r
// and 2e-18.
__device__ __forceinline__ void fast_sincos(double x, double* sn, double* cs) {
    const double n = rint(x * 0.63661977236758134308);  // 2 / pi
    double r = fma(-n, 1.57079632679489655800e+00, x);
    r = fma(-n, 6.12323399573676603587e-17, r);
    r = fma(-n, -1.49738490485916983271e-33, r);
    const double z = r * r;
    double s = -1.0 / 1307674368000.0;
    s = fma(s, z, 1.0 / 6227020800.0);
    s = fma(s, z, -1.0 / 39916800.0);
    s = fma(s, z, 1.0 / 362880.0);
    s = fma(s, z, -1.0 / 5040.0);
    s = fma(s, z, 1.0 / 120.0);
    s = fma(s, z, -1.0 / 6.0);
    s = fma(s * z, r, r);
    double c = 1.0 / 20922789888000.0;
    c = fma(c, z, -1.0 / 87178291200.0);
    c = fma(c, z, 1.0 / 479001600.0);
    c = fma(c, z, -1.0 / 3628800.0);
    c = fma(c, z, 1.0 / 40320.0);
    c = fma(c, z, -1.0 / 720.0);
    c = fma(c, z, 1.0 / 24.0);
    c = fma(c, z, -0.5);
    c = fma(c, z, 1.0);
    const int q = (int)n;
    const double a = (q & 1) ? c : s, b = (q & 1) ? s : c;
    *sn = (q & 2) ? -a : a;
    *cs = ((q + 1) & 2) ? -b : b;
}

}  // namespace pstd
