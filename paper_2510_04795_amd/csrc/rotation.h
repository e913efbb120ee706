// The plane rotation of the Jacobi eigensolvers.
#pragma once

#include <hip/hip_runtime.h>

namespace oz {

// Rotation that zeroes a_pq of [[app, apq], [apq, aqq]] by the smaller angle
// a: with x = aqq - app, y = 2 apq (scaled by a power of two so the squares
// stay in range) and r = sqrt(x^2 + y^2), cos 2a = |x| / r, so c^2 = (1 +
// |x| / r) / 2 and s = sgn(x) y / (2 r c): two reciprocal square roots in a
// row and no division.  Each is the hardware's estimate (about 2^-23) with one
// third-order correction; c^2 + s^2 = 1 to a few rounding errors.
__device__ __forceinline__ double rsqrt_refined(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}
__device__ __forceinline__ void schur_rotation(double app, double aqq, double apq, double *c, double *s) {
    double x = aqq - app, y = 2.0 * apq;
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(x), fabs(y)));
    x = ldexp(x, ex);
    y = ldexp(y, ex);
    const double r2 = fma(x, x, y * y);
    const double ir = rsqrt_refined(r2);
    const double cc = fma(0.5 * fabs(x), ir, 0.5);
    const double ic = rsqrt_refined(cc);
    *c = apq != 0.0 ? cc * ic : 1.0;
    *s = apq != 0.0 ? (x >= 0.0 ? 0.5 : -0.5) * y * ir * ic : 0.0;
}

// tan(a / 2) = s / (1 + c) of such a rotation (0 <= c <= 1).
__device__ __forceinline__ double half_tangent(double c, double s) {
    const double w = 1.0 + c;
    const double y = __builtin_amdgcn_rcp(w);
    const double e = fma(-w, y, 1.0);
    return s * fma(y, fma(e, e, e), y);
}

// (p, q) <- (c p - s q, s p + c q) with t = s / (1 + c), as corrections that
// are added: p - s (q + t p), q + s (p - t q).  A product with a c just below 1
// (1 - k u for a small angle) rounds the same way for all nearly equal values,
// rotation after rotation: diagonals of four clusters of 256 at n = 1024
// drifted by up to 7300 u with such products and by up to 680 u so, their
// residuals are 3.8e-15 |A|_F instead of 1.0e-14.  Also four operations instead
// of six (a truncation at n = 2048: 33.1 -> 32.3 ms).
__device__ __forceinline__ void rotate(double s, double t, double &p, double &q) {
    const double a = fma(t, p, q), b = fma(-t, q, p);
    p = fma(-s, a, p);
    q = fma(s, b, q);
}

}  // namespace oz
