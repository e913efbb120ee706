// The plane rotation of the Jacobi eigensolvers.
#pragma once

#include <hip/hip_runtime.h>

namespace oz {

// Rotation that zeroes a_pq of [[app, apq], [apq, aqq]]: tan of the smaller
// angle, t = y sgn(x) / (|x| + sqrt(x^2 + y^2)) with x = aqq - app, y = 2 apq
// (scaled by a power of two so the squares stay in range), c = 1 / sqrt(1 +
// t^2), s = t c.  Reciprocal (square root) estimates of the hardware (about
// 2^-23) with one third-order correction each: a third of the dependent
// instructions of the exact divisions and square roots; c^2 + s^2 = 1 to two
// rounding errors.
__device__ __forceinline__ double rsqrt_refined(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}
__device__ __forceinline__ double rcp_refined(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}
__device__ __forceinline__ void schur_rotation(double app, double aqq, double apq, double *c, double *s) {
    double x = aqq - app, y = 2.0 * apq;
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(x), fabs(y)));
    x = ldexp(x, ex);
    y = ldexp(y, ex);
    const double r2 = fma(x, x, y * y);
    const double t = (x >= 0.0 ? y : -y) * rcp_refined(fabs(x) + r2 * rsqrt_refined(r2));
    const double cc = rsqrt_refined(fma(t, t, 1.0));
    *c = apq != 0.0 ? cc : 1.0;
    *s = apq != 0.0 ? t * cc : 0.0;
}

}  // namespace oz
