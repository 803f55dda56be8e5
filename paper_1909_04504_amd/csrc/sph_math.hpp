// FP64 reciprocal, square root and reciprocal square root from an
// approximation of about 26 bits (v_rcp_f64, v_rsq_f64 on the device).
//
// The reciprocal and the reciprocal square root take one correction of third order
// (with e = 1 - x y the reciprocal is y (1 + e + e^2 + ..), with e = 1 - x y^2
// the reciprocal square root y (1 + e/2 + 3 e^2/8 + ..)), the square root
// two steps of Newton's iteration with an exact residual: 4, 6 and 8
// instructions where the correctly rounded division and square root take
// about 12 and 18, and at most one unit in the last place from the exact
// value (over 2^-60 .. 2^20, from approximations off by up to 2^-24: 0.50, 1.00
// and 0.50 units; 1 / sqrt(x) rounded twice 1.49).
#pragma once

#include <math.h>

namespace sph {

__host__ __device__ __forceinline__ double rcp_from(double x, double y) {
    const double e = fma(-x, y, 1.0);
    return fma(fma(e, e, e), y, y);
}
__host__ __device__ __forceinline__ double rsqrt_from(double x, double y) {
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}
// y: of the reciprocal square root
__host__ __device__ __forceinline__ double sqrt_from(double x, double y) {
    double g = x * y, h = 0.5 * y;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    return fma(fma(-g, g, x), h, g);
}

}  // namespace sph
