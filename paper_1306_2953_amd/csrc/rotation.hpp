// FP64 Jacobi rotations for the device: the symmetric eigensolver's and those
// of the small per-state problems.
#pragma once

#include <hip/hip_runtime.h>

namespace rs {
namespace {

// sqrt(x) and 1 / sqrt(x) for normal x: the hardware's estimate and two
// Goldschmidt steps.
__device__ __forceinline__ void sqrt_rsqrt(double x, double &root, double &inv) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double r = fma(-h, g, 0.5);
        g = fma(g, r, g);
        h = fma(h, r, h);
    }
    root = g;
    inv = 2.0 * h;
}

// Rotation that annihilates apq: columns p' = c p - s q, q' = s p + c q.
// tan = o / (|d| + sqrt(d^2 + o^2)), d = aqq - app, o = 2 apq, c = 1 /
// sqrt(1 + tan^2), s = c tan, with the roots and the reciprocal refined from
// the hardware's estimates: a shorter serial chain than three full divisions
// and two square roots.  d and o are scaled by a power of two first, so that
// no square over- or underflows.
__device__ __forceinline__ double2 jacobi_rotation(double app, double apq, double aqq) {
    double d = aqq - app, o = 2.0 * apq;
    if (apq == 0.0) return make_double2(1.0, 0.0);
    const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(d), fabs(o)));
    d = ldexp(d, e);
    o = ldexp(o, e);
    double root, c;
    sqrt_rsqrt(fma(d, d, o * o), root, c);
    const double den = fabs(d) + root;
    double r = __builtin_amdgcn_rcp(den);
    r = fma(fma(-den, r, 1.0), r, r);
    r = fma(fma(-den, r, 1.0), r, r);
    double t = o * r;
    t = fma(fma(-den, t, o), r, t);
    sqrt_rsqrt(fma(t, t, 1.0), root, c);
    return make_double2(c, (d >= 0.0 ? t : -t) * c);
}

}  // namespace
}  // namespace rs
