// Exact two-level propagator shared by the emitter kernels.
#pragma once

#include "mlk_internal.h"

namespace mlk {

// 1 / sqrt(x) for a positive x: the hardware's estimate and one third-order
// correction, y (1 + e/2 + 3 e^2/8) with e = 1 - x y^2 (the binomial series of
// (1 - e)^{-1/2}; the estimate's e is below 2^-20, so the dropped e^3 term is below
// FP64 rounding).  About a fifth of the instructions of 1.0 / sqrt(x).
__device__ __forceinline__ double rsqrt_refined(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-x * y, y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// Exact two-level step for one emitter; returns the new state and mu_dot.  The
// rotation by th = 2 om dt takes one sine and cosine, of th/2: sin th = 2 sin cos,
// 1 - cos th = 2 sin^2 without cancellation.
__device__ __forceinline__ void tls_advance(double w0, const double d[3], const double et[3],
                                            double dt, double st[3], double md[3]) {
  const double gg = et[0] * d[0] + et[1] * d[1] + et[2] * d[2];
  const double hx = -gg, hz = -0.5 * w0;
  const double om2 = hx * hx + hz * hz;
  const double p = st[0];
  const double rx = 2.0 * st[1], ry = -2.0 * st[2];
  double rx2 = rx, ry2 = ry, p2 = p;
  if (om2 > 0.0) {
    const double io = rsqrt_refined(om2);
    const double kx = hx * io, kz = hz * io;
    double sh, ch;
    sincos(om2 * io * dt, &sh, &ch);
    const double s = 2.0 * sh * ch, omc = 2.0 * sh * sh, c = 1.0 - omc;
    const double rz = 1.0 - 2.0 * p;
    const double kr = kx * rx + kz * rz;
    rx2 = rx * c - kz * ry * s + kx * kr * omc;
    ry2 = ry * c + (kz * rx - kx * rz) * s;
    // rho11' = (1 - rz')/2 written so that no O(1) terms cancel
    p2 = 0.5 * (omc * (kx * kx - kx * kz * rx + 2.0 * kz * kz * p) + 2.0 * p * c - kx * ry * s);
  }
  st[0] = p2;
  st[1] = 0.5 * rx2;
  st[2] = -0.5 * ry2;
  const double f = w0 * ry2;  // -2 w0 Im(rho01)
  md[0] = f * d[0];
  md[1] = f * d[1];
  md[2] = f * d[2];
}

}  // namespace mlk
