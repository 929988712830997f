// dirac_cos_sinc.h -- cos(A) and sin(A)/A from A^2 for the FP32 state's vector potential
// (host and device code).  Internal to libdirac.
#pragma once

namespace dirac {

// cos(A) and sin(A)/A as functions of z = A^2 <= kCosSincMax (A <= 12.5), for
// the FP32 state: Taylor series at x = A/16 <= pi/4 (to r^15 and r^16,
// truncation below 1e-16), then the angle doubled four times:
// sinc 2x = sinc x cos x and cos 2x = 1 - 2 sin^2 x.  No square root, division
// or quadrant: 31 FP64 operations in one block against 82 with them, with
// errors below 7e-15 (cos A: 6.3e-15 at A = 9.17, sin A: 3.6e-15; the general
// form with sincos_fast<1>: 2.1e-14).
constexpr double kCosSincMax = 156.8;  // (A/16)^2 below (pi/4)^2

__host__ __device__ __forceinline__ void cos_sinc(double z, double* c_out, double* s_out) {
  double w = 0.00390625 * z;               // x^2
  double s = -1.0 / 1307674368000.0;       // 1/15!
  s = fma(s, w, 1.0 / 6227020800.0);       // 1/13!
  s = fma(s, w, -1.0 / 39916800.0);        // 1/11!
  s = fma(s, w, 1.0 / 362880.0);           // 1/9!
  s = fma(s, w, -1.0 / 5040.0);            // 1/7!
  s = fma(s, w, 1.0 / 120.0);              // 1/5!
  s = fma(s, w, -1.0 / 6.0);               // 1/3!
  s = fma(s, w, 1.0);
  double c = 1.0 / 20922789888000.0;       // 1/16!
  c = fma(c, w, -1.0 / 87178291200.0);     // 1/14!
  c = fma(c, w, 1.0 / 479001600.0);        // 1/12!
  c = fma(c, w, -1.0 / 3628800.0);         // 1/10!
  c = fma(c, w, 1.0 / 40320.0);            // 1/8!
  c = fma(c, w, -1.0 / 720.0);             // 1/6!
  c = fma(c, w, 1.0 / 24.0);               // 1/4!
  c = fma(c, w, -0.5);                     // 1/2!
  c = fma(c, w, 1.0);
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const double q = s * s * w;            // sin^2 of the current angle
    s = s * c;
    c = fma(-2.0, q, 1.0);
    w = 4.0 * w;
  }
  *s_out = s;
  *c_out = c;
}

}  // namespace dirac
