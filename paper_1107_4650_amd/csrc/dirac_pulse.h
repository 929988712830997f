// dirac_pulse.h -- the laser pulse of dl_step_pulse and its integral over a
// step (host code).  Internal to libdirac.
#pragma once
#include <cmath>
#include <cstdint>

namespace dirac {

// A time-dependent vector potential A(t, x) = f(t) P(x): a laser pulse with a
// linear turn-on ramp, the kind of field whose integral Sec. 2.3 notes can be
// found analytically.  f(t) = w(t) sin(omega t + phase) with the trapezoid
// envelope w: 0 before t = 0, t / t_on on [0, t_on), 1 for t_flat, a linear
// fall to 0 over t_off, 0 afterwards.  The local step of step n carries the
// field integral At^n(x) = P(x) F_n, F_n = int f over [t0 + n dt,
// t0 + (n + 1) dt] (eq:field_dis1), evaluated here in closed form per step,
// on the host: a pass takes the few values of its steps as arguments, where
// every wave of the kernels would spend some 400 FP64 operations on each.
struct PulseK {
  double omega, phase;           // carrier
  double t_on, t_flat, t_off;    // envelope
  double t0, dt;                 // step n starts at t0 + n dt
  int64_t n0;                    // first step of the pass
};

// sin(u) / u
inline double sinc_d(double u) {
  const double u2 = u * u;
  if (std::fabs(u) < 1e-3) return 1.0 - u2 * (1.0 / 6.0 - u2 * (1.0 / 120.0));
  return std::sin(u) / u;
}

// (sin u - u cos u) / u^2: a series below |u| = 1/4 (terms to u^11, the next
// below 2e-19 relative), the direct form above (cancellation costs at most
// 3 eps / u^2 < 5e-15 relative there)
inline double j1_d(double u) {
  if (std::fabs(u) < 0.25) {
    const double u2 = u * u;
    double p = -1.0 / 518918400.0;          // -12 / 13!
    p = std::fma(p, u2, 1.0 / 3991680.0);        //  10 / 11!
    p = std::fma(p, u2, -1.0 / 45360.0);         //  -8 / 9!
    p = std::fma(p, u2, 1.0 / 840.0);            //   6 / 7!
    p = std::fma(p, u2, -1.0 / 30.0);            //  -4 / 5!
    p = std::fma(p, u2, 1.0 / 3.0);              //   2 / 3!
    return u * p;
  }
  const double s = std::sin(u), c = std::cos(u);
  return (s - u * c) / (u * u);
}

// int_a^b (w_m + beta (t - m)) sin(omega t + phase) dt with m = (a + b) / 2,
// h = (b - a) / 2, psi = omega m + phase:
//   int sin(omega t + phase)        = 2 h sin(psi) sinc(omega h)
//   int (t - m) sin(omega t + phase) = 2 h^2 cos(psi) j1(omega h)
// (the product forms avoid the cancellation of a difference of cosines)
inline double lin_sin_integral(double a, double b, double w_m, double beta,
                                                   double omega, double phase) {
  const double h = 0.5 * (b - a), m = 0.5 * (a + b);
  const double u = omega * h;
  const double arg = std::fma(omega, m, phase);
  const double sp = std::sin(arg), cp = std::cos(arg);
  const double i0 = 2.0 * h * sp * sinc_d(u);
  const double i1 = 2.0 * h * h * cp * j1_d(u);
  return std::fma(w_m, i0, beta * i1);
}

// F = int_ta^tb f(t) dt, over the pieces of [ta, tb] on which w is linear
inline double pulse_integral(const PulseK& p, double ta, double tb) {
  const double t1 = p.t_on + p.t_flat, t2 = t1 + p.t_off;
  double sum = 0.0;
  if (p.t_on > 0.0) {  // rise: w = t / t_on
    const double a = std::fmax(ta, 0.0), b = std::fmin(tb, p.t_on);
    if (a < b) sum += lin_sin_integral(a, b, 0.5 * (a + b) / p.t_on, 1.0 / p.t_on, p.omega, p.phase);
  }
  {  // flat top: w = 1
    const double a = std::fmax(ta, p.t_on), b = std::fmin(tb, t1);
    if (a < b) sum += lin_sin_integral(a, b, 1.0, 0.0, p.omega, p.phase);
  }
  if (p.t_off > 0.0) {  // fall: w = (t2 - t) / t_off
    const double a = std::fmax(ta, t1), b = std::fmin(tb, t2);
    if (a < b)
      sum += lin_sin_integral(a, b, (t2 - 0.5 * (a + b)) / p.t_off, -1.0 / p.t_off, p.omega,
                              p.phase);
  }
  return sum;
}

// F of step n0 + s of the pass (the time of a step is formed from its global
// index, so a pass of K steps and K passes of one step see the same values)
inline double pulse_step_integral(const PulseK& p, int64_t s) {
  const double n = static_cast<double>(p.n0 + s);
  return pulse_integral(p, std::fma(n, p.dt, p.t0), std::fma(n + 1.0, p.dt, p.t0));
}

}  // namespace dirac
