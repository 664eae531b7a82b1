// The validity limit of a fisheye lens (host code without HIP).
#pragma once
#include <cmath>

namespace gut {

// Whether d theta_d/d theta is positive on all of [a, b], 0 <= a <= b, by more
// than it is rounded: each term at the end where it is least.
inline bool thetad_rises(const double* k, double a, double b) {
  const double a2 = a * a, b2 = b * b;
  double lo = 1.0, sum = 1.0, mag = 0.0, ap = 1.0, bp = 1.0;
  for (int j = 0; j < 4; j++) {
    ap *= a2; bp *= b2;
    const double c = (2 * j + 3) * k[j];
    lo += c > 0.0 ? c * ap : c * bp;
    sum += std::fabs(c) * bp;
    mag += std::fabs(c);
  }
  return lo > 1e-12 * sum && mag < 1e300;  // (deriv itself could overflow)
}

// Fisheye validity limit: first angle in (0, pi/2] where d theta_d/d theta
// reaches zero (scan, then bisection), else pi/2.  deriv(k, theta) evaluates
// 1 + 3 k1 theta^2 + 5 k2 theta^4 + 7 k3 theta^6 + 9 k4 theta^8.  The scan passes over spans
// on which the derivative's bound is positive, the whole range for most
// lenses: 4096 evaluations took 41 us a camera and call, more than the rest of
// a call's host work.
template <class D>
double fisheye_limit(const double* k, D deriv) {
  const int steps = 4096, span = 64;
  const double half_pi = 1.5707963267948966;
  if (thetad_rises(k, 0.0, half_pi)) return half_pi;
  for (int i0 = 0; i0 < steps; i0 += span) {
    if (thetad_rises(k, half_pi * i0 / steps, half_pi * (i0 + span) / steps)) continue;
    for (int i = i0 + 1; i <= i0 + span; i++) {
      const double th = half_pi * i / steps;
      if (!(deriv(k, th) <= 0.0)) continue;
      double lo = half_pi * (i - 1) / steps, hi = th;
      for (int it = 0; it < 200; it++) {
        const double mid = 0.5 * (lo + hi);
        if (mid == lo || mid == hi) break;
        if (deriv(k, mid) > 0.0) lo = mid; else hi = mid;
      }
      return lo;
    }
  }
  return half_pi;
}

}  // namespace gut
