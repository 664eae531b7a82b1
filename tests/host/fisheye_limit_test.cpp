// The fisheye limit against the plain scan of all 4096 angles, bit for bit:
// lenses without a limit, with one anywhere in (0, pi/2], at the ends of the
// range, and with coefficients so large that the derivative overflows.
#include <cstdio>
#include <random>

#include "fisheye_limit.h"

static double deriv(const double* k, double th) {
  const double t2 = th * th;
  return std::fma(t2, std::fma(t2, std::fma(t2, std::fma(t2, 9.0 * k[3], 7.0 * k[2]), 5.0 * k[1]), 3.0 * k[0]), 1.0);
}

static double plain(const double* k) {
  const double half_pi = 1.5707963267948966;
  double prev = 0.0;
  for (int i = 1; i <= 4096; i++) {
    const double th = half_pi * i / 4096;
    if (deriv(k, th) <= 0.0) {
      double lo = prev, hi = th;
      for (int it = 0; it < 200; it++) {
        const double mid = 0.5 * (lo + hi);
        if (deriv(k, mid) > 0.0) lo = mid; else hi = mid;
      }
      return lo;
    }
    prev = th;
  }
  return half_pi;
}

int main() {
  std::mt19937_64 r(5);
  std::normal_distribution<double> g;
  long limited = 0, bad = 0, n = 0;
  auto check = [&](const double* k) {
    const double a = plain(k), b = gut::fisheye_limit(k, deriv);
    limited += a < 1.57;
    n++;
    if (a != b && bad++ < 5) printf("%g %g %g %g: %.17g, not %.17g\n", k[0], k[1], k[2], k[3], b, a);
  };
  for (double scale : {0.01, 0.05, 0.2, 1.0, 1e4, 1e150, 1e308})
    for (int t = 0; t < 1500; t++) {
      double k[4];
      for (double& x : k) {
        x = r() % 4 == 0 ? 0.0 : scale * g(r);
        if (!std::isfinite(x)) x = 1e308;
      }
      check(k);
    }
  for (double th : {1e-9, 3e-4, 3.8e-4, 0.7, 1.5704, 1.5707963267948966, 1.5708}) {  // 1 + 3 k1 th^2 = 0
    const double k[4] = {-1.0 / (3.0 * th * th), 0.0, 0.0, 0.0};
    check(k);
  }
  printf("%ld lenses, %ld limited, %ld differ\n", n, limited, bad);
  if (bad == 0 && limited > 1000 && n - limited > 1000) printf("ALL OK\n");
  return bad != 0;
}
