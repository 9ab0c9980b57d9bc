// Extreme eigenpairs of random symmetric tridiagonal matrices by the
// library's bisection and inverse iteration against its Jacobi rotations.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>

#include "common.h"

int main() {
  std::mt19937 g(3);
  std::normal_distribution<double> N;
  for (int n : {1, 2, 3, 8, 40, 61, 150})
    for (int kind = 0; kind < 3; ++kind) {
      std::vector<double> a(n), b(n), T((size_t)n * n), vals, vecs;
      for (int i = 0; i < n; ++i) {
        a[i] = kind == 2 ? 0.0 : 14 + 5 * N(g);
        b[i] = kind == 1 ? 1e-9 * std::fabs(N(g)) : std::fabs(7 + N(g));
      }
      for (int i = 0; i < n; ++i) {
        T[(size_t)i * n + i] = a[i];
        if (i + 1 < n) T[(size_t)i * n + i + 1] = T[(size_t)(i + 1) * n + i] = b[i];
      }
      sgw::jacobi_eigen(n, T, vals, vecs);
      double lo, hi, y0, y1;
      sgw::tridiagonal_extremes(a, b, lo, hi, y0, y1);
      const double w = 1e-13 * n * (1 + std::fabs(vals[0]) + std::fabs(vals[n - 1]));
      const double *last = &vecs[(size_t)(n - 1) * n];
      // residual norms b |y_last|, the quantity the interval is widened by
      const bool ok = std::fabs(lo - vals[0]) < w && std::fabs(hi - vals[n - 1]) < w &&
                      b[n - 1] * std::fabs(std::fabs(y0) - std::fabs(last[0])) < 1e-9 &&
                      b[n - 1] * std::fabs(std::fabs(y1) - std::fabs(last[n - 1])) < 1e-9;
      if (!ok) {
        std::printf("n %d kind %d: %g %g %g %g against %g %g %g %g\n", n, kind, lo, hi, y0, y1,
                    vals[0], vals[n - 1], last[0], last[n - 1]);
        return 1;
      }
    }
  std::puts("ALL OK");
  return 0;
}
