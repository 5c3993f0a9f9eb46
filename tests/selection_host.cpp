// Host check of the kernels' shortcuts of the TENO-D selection that no C ABI call
// reaches: wherever teno_smooth reports the large stencil as certain, the exact
// weights keep it (EQ: or the five values are equal).  Prints the violations
// and how often the shortcut applied.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <limits>
#include <random>

#include "tgks_device.hpp"

using namespace tgks;

static long long applied = 0, wrong = 0;

static void check(const double* Q, const TenoCfg& c) {
  TenoParts<double> p;
  teno_parts(Q, p);
  const bool eq = Q[0] == Q[1] && Q[1] == Q[2] && Q[2] == Q[3] && Q[3] == Q[4];
  const bool s0 = teno_smooth<false>(p), s1 = teno_smooth<true>(p);
  if (!s0 && !s1) return;
  ++applied;
  const bool large = teno_exact(Q, c) == 1u;
  if ((s0 && !large) || (s1 && !large && !eq)) {
    if (++wrong <= 5) printf("violation: %g %g %g %g %g\n", Q[0], Q[1], Q[2], Q[3], Q[4]);
  }
}

int main() {
  const double inf = std::numeric_limits<double>::infinity(), nan = std::numeric_limits<double>::quiet_NaN();
  const TenoCfg cfg[2] = {teno_cfg(1e-7, 1e-5, 1e-40, 7), teno_cfg(2e-5, 1e-6, 1e-12, 7)};
  std::mt19937_64 g(3);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  std::normal_distribution<double> z;
  for (const TenoCfg& c : cfg) {
    if (!(c.fast & TENO_RATIO_OK)) return 2;
    // a jump, a constant and a ramp at every magnitude, also beside zeros
    for (int e = -320; e <= 308; ++e) {
      const double x = std::pow(10.0, e);
      for (int k = 0; k < 5; ++k) {
        double Q[5], R[5], S[5], T[5];
        for (int i = 0; i < 5; ++i) {
          Q[i] = i >= k ? x : 0.0;
          R[i] = i == k ? x : 0.0;
          S[i] = x * (1.0 + 0.1 * i);
          T[i] = i == k ? (e & 1 ? inf : nan) : x;
        }
        check(Q, c);
        check(R, c);
        check(S, c);
        check(T, c);
      }
    }
    for (long long n = 0; n < 400000; ++n) {
      double Q[5];
      const double mag = std::pow(10.0, 620.0 * u(g) - 312.0), rel = std::pow(10.0, -18.0 * u(g)), s = u(g), ph = 6.3 * u(g);
      const double rough = std::pow(10.0, -6.0 * u(g)), base = n & 1 ? 1.0 : 0.0;
      for (int i = 0; i < 5; ++i) Q[i] = mag * (base + rel * (std::sin(ph + s * i) + rough * z(g)));
      check(Q, c);
    }
  }
  printf("applied %lld wrong %lld\n", applied, wrong);
  return wrong != 0;
}
