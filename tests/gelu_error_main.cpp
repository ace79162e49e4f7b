// Error of the bf16 epilogues' GELU against long double: lines "max LO HI error" (largest absolute
// error at LO <= |v| < HI) and "rms S error" (relative root mean square for v ~ N(0, S)).
#include <stdio.h>

#include "gelu.hpp"

static long double exact(float v) { return 0.5L * v * erfcl(-(long double)v / sqrtl(2.0L)); }

int main() {
  const double edges[] = {0, 0.1, 0.25, 0.5, 1, 1.5, 2, 2.5, 3, 3.5, 4, 4.2, 12};
  const int n = sizeof edges / sizeof *edges - 1;
  const double sigmas[] = {0.1, 0.25, 0.5, 1, 1.5, 2, 4};
  double worst[n] = {}, err[7] = {}, ref[7] = {};
  for (int i = -600000; i <= 600000; ++i) {
    const float v = (float)(i * 2e-5);
    const long double g = exact(v), d = scmoe::gelu_erf_fast(v) - g;
    for (int q = 0; q < n; ++q)
      if (fabs(v) >= edges[q] && fabs(v) < edges[q + 1] && fabsl(d) > worst[q]) worst[q] = (double)fabsl(d);
    for (int q = 0; q < 7; ++q) {
      const double w = exp(-0.5 * v * v / (sigmas[q] * sigmas[q]));
      err[q] += w * (double)(d * d);
      ref[q] += w * (double)(g * g);
    }
  }
  for (int q = 0; q < n; ++q) printf("max %g %g %.4e\n", edges[q], edges[q + 1], worst[q]);
  for (int q = 0; q < 7; ++q) printf("rms %g %.4e\n", sigmas[q], sqrt(err[q] / ref[q]));
  const float inf = INFINITY;
  printf("special %d %d %d\n", scmoe::gelu_erf_fast(inf) == inf, scmoe::gelu_erf_fast(-inf) != scmoe::gelu_erf_fast(-inf),
         scmoe::gelu_erf_fast(NAN) != scmoe::gelu_erf_fast(NAN));
  return 0;
}
