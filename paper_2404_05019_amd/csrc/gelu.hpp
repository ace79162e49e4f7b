// erf-form GELU of the bf16 epilogues.  No device header is needed, so that its error can be
// measured on the host.
#pragma once

#include <math.h>

#if defined(__HIPCC__)
#define SCMOE_GELU_FN __host__ __device__ __forceinline__
#else
#define SCMOE_GELU_FN static inline
#endif

namespace scmoe {

SCMOE_GELU_FN float clamp01(float v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_fmed3f(v, 0.0f, 1.0f);         // (an output modifier of the instruction before it)
#else
  return fminf(fmaxf(v, 0.0f), 1.0f);
#endif
}

// v * Phi(v) with Phi(v) ~ 0.5 + v * Q(v^2), clamped to [0, 1].  Q: degree-8 minimax fit of
// (Phi(v) - 0.5) / v on |v| <= 3 sqrt 2 whose error is spread evenly over Phi, so that the error of
// GELU falls with |v|; its leading coefficient is positive, so beyond the interval the clamp
// saturates it the right way.  11 VALU operations (the clamp is free), no transcendental; +-inf and
// NaN come out as in v * Phi(v).  A first GEMM's epilogue is bound by these operations.
//   largest error   |v| < 0.1: 3.8e-7, < 0.5: 3.3e-6, < 1: 8.4e-6, < 2: 1.4e-5, < 4: 2.9e-5 (4.0e-5
//                   at 3.5 .. 4), all v: 4.7e-5 (at 4.24; the saturation at 4.3: 3.7e-5)
//   relative RMS    for v ~ N(0, s): s = 0.1: 1.1e-5, 0.25: 1.3e-5, 0.5: 1.0e-5, 1: 9.0e-6, 2: 7.9e-6,
//                   4: 4.4e-6; the bf16 rounding of the stored value is 1.7e-3
// A fit for the smallest error at any v (3.4e-5) has two to five times these relative errors where
// hidden values lie (s = 0.25: 7.0e-5, 1: 2.2e-5).
SCMOE_GELU_FN float gelu_erf_fast(float v) {
  const float u = v * v;
  float p = 5.6267362297246496e-11f;
  p = fmaf(p, u, -5.371846523161139e-09f);
  p = fmaf(p, u, 2.2682897338199837e-07f);
  p = fmaf(p, u, -5.646204954246059e-06f);
  p = fmaf(p, u, 9.35905336518772e-05f);
  p = fmaf(p, u, -0.0011093998327851295f);
  p = fmaf(p, u, 0.009818118065595627f);
  p = fmaf(p, u, -0.0663469210267067f);
  p = fmaf(p, u, 0.39890313148498535f);
  return v * clamp01(fmaf(p, v, 0.5f));
}

}  // namespace scmoe
