// The coefficient gates of ScMoE paper Eq. (14)-(17) as a piece of device code that a workgroup of any launch can run.
#pragma once
#include "common.hpp"

namespace scmoe {

template <bool BF16>
__device__ __forceinline__ void load8(const unsigned char* p, float* v) {
  // 16 bytes: 8 bf16 or 4 fp32 (then only v[0..3] are used)
  const uint4 q = *reinterpret_cast<const uint4*>(p);
  if (BF16) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  } else {
    v[0] = __uint_as_float(q.x);
    v[1] = __uint_as_float(q.y);
    v[2] = __uint_as_float(q.z);
    v[3] = __uint_as_float(q.w);
  }
}

// Coefficient gate: one wave per token at a time, fp32 dot products reduced across the wave.
// LDS_W: the gate's one or two weight rows are staged in LDS once per workgroup, which then
// walks over many tokens (read from global memory per token they cost two to four times
// the bytes of the token's row in cache traffic); otherwise they are read in place (rows too
// long for the LDS).
// Workgroup `block` of `blocks` that share the tokens.  cg_w: 4 d bytes of LDS, 8 d with mode SCMOE_CG_2.
// WAVES: of the workgroup (asked for at run time, its size is a dependent load from memory ahead of the first weights: 50 drawn
// calls took 3 % longer, 7208 tokens, d = 120 4.72 us against 4.45).
template <bool BF16, bool LDS_W, int WAVES>
__device__ __forceinline__ void coef_gate_rows(float* cg_w, int block, int blocks, const unsigned char* __restrict__ x,
                                               int64_t ldx_bytes, const float* __restrict__ Wcg, int mode, int T, int d,
                                               float* __restrict__ coef) {
  constexpr int NV = BF16 ? 8 : 4;
  if (LDS_W) {
    const int n = (mode == SCMOE_CG_2 ? 2 : 1) * d;
    for (int i = threadIdx.x; i < n; i += 64 * WAVES) cg_w[i] = Wcg[i];
    __syncthreads();
  }
  auto w = [&](int i) { return LDS_W ? cg_w[i] : Wcg[i]; };
  const int lane = threadIdx.x & 63;
  for (int t = block * WAVES + (threadIdx.x >> 6); t < T; t += blocks * WAVES) {
    const unsigned char* row = x + static_cast<int64_t>(t) * ldx_bytes;
    float a = 0.0f, b = 0.0f;
    for (int i0 = lane * NV; i0 < d; i0 += 64 * NV) {
      float v[8];
      load8<BF16>(row + static_cast<int64_t>(i0) * (BF16 ? 2 : 4), v);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        a = fmaf(v[i], w(i0 + i), a);
        if (mode == SCMOE_CG_2) b = fmaf(v[i], w(d + i0 + i), b);
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      a += __shfl_xor(a, off, 64);
      b += __shfl_xor(b, off, 64);
    }
    if (lane == 0) {
      float c0, c1;
      if (mode == SCMOE_CG_1) {
        c0 = 1.0f / (1.0f + expf(-a));
        c1 = 1.0f;
      } else {
        const float m = fmaxf(a, b);
        const float ea = expf(a - m), eb = expf(b - m);
        c0 = ea / (ea + eb);
        c1 = eb / (ea + eb);
      }
      coef[2 * static_cast<int64_t>(t)] = c0;
      coef[2 * static_cast<int64_t>(t) + 1] = c1;
    }
  }
}

}  // namespace scmoe
