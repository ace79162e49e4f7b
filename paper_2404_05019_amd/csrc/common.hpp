// Internal helpers shared by the HIP sources of libscmoe (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "scmoe.h"

namespace scmoe {

// Last HIP error seen by an entry point on this thread (reported by scmoe_last_hip_error).
extern thread_local int g_last_hip_error;

inline int hip_fail(hipError_t e) {
  g_last_hip_error = static_cast<int>(e);
  return SCMOE_ERR_HIP;
}

// Status of the kernel launch that was just enqueued.
inline int launch_status() {
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? SCMOE_OK : hip_fail(e);
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline int elem_bytes(int dtype) { return dtype == SCMOE_BF16 ? 2 : 4; }

// Elements per 16-byte vector.
inline int vec_elems(int dtype) { return dtype == SCMOE_BF16 ? 8 : 4; }

inline bool dtype_ok(int dtype) { return dtype == SCMOE_F32 || dtype == SCMOE_BF16; }

// A matrix view is acceptable when its base is 16-byte aligned and its row stride keeps
// every row 16-byte aligned and covers `cols`.
inline bool view_ok(const void* p, int64_t ld, int64_t cols, int dtype) {
  return aligned16(p) && ld >= cols && (ld % vec_elems(dtype)) == 0;
}

// ---- bf16 <-> fp32 on the device (bit manipulation; round to nearest even) -------------
__device__ __forceinline__ float bf16_to_f32(uint16_t v) {
  return __uint_as_float(static_cast<uint32_t>(v) << 16);
}

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) {  // inf / nan: keep the class, quiet a nan
    return static_cast<uint16_t>((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  }
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return static_cast<uint32_t>(f32_to_bf16(lo)) | (static_cast<uint32_t>(f32_to_bf16(hi)) << 16);
}

// GELU of the expert MLPs: exact erf form or the tanh approximation.
__device__ __forceinline__ float gelu_f32(float v, int mode) {
  if (mode == SCMOE_GELU_TANH) {
    const float c = 0.7978845608028654f;
    return 0.5f * v * (1.0f + tanhf(c * (v + 0.044715f * v * v * v)));
  }
  return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
}

// Small chores that a layer call would otherwise launch kernels of their own for; the input encode
// (one workgroup of its launch, or the gate workgroup that encodes) does them on the side: pair[0..1] = {0, pair_hi} (the segment
// bounds of the shared expert) and nzero zeros at each of zero_a, zero_b.  All optional.
struct ScanChores {
  int32_t* pair = nullptr;
  int pair_hi = 0;
  int* zero_a = nullptr;
  int* zero_b = nullptr;
  int nzero = 0;
  // For the joint second GEMM (one-launch dispatch, k = 1; token_of == nullptr: off): all tokens in
  // the packed order, those without a row behind the others in ascending order; the gate weight
  // of every packed row; and offsets with T as one more entry.
  int32_t* token_of = nullptr;
  float* row_gate = nullptr;
  const float* gate_w = nullptr;
  int32_t* joint_offsets = nullptr;
};

// What the input encode of a layer call writes (its inputs are the gate's choices).
struct DispatchOut {
  int32_t* counts = nullptr;
  int32_t* offsets = nullptr;
  int32_t* dst_row = nullptr;
  int32_t* src_token = nullptr;
  int capacity = 0;
  ScanChores ch;
};

// The gate of a layer call, its input encode and its coefficient gate, as work that the launch of the shared expert's
// first GEMM does on the side (they do not depend on each other).
struct GateWork {
  const void* x; int64_t ldx;      // gate input [T, d]
  const float* Wg; const float* bias;
  int T, d, E, k, normalize;
  int32_t* idx; float* gw;
  DispatchOut enc;
  unsigned long long* marks;       // 8 bytes of scratch for every 64 tokens, whatever they hold (all_arrived)
  unsigned long long call;         // another number for every call, not zero (call_number)
  int workgroups;                  // set by the launch: of the gate, and of the coefficient gate
  int coef_workgroups;
  const void* xc; int64_t ldxc; const float* Wcg; int cg_mode; float* coef;   // (cg_mode SCMOE_CG_NONE: none)
};

// ---- entry points implemented in one source and used by the layer orchestration --------
enum { FFN_AUTO = 0, FFN_TILED = 1, FFN_DIRECT = 2 };
// One expert-FFN call over packed segments.  All strides in elements.
struct FfnArgs {
  const void* x; int64_t ldx;      // [rows, d] activations
  const int32_t* gather;           // row r reads x[gather[r]] (the dispatch permutation applied
                                   // on load); nullptr = identity
  int64_t x_rows;                  // with gather: rows of x that gather may name
  const int32_t* offsets;          // [E + 1] segment starts, device (direct kernel: nullptr = one segment of max_rows rows)
  int max_rows, E, d, F;
  int path;                        // FFN_AUTO: by ffn_is_tiled; else the caller has decided
  bool beside;                     // another chain runs beside this one on a second stream
  bool slots;                      // segments are pool slots: which expert has which depends on the other rows
  const void* W1; int64_t ldw1; const float* b1;   // [E, F, d]
  const void* W2; int64_t ldw2; const float* b2;   // [E, d, F]
  void* hidden; int64_t ldh;       // [rows, F] scratch
  void* y; int64_t ldy;            // [rows, d]
  int gelu_mode;
  // Fused output decode of the second GEMM (all three pointers nullptr: off).
  // With scatter (addend optional):
  //   y[scatter[r], :] = addend[scatter[r], :] + row_scale[scatter[r]] * (W2 . hidden[r] + b2)
  // Without scatter (rows stay in place), row_scale holding PAIRS of coefficients per row of
  // which the first is used, either pointer optional:
  //   y[r, :] = addend[r, :] + row_scale[2 r] * (W2 . hidden[r] + b2)
  const int32_t* scatter; const float* row_scale; const void* addend; int64_t ldadd;
  // In the routed call of ffn_forward_pair: both second GEMMs as one product (GemmArgs::A2), over the
  // E + 1 segments of joint_offsets; scatter: the tokens in packed order, which is also the gather
  // array of the shared call; row_scale: per packed row.
  const int32_t* joint_offsets;
  // In the shared call of ffn_forward_pair: the first GEMM's launch does this on the side, ahead of everything else of
  // the pair (nullptr: done already).
  const GateWork* gate;
  // Scratch of the tiled path (split-K of the last round of tiles); may be nullptr: no split.
  void* scratch; size_t scratch_bytes;
  bool scratch_zeroed;             // the arrival counters at the start of scratch are zero already
  // Event the stream waits for between the first and the second GEMM (nullptr: none).
  hipEvent_t before_second;
};

// The tiled bf16 kernel runs a call of this many packed rows over E segments (else: the direct
// one).  mean_rows, all_rows: rows per chain and of all chains of the whole call (a layer has two).
bool ffn_is_tiled(int dtype, int d, int F, int max_rows, int E, int64_t mean_rows, int64_t all_rows);
// One expert-FFN call, whichever kernel it takes.
int ffn_forward(const FfnArgs& a, int dtype, hipStream_t stream);
// The shared expert `se` (one dense segment) and the routed experts `rt`.  Both tiled: their
// first GEMMs share a launch; the second GEMMs are one product with rt.joint_offsets, else one
// launch if neither decodes, else two: the shared expert's first (the routed one may decode into
// its rows).  Both direct: first GEMMs in one launch, second GEMMs in one launch (no decode into
// the other's rows).
int ffn_forward_pair(const FfnArgs& se, const FfnArgs& rt, int dtype, hipStream_t stream);

// Row stride the grouped GEMM likes for an operand of `width` columns: rows at a multiple
// of 512 bytes get 128 bytes of padding.
inline int64_t padded_ld(int64_t width, int dtype) {
  const int64_t eb = elem_bytes(dtype);
  return ((width * eb) % 512 == 0) ? width + 128 / eb : width;
}
bool ffn_mfma_supported(int d, int F);
bool ffn_joint_second_fits(int T, int rows, int d, int F, int E, int64_t ldh, int64_t ldw2);   // sizes that the joint second GEMM takes
bool ffn_second_in_one_launch(int T, int rows, int d, int F, int E);   // top-1 layer: both second GEMMs as one launch and the combine kernel
bool ffn_gate_on_the_side(const GateWork& g, int rows, int F, int64_t ldw1);   // a call whose gate may be FfnArgs::gate
size_t ffn_mfma_scratch_bytes();   // scratch the tiled path can use (16-byte aligned)
int ffn_mfma_counter_ints();       // ints at the start of that scratch that must be zero before a call

// Compute units of the current device (256 on MI355X), cached per device.
inline int num_cus() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

}  // namespace scmoe
