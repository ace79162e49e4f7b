// Pieces shared by the bf16 MFMA grouped-GEMM kernels (expert computation, ScMoE paper
// Eq. (1)): vector types, the LDS swizzle, the argument block, the epilogue's GELU forms and
// the persistent tile schedule.
#pragma once
#include "common.hpp"
#include "gelu.hpp"
#include "tile_schedule.hpp"

#include <type_traits>

namespace scmoe {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

#define SCMOE_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
#define SCMOE_GLB_PTR(p) ((const __attribute__((address_space(1))) void*)(p))

// XOR swizzle of the 16-byte chunk index inside an LDS row.  A 64-lane ds_read_b128 is
// served in four passes of 16 lanes, and on gfx950 the passes are NOT runs of consecutive
// lanes (measured with a pairwise timing probe): {0-3, 12-15, 20-27}, {4-11, 16-19, 28-31}
// and the same two sets + 32.  A fragment read of the 16x16x32 MFMA has lane l on row l % 16
// and chunk l / 16, so one pass covers rows 0-3 and 12-15 with one chunk and rows 4-11 with
// the next; the 16 accesses must fall into 16 distinct 16-byte bank groups of the 256-byte
// bank window.  With 128-byte rows (two rows per window) chunk ^ (row/2 % 8) does that; with
// 64-byte rows (four per window) chunk ^ (-(row/4) % 4).  (Checked by enumeration.)
template <int CPR>
__host__ __device__ constexpr int swz(int r) {
  return CPR == 8 ? ((r >> 1) & 7) : ((0 - (r >> 2)) & 3);
}


struct GemmArgs {
  const unsigned char* A;   // activations, bf16 [rows, Kd]
  int64_t lda;              // row stride of A in elements
  const int32_t* gather;    // row r of the packed order reads A[gather[r]]; nullptr = identity
  const int32_t* offsets;   // [E + 1] segment starts, device
  const unsigned char* W;   // bf16 [E, N, Kd], row stride ldw
  int64_t ldw;              // row stride of W in elements (>= Kd)
  const float* bias;        // [E, N] or nullptr
  unsigned char* C;         // bf16 [rows, N], row stride ldc
  int64_t ldc;
  int E, N, Kd;
  int nt;                   // column tiles
  int gelu_mode;
  int rotk;                 // tiled: column tile c starts its walk over K at k-tile rotk * c (mod the k-tiles); 0: at the first.
                            // direct, fp32: what the segment index adds to the place of the first step
  bool beside;              // (host) another chain runs beside this launch on a second stream
  int stream_out;           // store C with the streaming (non-temporal) hint
  // Fused output decode (optional; scatter == nullptr stores C[r, :] as is).  Packed row r
  // is written to row t = scatter[r] of C as  addend[t, :] + row_scale[t] * (sum + bias).
  const int32_t* scatter;
  const float* row_scale;
  const unsigned char* addend;   // bf16 [*, N], row stride ldadd; may be C itself
  int64_t ldadd;
  // Split-K of the last, partly filled round of tiles (optional; splitk_part == nullptr: off).
  float* splitk_part;            // SPLITK_PARTS partial tiles of BM x BN floats
  int* splitk_count;             // SPLITK_PARTS arrival counters, zero between launches
  int* splitk_zero;              // first GEMM: SPLITK_PARTS counters to clear (nullptr: none)
  // Optional dense extra segment with operands of its own (xrows == 0: none): xC[r, :] =
  // act(xA[r, :] . xW^T + xbias) for r < xrows, same N and Kd.  Its tiles come first in the
  // tile order and it has the segment id E.  (The shared expert riding in the routed experts'
  // launch.)  Not combined with the output decode.
  int xrows;
  const unsigned char* xA;
  int64_t xlda;
  const unsigned char* xW;       // bf16 [N, Kd], row stride xldw
  int64_t xldw;
  const float* xbias;            // [N] or nullptr
  const int32_t* xgather;        // row r reads xA[xgather[r]]; nullptr = identity
  unsigned char* xC;
  int64_t xldc;
  // Joint second GEMM of a top-1 layer (optional; A2 == nullptr: off).  A row of the packed order is
  // a token, and a tile's k loop runs over both its products: first A . W[e]^T + bias[e], Kd wide;
  // the sum times row_scale[r] (r: packed row); then A2 . W2^T + bias2 is added, the same Kd, lda and
  // ldw; row r goes to C[scatter[r], :], plus addend[scatter[r], :] if there is one.  The last of the E
  // segments holds the tokens without a routed row, whose tiles run the second product alone.
  const unsigned char* A2;
  const unsigned char* W2;
  const float* bias2;
};

// Scratch of the split-K tail: per XCD as many partial tiles as workgroups are resident
// there (64 at most on a 256-CU device: 32 CUs x 2 workgroups), 256 KiB each at most.
constexpr int SPLITK_PARTS = 8 * 64;
constexpr size_t SPLITK_TILE_BYTES = 256 * 256 * 4;
constexpr size_t SPLITK_COUNT_BYTES = SPLITK_PARTS * sizeof(int);
constexpr size_t SPLITK_WS_BYTES = SPLITK_COUNT_BYTES + 8 * 32 * SPLITK_TILE_BYTES;
// Tiles are cut along K only from this K on.  Writing a part's partial sums and reading them
// back costs about as much as 20 k-tiles of 64, whatever K is (all workgroups do it at the same
// time, so it is memory traffic, not latency); below K = 2048 a tile is done sooner than that.
// (Measured, layer step: small 0.129 -> 0.119 ms, medium 0.659 -> 0.647 ms with the limit.)
constexpr int SPLITK_MIN_K = 2048;

// tanh-form GELU: 0.5 v (1 + tanh u) == v / (1 + exp(-2 u)) == v / (1 + 2^(v (c1 + c2 v^2))).
// The reciprocal is the hardware's (1 ulp), like the exponential: both far below the bf16 rounding
// of the stored value; a correctly rounded division took 10 of 20 instructions.
__device__ __forceinline__ float gelu_tanh_fast(float v) {
  const float e = __builtin_amdgcn_exp2f(v * fmaf(-0.10294324f, v * v, -2.3022082f));
  return v * __builtin_amdgcn_rcpf(1.0f + e);
}

__device__ __forceinline__ uint32_t cvt_pk_bf16(float a, float b) {
  f32x2_t f = {a, b};
  bf16x2_t h = __builtin_convertvector(f, bf16x2_t);
  return __builtin_bit_cast(uint32_t, h);
}

// Sum of two pairs of bf16 in fp32, rounded once.
__device__ __forceinline__ uint32_t add_bf16x2(uint32_t a, uint32_t b) {
  const float lo = __uint_as_float(a << 16) + __uint_as_float(b << 16);
  const float hi = __uint_as_float(a & 0xffff0000u) + __uint_as_float(b & 0xffff0000u);
  return cvt_pk_bf16(lo, hi);
}

// A precaution between the last matrix instruction and instructions written out in asm that
// read its results: the compiler inserts the wait states an MFMA result needs ahead of the
// instructions it schedules itself, and is not known to do so ahead of these.
__device__ __forceinline__ void mfma_results_settle() {
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
}

// 16-byte store / loads at device scope (sc1: past the caches that are not shared by the whole
// device), for data handed from one workgroup to another inside a kernel.  The store is not
// waited for here (follow it with a vmcnt(0) wait before publishing); the loads return when they
// have arrived.
__device__ __forceinline__ void store16_device_scope(float* p, f32x4_t v) {
  // (the wait state after it: a store of more than 8 bytes per lane still reads its data
  // registers when the next instruction issues, and the compiler, which keeps that hazard for
  // its own stores, does not know that this is one)
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}

// Sixteen loads in flight at once: four pieces 1 KiB apart from each of four bases.  (The
// reader of split-K partial sums has nothing to overlap a round trip to memory with: what
// counts is how few round trips it makes.)
__device__ __forceinline__ void load16x16_device_scope(const float* p0, const float* p1, const float* p2,
                                                       const float* p3, f32x4_t (&t)[16]) {
  asm volatile(
      "global_load_dwordx4 %0, %16, off sc1\n\t"
      "global_load_dwordx4 %1, %16, off offset:1024 sc1\n\t"
      "global_load_dwordx4 %2, %16, off offset:2048 sc1\n\t"
      "global_load_dwordx4 %3, %16, off offset:3072 sc1\n\t"
      "global_load_dwordx4 %4, %17, off sc1\n\t"
      "global_load_dwordx4 %5, %17, off offset:1024 sc1\n\t"
      "global_load_dwordx4 %6, %17, off offset:2048 sc1\n\t"
      "global_load_dwordx4 %7, %17, off offset:3072 sc1\n\t"
      "global_load_dwordx4 %8, %18, off sc1\n\t"
      "global_load_dwordx4 %9, %18, off offset:1024 sc1\n\t"
      "global_load_dwordx4 %10, %18, off offset:2048 sc1\n\t"
      "global_load_dwordx4 %11, %18, off offset:3072 sc1\n\t"
      "global_load_dwordx4 %12, %19, off sc1\n\t"
      "global_load_dwordx4 %13, %19, off offset:1024 sc1\n\t"
      "global_load_dwordx4 %14, %19, off offset:2048 sc1\n\t"
      "global_load_dwordx4 %15, %19, off offset:3072 sc1\n\t"
      "s_waitcnt vmcnt(0)"
      : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]), "=&v"(t[7]),
        "=&v"(t[8]), "=&v"(t[9]), "=&v"(t[10]), "=&v"(t[11]), "=&v"(t[12]), "=&v"(t[13]), "=&v"(t[14]), "=&v"(t[15])
      : "v"(p0), "v"(p1), "v"(p2), "v"(p3)
      : "memory");
}

// Direct-to-LDS copy through a buffer descriptor: 16 bytes per lane from base + voff + soff to 1 KiB
// of consecutive LDS.  An offset of BUFFER_SPAN or more is outside the buffer and reads zero;
// BUFFER_NOWHERE is, whether or not the range check counts soff (at most two rows of BUFFER_K bf16).
constexpr int64_t BUFFER_SPAN = 0xF0000000ll;
constexpr int BUFFER_K = 1 << 24;
constexpr uint32_t BUFFER_NOWHERE = 0xF8000000u;
__device__ __forceinline__ void buffer_to_lds16(const unsigned char* base, unsigned char* lds, uint32_t voff, uint32_t soff) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(
      __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), 0, static_cast<uint32_t>(BUFFER_SPAN), 0x00020000),
      SCMOE_LDS_PTR(lds), 16, voff, soff, 0, 0);
#endif
}

// f(integral_constant<int, I>) for I = B .. N-1, unrolled at compile time.
template <int B, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < N) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, N>(f);
  }
}

// Workgroup barrier of the main loops.  __syncthreads() carries workgroup-scope fences, for
// which the compiler drains the vector-memory counter (s_waitcnt vmcnt(0)): that would wait
// for every global -> LDS copy in flight, including the ones requested for later k-tiles, and
// undo the multi-stage pipeline.  The kernels wait for exactly the copies they need with an
// explicit vmcnt before the barrier; this barrier only orders the LDS traffic.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One product of a launch of the direct grouped GEMM (ffn_direct.hip).  g.offsets == nullptr: one
// dense segment of max_rows rows; otherwise max_rows bounds the packed rows.
struct DirectJob {
  GemmArgs g;
  bool act;
  int max_rows;
};
// One launch for one or two products (any width that is a multiple of 8, either storage type).
int launch_gemm_direct(const DirectJob* jobs, int n, int dtype, hipStream_t stream);

}  // namespace scmoe
