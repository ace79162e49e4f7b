// Grouped GEMM whose operands go straight from global memory into matrix-instruction
// registers: the fp32 expert computation, bf16 layers whose widths the tiled kernel does not
// cover, and bf16 calls of a few rows per expert (decode steps), which are bound by streaming
// the weights (ScMoE paper Eq. (1); experts are two-layer MLPs, Sec. 2.1; the memory-limited
// inference setting is Sec. 5.3).
//
//   C[r, n] = act( sum_k A[row(r), k] * W[e, n, k] + bias[e, n] ),  r in segment e
//
// A workgroup owns 16 MI rows x 16 NJ columns of one segment and its waves split K among
// themselves: every wave walks its own share of k for the whole tile, so no wave ever waits for
// another one, there is no LDS and no barrier in the loop, and a call whose tiles are few still
// has WK times as many waves in flight.  At the end the waves' sums meet in LDS, are added in
// wave order (the result does not depend on timing), and every wave finishes a share of the tile.
//  * An operand fragment is 16 rows x 64 bytes, lane l holding 16-byte piece l / 16 of row
//    l % 16: 32 k of bf16, one v_mfma_f32_16x16x32_bf16; or 16 k of fp32, four
//    v_mfma_f32_16x16x4_f32, the c-th of which takes the c-th element of every piece (the k
//    order inside a fragment is permuted alike for both operands, which a sum does not notice).
//    fp32 products and sums are exact fused multiply-adds in fp32, like the vector ALU's.
//  * The fragments of the next PF steps are in flight while one is multiplied (a ring of
//    registers; loads complete in order, so the wait for a step leaves the others in flight).
//  * fp32: 64 x 64 tiles need 16 bytes per clock and compute unit from the L1 at the full rate of
//    the fp32 matrix instruction, so the loop runs at that rate without LDS.
//  * A segment's last tile multiplies only the 16-row subtiles that hold rows (loop variants of
//    1, 2 and 4 subtiles).
//  * One launch can run two products of different shapes (the routed and the shared experts').
#include "mfma_common.hpp"

namespace scmoe {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

struct DirectArgs {
  GemmArgs j[2];       // offsets == nullptr: one dense segment of rows[] rows
  int rows[2];
  int act[2];
  int blocks0;         // workgroups of job 0; the others belong to job 1
};

template <bool F32, int MI, int NJ, int WK>
struct DirectCfg {
  static constexpr int BM = 16 * MI, BN = 16 * NJ, THREADS = 64 * WK;
  static constexpr int PARTS = WK > 4 ? 4 : WK;                 // sums that meet in LDS at the end
  static constexpr int LDS = PARTS * MI * NJ * 1024;
  static_assert(MI == 2 || MI == 4, "row subtiles");
  static_assert(WK == 4 || WK == 8, "waves");
  static_assert(LDS <= 64 * 1024, "static LDS");
};

template <bool F32>
__device__ __forceinline__ f32x4_t direct_mfma(u32x4_t w, u32x4_t x, f32x4_t acc) {
  if constexpr (F32) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[c]), __uint_as_float(x[c]), acc, 0, 0, 0);
    return acc;
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), acc, 0, 0, 0);
  }
}

template <bool F32, int MI, int NJ, int WK>
__global__ __launch_bounds__(64 * WK, 2) void gemm_direct_kernel(const DirectArgs args) {
  using CFG = DirectCfg<F32, MI, NJ, WK>;
  constexpr int EB = F32 ? 4 : 2;
  __shared__ __attribute__((aligned(16))) f32x4_t red[CFG::PARTS][MI * NJ][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  int b = blockIdx.x;
  const int which = b >= args.blocks0 ? 1 : 0;
  if (which) b -= args.blocks0;
  const GemmArgs& p = args.j[which];
  const int act = args.act[which];
  const int mt = b / p.nt;
  const int n0 = (b - mt * p.nt) * CFG::BN;

  // ---- which segment: 64 at a time, one per lane ---------------------------------------------
  int e = 0, row0 = 0, row_end = 0;
  if (p.offsets == nullptr) {
    row0 = mt * CFG::BM;
    row_end = args.rows[which];
    if (row0 >= row_end) return;
  } else {
    int left = mt;
    bool found = false;
    for (int e0 = 0; e0 < p.E; e0 += 64) {
      const int q = e0 + lane;
      const int s = p.offsets[q < p.E ? q : p.E], t = p.offsets[q + 1 < p.E ? q + 1 : p.E];
      const int tiles = (t - s + CFG::BM - 1) / CFG::BM;        // (0 past the last segment)
      int incl = tiles;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off, 64);
        if (lane >= off) incl += up;
      }
      const unsigned long long hit = __ballot(incl > left);
      if (hit != 0) {
        const int at = __builtin_ctzll(hit);
        e = e0 + at;
        row0 = __builtin_amdgcn_readlane(s, at) +
               (left - (__builtin_amdgcn_readlane(incl, at) - __builtin_amdgcn_readlane(tiles, at))) * CFG::BM;
        row_end = __builtin_amdgcn_readlane(t, at);
        found = true;
        break;
      }
      left -= __builtin_amdgcn_readlane(incl, 63);
    }
    if (!found) return;
  }

  // ---- operand rows of this lane (rows past the segment or past N re-read the last one) --------
  const unsigned char* ap[MI];
  const unsigned char* bp[NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    int r = row0 + i * 16 + l16;
    if (r > row_end - 1) r = row_end - 1;
    const int64_t src = p.gather ? p.gather[r] : r;
    ap[i] = p.A + src * p.lda * EB + lq * 16;
  }
  const unsigned char* We = p.W + static_cast<int64_t>(e) * p.N * p.ldw * EB + lq * 16;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    int n = n0 + j * 16 + l16;
    if (n > p.N - 1) n = p.N - 1;
    bp[j] = We + static_cast<int64_t>(n) * p.ldw * EB;
  }
  // ---- this wave's share of the finished tile: fragments wave, wave + WK, ... -------------------
  constexpr int FPW = (MI * NJ + WK - 1) / WK;
  f32x4_t bias4[FPW];
  int orow[FPW];                       // output row
  float rscale[FPW];
#pragma unroll
  for (int f = 0; f < FPW; ++f) {
    const int q = wave + f * WK, i = q / NJ, jj = q - i * NJ;
    const int n = n0 + jj * 16 + 4 * lq;
    int r = row0 + i * 16 + l16;
    if (r > row_end - 1) r = row_end - 1;
    bias4[f] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    if (p.bias != nullptr && n < p.N) bias4[f] = *reinterpret_cast<const f32x4_t*>(p.bias + static_cast<int64_t>(e) * p.N + n);
    orow[f] = r;
    rscale[f] = 1.0f;
    if (p.scatter != nullptr) {
      orow[f] = p.scatter[r];
      rscale[f] = p.row_scale[orow[f]];
    } else if (p.row_scale != nullptr) {
      rscale[f] = p.row_scale[2 * static_cast<int64_t>(r)];
    }
  }

  // ---- the sums over this wave's share of k ---------------------------------------------------
  const int pieces = p.Kd * EB / 16;                            // 16-byte pieces per row
  const int full = pieces >> 2, tail = pieces & 3;              // whole 64-byte steps, pieces of a last one
  const int s0 = static_cast<int>(static_cast<int64_t>(wave) * full / WK);
  const int s1 = static_cast<int>(static_cast<int64_t>(wave + 1) * full / WK);
  const bool has_tail = tail != 0 && wave == WK - 1;
  const int subs = (row_end - row0 + 15) >> 4;                  // subtiles that hold rows
  auto body = [&](auto ns_c) {
    constexpr int NS = decltype(ns_c)::value;
    constexpr int PF = F32 ? (NS >= 4 ? 2 : 3) : (NS >= 4 ? 3 : NS == 2 ? 4 : 6);
    f32x4_t acc[NS][NJ];
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    u32x4_t ra[PF][NS], rb[PF][NJ];
    const unsigned char* a[NS];
    const unsigned char* w[NJ];
#pragma unroll
    for (int i = 0; i < NS; ++i) a[i] = ap[i] + static_cast<int64_t>(s0) * 64;
#pragma unroll
    for (int j = 0; j < NJ; ++j) w[j] = bp[j] + static_cast<int64_t>(s0) * 64;
    auto load = [&](int u) {                                    // step u from the pointers into ring slot u
#pragma unroll
      for (int j = 0; j < NJ; ++j) rb[u][j] = *reinterpret_cast<const u32x4_t*>(w[j] + u * 64);
#pragma unroll
      for (int i = 0; i < NS; ++i) ra[u][i] = *reinterpret_cast<const u32x4_t*>(a[i] + u * 64);
    };
    auto compute = [&](int u) {
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = direct_mfma<F32>(rb[u][j], ra[u][i], acc[i][j]);
    };
    auto advance = [&]() {
#pragma unroll
      for (int i = 0; i < NS; ++i) a[i] += PF * 64;
#pragma unroll
      for (int j = 0; j < NJ; ++j) w[j] += PF * 64;
    };
    int n = s1 - s0;
    if (n >= PF) {
#pragma unroll
      for (int u = 0; u < PF; ++u) load(u);
      advance();
      n -= PF;
      for (; n >= PF; n -= PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
          compute(u);
          load(u);
        }
        advance();
      }
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        compute(u);
        if (u < n) load(u);                                     // (uniform)
      }
    } else {
#pragma unroll
      for (int u = 0; u < PF; ++u)
        if (u < n) load(u);
    }
#pragma unroll
    for (int u = 0; u < PF; ++u)
      if (u < n) compute(u);
    if (has_tail) {                                             // pieces past the end of a row count as zeros
      const bool in = lq < tail;
      const int64_t off = in ? static_cast<int64_t>(full) * 64 : 0;
      const u32x4_t zero = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(in ? bp[j] + off : bp[j] - lq * 16);
        rb[0][j] = in ? v : zero;
      }
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(in ? ap[i] + off : ap[i] - lq * 16);
        ra[0][i] = in ? v : zero;
      }
      compute(0);
    }
    // more than four waves: the upper half hands its sums to the lower half first
    constexpr int P = CFG::PARTS;
    if constexpr (WK > P) {
      if (wave >= P) {
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) red[wave - P][i * NJ + j][lane] = acc[i][j];
      }
      __syncthreads();
      if (wave < P) {
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) red[wave][i * NJ + j][lane] += acc[i][j];   // (this lane's own slots)
      }
    } else {
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) red[wave][i * NJ + j][lane] = acc[i][j];
    }
  };
  if (subs <= 1) body(std::integral_constant<int, 1>{});
  else if (MI == 2 || subs == 2) body(std::integral_constant<int, 2>{});
  else body(std::integral_constant<int, MI>{});
  __syncthreads();

  // ---- sum of the waves' parts, bias, activation, decode, store ---------------------------------
  // acc[v] = output row l16 of its subtile, column 4 lq + v of its column block
#pragma unroll
  for (int f = 0; f < FPW; ++f) {
    const int q = wave + f * WK, i = q / NJ, jj = q - i * NJ;
    if (i >= subs || i >= MI) continue;                         // (wave-uniform)
    f32x4_t v = red[0][q][lane];
#pragma unroll
    for (int s = 1; s < CFG::PARTS; ++s) v += red[s][q][lane];
    v += bias4[f];
    if (act) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if constexpr (F32) v[c] = gelu_f32(v[c], p.gelu_mode);
        else v[c] = (p.gelu_mode == SCMOE_GELU_TANH) ? gelu_tanh_fast(v[c]) : gelu_erf_fast(v[c]);
      }
    }
    v *= rscale[f];
    const int r = row0 + i * 16 + l16, n = n0 + jj * 16 + 4 * lq;
    if (r >= row_end || n >= p.N) continue;
    if (p.addend != nullptr) {
      const unsigned char* ad = p.addend + (static_cast<int64_t>(orow[f]) * p.ldadd + n) * EB;
      if constexpr (F32) {
        v += *reinterpret_cast<const f32x4_t*>(ad);
      } else {
        const uint2 q2 = *reinterpret_cast<const uint2*>(ad);
        v[0] += __uint_as_float(q2.x << 16);
        v[1] += __uint_as_float(q2.x & 0xffff0000u);
        v[2] += __uint_as_float(q2.y << 16);
        v[3] += __uint_as_float(q2.y & 0xffff0000u);
      }
    }
    unsigned char* out = p.C + (static_cast<int64_t>(orow[f]) * p.ldc + n) * EB;
    if constexpr (F32) {
      *reinterpret_cast<f32x4_t*>(out) = v;
    } else {
      uint2 o;
      o.x = cvt_pk_bf16(v[0], v[1]);
      o.y = cvt_pk_bf16(v[2], v[3]);
      *reinterpret_cast<uint2*>(out) = o;
    }
  }
}

// ---- host side ----------------------------------------------------------------------------------

template <bool F32, int MI, int NJ, int WK>
static int launch_direct_cfg(const DirectJob* jobs, int n, hipStream_t stream) {
  using CFG = DirectCfg<F32, MI, NJ, WK>;
  DirectArgs a{};
  int64_t blocks[2] = {0, 0};
  for (int q = 0; q < n; ++q) {
    a.j[q] = jobs[q].g;
    a.j[q].nt = (a.j[q].N + CFG::BN - 1) / CFG::BN;
    a.rows[q] = jobs[q].max_rows;
    a.act[q] = jobs[q].act ? 1 : 0;
    // upper bound on row tiles: sum_e ceil(c_e / BM) <= rows / BM + (segments that can hold a row)
    const int64_t rows = jobs[q].max_rows;
    const int64_t segs = a.j[q].offsets == nullptr ? 1 : (a.j[q].E < rows ? a.j[q].E : rows);
    blocks[q] = (a.j[q].offsets == nullptr ? (rows + CFG::BM - 1) / CFG::BM : rows / CFG::BM + segs) * a.j[q].nt;
  }
  if (blocks[0] + blocks[1] > 0x7fffffffLL) return SCMOE_ERR_SHAPE;
  a.blocks0 = static_cast<int>(blocks[0]);
  hipLaunchKernelGGL((gemm_direct_kernel<F32, MI, NJ, WK>), dim3(static_cast<unsigned>(blocks[0] + blocks[1])),
                     dim3(CFG::THREADS), 0, stream, a);
  return launch_status();
}

template <bool F32>
static int launch_direct_type(const DirectJob* jobs, int n, hipStream_t stream) {
  // 64 x 64 tiles; 32 x 32 when those would leave compute units idle
  int64_t tiles = 0;
  for (int q = 0; q < n; ++q) {
    const int64_t rows = jobs[q].max_rows, segs = jobs[q].g.offsets == nullptr ? 1 : (jobs[q].g.E < rows ? jobs[q].g.E : rows);
    tiles += ((rows + 63) / 64 + segs - 1) * ((jobs[q].g.N + 63) / 64);
  }
  if (tiles <= num_cus()) return launch_direct_cfg<F32, 2, 2, 8>(jobs, n, stream);
  return launch_direct_cfg<F32, 4, 4, 4>(jobs, n, stream);
}

int launch_gemm_direct(const DirectJob* jobs, int n, int dtype, hipStream_t stream) {
  if (n < 1 || n > 2) return SCMOE_ERR_ARG;
  for (int q = 0; q < n; ++q)
    if (jobs[q].g.xrows != 0 || jobs[q].g.N < 1 || jobs[q].g.Kd < 1 || (jobs[q].g.Kd % 8) || (jobs[q].g.N % 8)) return SCMOE_ERR_ARG;
  return dtype == SCMOE_BF16 ? launch_direct_type<false>(jobs, n, stream) : launch_direct_type<true>(jobs, n, stream);
}

}  // namespace scmoe
