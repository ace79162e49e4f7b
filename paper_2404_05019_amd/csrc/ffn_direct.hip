// Grouped GEMM without operand tiles that a workgroup shares: the fp32 expert computation, bf16 layers whose
// widths the tiled kernel does not cover, and bf16 calls of a few rows per expert (decode steps), which are bound by streaming
// the weights (ScMoE paper Eq. (1); experts are two-layer MLPs, Sec. 2.1; the memory-limited
// inference setting is Sec. 5.3).
//
//   C[r, n] = act( sum_k A[row(r), k] * W[e, n, k] + bias[e, n] ),  r in segment e
//
// A workgroup owns 16 MI rows x 16 NJ columns of one segment and its four waves split K among
// themselves: every wave walks its own share of k for the whole tile, so no wave ever waits for
// another one, there is no barrier in the loop, and a call whose tiles are few still has four times as
// many waves in flight.  At the end the waves' sums meet in LDS, are added in wave order (the
// result does not depend on timing), and every wave finishes a share of the tile.
//  * An operand fragment is 16 rows x 64 bytes, lane l holding 16-byte piece l / 16 of row
//    l % 16: 32 k of bf16, one v_mfma_f32_16x16x32_bf16; or 16 k of fp32, four
//    v_mfma_f32_16x16x4_f32, the c-th of which takes the c-th element of every piece (the k
//    order inside a fragment is permuted alike for both operands, which a sum does not notice).
//    fp32 products and sums are exact fused multiply-adds in fp32, like the vector ALU's.
//  * Small tiles: a wave's fragments come through a ring of its own in LDS, by copies whose lanes 4 r to
//    4 r + 3 share the 64 bytes of row r.  Loaded as the instruction takes them, 16 neighbouring lanes
//    read 16 rows, which takes the compute unit's address path up to four times as long: from the
//    caches 18-38 B/ns a compute unit, so 63-125, and streaming weights asks for 25 of them and as much
//    again of activations.  Layer us, registers / rings: 16 tokens, d = 1024, E = 16 75 / 70, 32 tokens,
//    d = 2048 235 / 213, 300 tokens, d = 512 52 / 47; fp32, 200 tokens, d = 1024 223 / 202, 64 tokens, d = 2048,
//    E = 8 340 / 308.  The copies of the next PF steps are in flight while a step is multiplied.
//  * 64 x 64 tiles: fragments straight into registers, two or three steps ahead; fp32 94 of 153 TFLOP/s at
//    4096 tokens, d = 1024, F = 2048, E = 8 (the vector ALUs: 20-30).  Small tiles the same way where rows do not
//    begin at 128-byte lines: the 64 bytes of a copy then mostly lie in two lines, and that costs more than the
//    address path saves (figures at launch_direct_type).
//  * Few rows: the weights arrive at 4.7 TB/s (8 tokens, 235 MB a launch) to 5.7 TB/s (64 tokens, 537
//    MB); a plain read of that size reaches 6.3.
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
constexpr int GRID_X = 1 << 16;   // workgroups per row of the grid (the runtime takes fewer than 2^32 work-items in x);
                                  // those past the last tile find no row and leave

constexpr int REGS = -1;          // SLOTS: no rings, operands straight into registers

template <bool F32, int MI, int NJ, int SLOTS>
struct DirectCfg {
  static constexpr int BM = 16 * MI, BN = 16 * NJ, WK = 4, THREADS = 64 * WK;
  // Operands through rings in LDS, except where REGS asks for registers and for 64 x 64 tiles, whose rings would hold two steps only
  // (fp32: 4096 tokens, d = 1024, E = 8 727 us of layer time through registers, 739 through LDS; 3000 tokens
  // of 1000 columns, bf16, 355 / 394).
  static constexpr bool RING = MI * NJ < 16 && SLOTS != REGS;
  static constexpr int STEP = (MI + NJ) * 1024;                 // bytes of a ring slot: one step's fragments
  static constexpr int FIT = 64 / (WK * (MI + NJ));             // 64 KiB, so that two workgroups fit a compute unit
  static constexpr int PF = SLOTS > 0 ? SLOTS : FIT < 5 ? FIT : 5;  // ring slots per wave (SLOTS = 0: what fits)
  static constexpr int RED = WK * MI * NJ * 1024;               // sums (in the rings' place at the end)
  static constexpr int LDS = RING && WK * PF * STEP > RED ? WK * PF * STEP : RED;
  static_assert(MI == 1 || MI == 2 || MI == 4, "row subtiles");
  static_assert(LDS <= 64 * 1024, "static LDS");
};

template <bool F32, int MI, int NJ, int SLOTS>
__global__ __launch_bounds__(256, 2) void gemm_direct_kernel(const DirectArgs args) {
  using CFG = DirectCfg<F32, MI, NJ, SLOTS>;
  constexpr int EB = F32 ? 4 : 2, WK = CFG::WK;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[CFG::LDS];
  auto& red = *reinterpret_cast<f32x4_t(*)[WK][MI * NJ][64]>(smem);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  int b = blockIdx.y * GRID_X + blockIdx.x;
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
  const unsigned char* const abase = p.A;
  const unsigned char* const wbase = p.W + static_cast<int64_t>(e) * p.N * p.ldw * EB;
  // RING: lane l of a copy fetches 16 bytes of row l / 4 of a fragment, so that four lanes share 64
  // bytes; otherwise a lane loads what it multiplies.
  const int crow = CFG::RING ? lane >> 2 : l16, cpiece = CFG::RING ? (lane & 3) ^ swz<4>(crow) : lq;
  int64_t ao[MI], wo[NJ];
  auto a_row = [&](int r) {                                     // byte offset of the packed row r
    if (r > row_end - 1) r = row_end - 1;
    const int64_t src = p.gather ? p.gather[r] : r;
    return src * p.lda * EB;
  };
  auto w_row = [&](int n) {
    if (n > p.N - 1) n = p.N - 1;
    return static_cast<int64_t>(n) * p.ldw * EB;
  };
#pragma unroll
  for (int i = 0; i < MI; ++i) ao[i] = a_row(row0 + i * 16 + crow) + cpiece * 16;
#pragma unroll
  for (int j = 0; j < NJ; ++j) wo[j] = w_row(n0 + j * 16 + crow) + cpiece * 16;
  // ---- what the epilogue needs of fragment (i, j) of the tile ------------------------------------
  struct Finish { f32x4_t bias; int orow; float rscale; };
  auto finish_loads = [&](int i, int jj) {
    Finish t;
    const int n = n0 + jj * 16 + 4 * lq;
    int r = row0 + i * 16 + l16;
    if (r > row_end - 1) r = row_end - 1;
    t.bias = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    if (p.bias != nullptr && n < p.N) t.bias = *reinterpret_cast<const f32x4_t*>(p.bias + static_cast<int64_t>(e) * p.N + n);
    t.orow = r;                                                 // output row
    t.rscale = 1.0f;
    if (p.scatter != nullptr) {
      t.orow = p.scatter[r];
      t.rscale = p.row_scale[t.orow];
    } else if (p.row_scale != nullptr) {
      t.rscale = p.row_scale[2 * static_cast<int64_t>(r)];
    }
    return t;
  };
  // bias, activation, decode, store: v[c] = row l16 of subtile i, column 4 lq + c of column block jj
  auto finish = [&](int i, int jj, f32x4_t v, const Finish& t) {
    v += t.bias;
    if (act) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if constexpr (F32) v[c] = gelu_f32(v[c], p.gelu_mode);
        else v[c] = (p.gelu_mode == SCMOE_GELU_TANH) ? gelu_tanh_fast(v[c]) : gelu_erf_fast(v[c]);
      }
    }
    v *= t.rscale;
    const int r = row0 + i * 16 + l16, n = n0 + jj * 16 + 4 * lq;
    if (r >= row_end || n >= p.N) return;
    if (p.addend != nullptr) {
      const unsigned char* ad = p.addend + (static_cast<int64_t>(t.orow) * p.ldadd + n) * EB;
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
    unsigned char* out = p.C + (static_cast<int64_t>(t.orow) * p.ldc + n) * EB;
    if constexpr (F32) {
      *reinterpret_cast<f32x4_t*>(out) = v;
    } else {
      uint2 o;
      o.x = cvt_pk_bf16(v[0], v[1]);
      o.y = cvt_pk_bf16(v[2], v[3]);
      *reinterpret_cast<uint2*>(out) = o;
    }
  };
  // split K: a wave finishes fragments wave, wave + WK, ... of the tile
  constexpr int FPW = (MI * NJ + WK - 1) / WK;
  Finish fin[FPW];
#pragma unroll
  for (int f = 0; f < FPW; ++f) fin[f] = finish_loads((wave + f * WK) / NJ, (wave + f * WK) % NJ);

  // ---- the sums over this wave's share of k ---------------------------------------------------
  const int pieces = p.Kd * EB / 16;                            // 16-byte pieces per row
  const int full = pieces >> 2, tail = pieces & 3;              // whole 64-byte steps, pieces of a last one
  const int s0 = static_cast<int>(static_cast<int64_t>(wave) * full / WK);
  const int s1 = static_cast<int>(static_cast<int64_t>(wave + 1) * full / WK);
  const bool has_tail = tail != 0 && wave == WK - 1;
  const int subs = (row_end - row0 + 15) >> 4;                  // subtiles that hold rows
  unsigned char* const ring = smem + wave * (CFG::PF * CFG::STEP);
  uint32_t rbase = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(SCMOE_LDS_PTR(ring)));
  asm volatile("" : "+s"(rbase));                               // (plain integers: see gemm_bf16_kernel's lds0)
  const uint32_t rlane = rbase + (l16 * 4 + (lq ^ swz<4>(l16))) * 16;      // this lane's piece of a fragment
  typedef const __attribute__((address_space(3))) u32x4_t* lds_piece_ptr;
  auto sums_ring = [&](auto ns_c, auto& acc) {
    constexpr int NS = decltype(ns_c)::value;
    constexpr int PF = CFG::PF, LPS = NS + NJ;                  // copies per step
    static_assert(PF * LPS < 64, "vmcnt field");
    u32x4_t ra[2][NS], rb[2][NJ];
    // A wave starts in the middle of its share (another place for each tile) and wraps round: with
    // row strides of a power of two, tiles that walk k in step would all be at the same few memory
    // channels.
    // fp32: it starts at a multiple of 6 steps that depends on the columns and the segment alone, and
    // the steps past the last such multiple come last: the order of a row's sum, and so its bits, do
    // not depend on the other rows of the call or on the tile shape.  (Layer us with the place depending
    // on the tile / so, before the rings: 2048 tokens, d = 384, E = 8 158.6 / 160.8; 200 tokens, d = 1024,
    // E = 16 216 / 221; 64, d = 2048, E = 8 364 / 340; 8, d = 2048, E = 16 233 / 224; by the columns alone
    // the first is 164.8, not at all 162.6.)
    const int n = s1 - s0;
    constexpr int UNIT = F32 ? 6 : 4;
    const int starts = n / UNIT, round = starts * UNIT;           // steps that take part in the rotation
    const int first = starts > 0 ? ((F32 ? n0 / 64 * 5 + e * p.rotk : b * 5) + wave) % starts * UNIT : 0;
    int at = first, done = 0;                                     // the step to be requested next, and how many have been
    auto issue = [&](int slot) {
      const int step = s0 + (done < round ? at : done);
      ++done;
      at = at + 1 == round ? 0 : at + 1;
      const unsigned char* a = abase + static_cast<int64_t>(step) * 64;
      const unsigned char* w = wbase + static_cast<int64_t>(step) * 64;
      unsigned char* dst = ring + slot * CFG::STEP;
#pragma unroll
      for (int j = 0; j < NJ; ++j) __builtin_amdgcn_global_load_lds(SCMOE_GLB_PTR(w + wo[j]), SCMOE_LDS_PTR(dst + j * 1024), 16, 0, 0);
#pragma unroll
      for (int i = 0; i < NS; ++i) __builtin_amdgcn_global_load_lds(SCMOE_GLB_PTR(a + ao[i]), SCMOE_LDS_PTR(dst + (NJ + i) * 1024), 16, 0, 0);
    };
    auto read = [&](auto buf_c, int slot) {                       // the fragments of the step in `slot`
      constexpr int buf = decltype(buf_c)::value;
      const uint32_t at0 = rlane + slot * CFG::STEP;
#pragma unroll
      for (int j = 0; j < NJ; ++j) rb[buf][j] = *reinterpret_cast<lds_piece_ptr>(static_cast<uintptr_t>(at0 + j * 1024));
#pragma unroll
      for (int i = 0; i < NS; ++i) ra[buf][i] = *reinterpret_cast<lds_piece_ptr>(static_cast<uintptr_t>(at0 + (NJ + i) * 1024));
    };
    auto compute = [&](auto buf_c) {
      constexpr int u = decltype(buf_c)::value;
      // (fp32: element by element over all accumulators, so that no instruction waits for the
      // one before it)
#pragma unroll
      for (int c = 0; c < (F32 ? 4 : 1); ++c)
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            if constexpr (F32)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(rb[u][j][c]), __uint_as_float(ra[u][i][c]), acc[i][j], 0, 0, 0);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, rb[u][j]),
                                                                  __builtin_bit_cast(bf16x8_t, ra[u][i]), acc[i][j], 0, 0, 0);
          }
    };
    // until the oldest step in flight has landed (copies complete in issue order); `flying` steps are
    auto landed = [&](int flying) {
      static_for<0, PF>([&](auto f_c) {
        constexpr int f = decltype(f_c)::value, c = f * LPS;      // f younger ones may still be on their way
        if (flying == f + 1 || (f == PF - 1 && flying > f)) __builtin_amdgcn_s_waitcnt((c & 15) | ((c >> 4) << 14) | 0x0F70);
      });
      asm volatile("" ::: "memory");
    };
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    for (int t = 0; t < PF; ++t)
      if (t < n) issue(t);
    if (n > 0) {
      landed(done);
      read(B0{}, 0);
    }
    int slot = 0;                                                 // of the step in the registers
    // step t is in registers; step t + 1 is read while t is multiplied, then its slot's predecessor is refilled
    auto turn = [&](auto cur, auto next, int t) {
      const int after = slot + 1 == PF ? 0 : slot + 1;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // step t is in registers: its slot is free
      if (done < n) issue(slot);
      if (t + 1 < n) {
        landed(done - (t + 1));
        read(next, after);
      }
      __builtin_amdgcn_sched_barrier(0);
      compute(cur);
      __builtin_amdgcn_sched_barrier(0);
      slot = after;
    };
    for (int t = 0; t < n; t += 2) {
      turn(B0{}, B1{}, t);
      if (t + 1 < n) turn(B1{}, B0{}, t + 1);
    }
    if (has_tail) {                                             // pieces past the end of a row count as zeros
      const bool in = lq < tail;
      const u32x4_t zero = {0u, 0u, 0u, 0u};
      const int64_t off = static_cast<int64_t>(full) * 64 + (in ? lq * 16 : 0);   // (else the step's first piece, unused)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(wbase + w_row(n0 + j * 16 + l16) + off);
        rb[0][j] = in ? v : zero;
      }
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(abase + a_row(row0 + i * 16 + l16) + off);
        ra[0][i] = in ? v : zero;
      }
      compute(B0{});
    }
  };
  auto sums_regs = [&](auto ns_c, auto& acc) {
    constexpr int NS = decltype(ns_c)::value;
    constexpr int PF = NS >= 4 ? 3 : NS == 2 ? (F32 ? 3 : 4) : 6;
    u32x4_t ra[PF][NS], rb[PF][NJ];
    // The PF steps of a block are read from where `seek` has put the bases.  A wave starts in
    // the middle of its share (another block for each tile) and wraps round: with row strides of
    // a power of two, tiles that walk k in step would all be at the same few memory channels.
    // fp32: it starts at a multiple of 6 steps (whole blocks for every PF) that depends on the
    // columns and the segment alone, and the steps past the last such multiple come last: the order
    // of a row's sum, and so its bits, do not depend on the other rows of the call or on the tile
    // shape.  (Layer us with the place depending on the tile, and any PF / so: 2048 tokens,
    // d = 384, E = 8 158.6 / 160.8; 200 tokens, d = 1024, E = 16 216 / 221; 64, d = 2048, E = 8 364 / 340;
    // 8, d = 2048, E = 16 233 / 224; by the columns alone the first is 164.8, not at all 162.6.)
    int n = s1 - s0;
    const int all = n;
    constexpr int UNIT = F32 ? 6 : PF;
    static_assert(UNIT % PF == 0, "whole blocks");
    const int starts = n / UNIT, nblk = starts * (UNIT / PF);     // blocks that take part in the rotation
    int blk = starts > 0 ? ((F32 ? n0 / 64 * 5 + e * p.rotk : b * 5) + wave) % starts * (UNIT / PF) : 0;
    const unsigned char* a = nullptr;
    const unsigned char* w = nullptr;
    auto seek = [&](int step) {
      a = abase + static_cast<int64_t>(step) * 64;
      w = wbase + static_cast<int64_t>(step) * 64;
    };
    auto next_block = [&](int left) {                             // left: steps that come after the block
      if (all - left < nblk * PF) {
        blk = blk + 1 == nblk ? 0 : blk + 1;
        seek(s0 + blk * PF);
      } else {
        seek(s0 + (all - left));
      }
    };
    auto load = [&](int u) {                                      // step u of the block into ring slot u
#pragma unroll
      for (int j = 0; j < NJ; ++j) rb[u][j] = *reinterpret_cast<const u32x4_t*>(w + wo[j] + u * 64);
#pragma unroll
      for (int i = 0; i < NS; ++i) ra[u][i] = *reinterpret_cast<const u32x4_t*>(a + ao[i] + u * 64);
    };
    auto compute = [&](int u) {
      // (fp32: element by element over all accumulators, so that no instruction waits for the
      // one before it: a dependent one issues after 50 cycles, an independent one after 32)
#pragma unroll
      for (int c = 0; c < (F32 ? 4 : 1); ++c)
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            if constexpr (F32)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(rb[u][j][c]), __uint_as_float(ra[u][i][c]), acc[i][j], 0, 0, 0);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, rb[u][j]),
                                                                  __builtin_bit_cast(bf16x8_t, ra[u][i]), acc[i][j], 0, 0, 0);
          }
    };
    seek(s0 + blk * PF);
    if (n >= PF) {
#pragma unroll
      for (int u = 0; u < PF; ++u) load(u);
      n -= PF;
      next_block(n);
      for (; n >= PF; n -= PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
          compute(u);
          load(u);
          if (F32) __builtin_amdgcn_sched_barrier(0);           // (or the compiler gathers the loads at the loop's end)
        }
        next_block(n - PF);
      }
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        compute(u);
        if (u < n) load(u);                                     // (uniform)
        if (F32) __builtin_amdgcn_sched_barrier(0);
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
      const u32x4_t zero = {0u, 0u, 0u, 0u};
      const int64_t back = in ? 0 : lq * 16;        // (then: the step's first piece, unused)
      seek(full);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(w + (wo[j] - back));
        rb[0][j] = in ? v : zero;
      }
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(a + (ao[i] - back));
        ra[0][i] = in ? v : zero;
      }
      compute(0);
    }
  };
  auto body = [&](auto ns_c) {
    constexpr int NS = decltype(ns_c)::value;
    f32x4_t acc[NS][NJ];
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (CFG::RING) {
      sums_ring(ns_c, acc);
      __syncthreads();                                          // the rings have been read: the sums take their place
    } else {
      sums_regs(ns_c, acc);
    }
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) red[wave][i * NJ + j][lane] = acc[i][j];
  };
  if (MI == 1 || subs <= 1) body(std::integral_constant<int, 1>{});
  else if (MI == 2 || subs == 2) body(std::integral_constant<int, 2>{});
  else body(std::integral_constant<int, MI < 2 ? 2 : MI>{});
  __syncthreads();
#pragma unroll
  for (int f = 0; f < FPW; ++f) {
    const int q = wave + f * WK, i = q / NJ, jj = q - i * NJ;
    if (i >= subs || i >= MI) continue;                           // (wave-uniform)
    f32x4_t v = red[0][q][lane];
#pragma unroll
    for (int s = 1; s < WK; ++s) v += red[s][q][lane];
    finish(i, jj, v, fin[f]);
  }
}

// ---- host side ----------------------------------------------------------------------------------

template <bool F32, int MI, int NJ, int SLOTS>
static int launch_direct_cfg(const DirectJob* jobs, int n, hipStream_t stream) {
  using CFG = DirectCfg<F32, MI, NJ, SLOTS>;
  DirectArgs a{};
  int64_t blocks[2] = {0, 0};
  for (int q = 0; q < n; ++q) {
    GemmArgs& g = a.j[q];
    g = jobs[q].g;
    g.nt = (g.N + CFG::BN - 1) / CFG::BN;
    a.rows[q] = jobs[q].max_rows;
    a.act[q] = jobs[q].act ? 1 : 0;
    // upper bound on row tiles: sum_e ceil(c_e / BM) <= rows / BM + (segments that can hold a row)
    const int64_t rows = jobs[q].max_rows;
    const int64_t segs = g.E < rows ? g.E : rows;
    blocks[q] = (g.offsets == nullptr ? (rows + CFG::BM - 1) / CFG::BM : rows / CFG::BM + segs) * g.nt;
  }
  const int64_t total = blocks[0] + blocks[1];
  if (total > 0x7fffffffLL - GRID_X) return SCMOE_ERR_SHAPE;
  a.blocks0 = static_cast<int>(blocks[0]);
  if (n == 1) a.j[1].nt = 1;                                    // (workgroups past the last tile: no rows there)
  const dim3 grid(static_cast<unsigned>(total < GRID_X ? total : GRID_X), static_cast<unsigned>((total + GRID_X - 1) / GRID_X)),
      block(CFG::THREADS);
  hipLaunchKernelGGL((gemm_direct_kernel<F32, MI, NJ, SLOTS>), grid, block, 0, stream, a);
  return launch_status();
}

// Which tile, measured as a layer call's time (us) at d = 2048, F = 8192, E = 16 unless noted:
//  * 64 x 64: when that gives every compute unit a tile and the segments average 32 rows or more
//    (fp32, 4096 tokens, d = 1024, F = 2048, E = 8 727 against 763 with 32 x 32 in the first product and 830 in
//    both; bf16, 3000 tokens of 1000 columns 354 against 609).
//  * fp32, short K: 32 x 32 with two ring slots, five workgroups on a compute unit, whose starts and ends
//    overlap.  Up to 24 steps (64 x 64 / so: 2048 tokens, d = 384, E = 8 161.3 / 153.2; 700, d = 384, E = 4 86.0 / 77.4;
//    8000, d = 128 95.1 / 88.1; 20000, d = 64 84.3 / 78.9, d = 384 552.7 / 552.2); up to 40 where 64 x 64 tiles are fewer than 14 per
//    compute unit, whose rounds hide starts and ends by themselves (E = 8; tiles per unit: 1000, top-2, d = 520 154.7 /
//    145.7; 3000, d = 640 (8) 257.0 / 256.0; 3000, d = 512, F = 2048 (13) 323.9 / 322.1; 3000, d = 640, F = 2560 (16) 461.6 / 465.2;
//    8000, d = 640 (20) 587.4 / 595.0; 20000 (49) 1381 / 1411); up to 64 where they are fewer than two (2000, d =
//    256, F = 1024 93.9 / 80.6).
//  * 32 x 32: everything smaller; weights are streamed (64 tokens, shared expert on a second stream: 243
//    against 252 with 32 x 16 where that fits and 250 with 16 x 32).
//  * 16 x 16, bf16: when 32 x 32 tiles would put fewer than 16 waves on a compute unit, K is long and
//    no segment has more than 16 rows (8 tokens 133.5 against 138 with 32 x 32 or 16 x 32; 16 tokens, d =
//    1024 68 / 73); fp32 takes 32 x 16 there.
//  * 16 x 32, bf16: other calls of 32 rows and fewer a product (32 tokens 213 against 229; top-2 of 8 tokens,
//    d = 768 35.1 / 35.5).
//  * K of 32 steps and fewer (a wave has eight): two or three ring slots instead of four or five, so that more
//    workgroups are resident, whose starts overlap, if there are more than those two per compute unit (16 tokens, d = 1024, E = 16 64.9 / 61.4; 60 tokens, top-2, d =
//    512, E = 64 64.9 / 57.3; at 64 steps 64 tokens, d = 2048 237 / 258;
//    160 tiles, fp32, 256 tokens, d = 64 20.2 / 21.3).
//  * Rings only where both operands' rows begin at 128-byte lines, else registers (rings / registers; E = 8, 16 or 32,
//    F = 8/3 d): bf16, one stream, 300 tokens of 32 experts, d = 776 106.5 / 94.0, d = 1424 269.8 / 252.8; 40, d = 1000 54.0 /
//    49.9; 8, d = 1424 73.8 / 65.7; shared expert on a second stream, 100, d = 1424 123.0 / 112.8; 30 125.2 / 110.5; d = 544,
//    rows at every other 64 bytes, 300 60.0 / 59.0.  fp32, 100, d = 1000 117.5 / 101.1; 20, d = 520 35.2 / 32.5; 500, d =
//    520 (111 rows per segment) 87.8 / 81.7; but rings from 128 rows per segment on, where less of the time is streaming
//    weights (second stream, 500, d = 1000 254.7 / 267.7; 1000, top-2, d = 520 147.8 / 151.0).  And registers in fp32 for one
//    product alone of fewer than 10 rows per segment (four operator calls, weights new in every pass: 40 tokens of 16
//    experts, d = 768 94.0 / 83.0; 3, top-4 of 12, d = 1536 106.4 / 95.1; 22 of 12, d = 960 100.1 / 95.1; but 200 of 16, d =
//    1024 159.0 / 166.6; 120 of 8 100.8 / 104.3).  With the shared expert's product in the launch neither is the better one
//    throughout (16 tokens of 8, d = 1024 76.8 / 83.2; 64, d = 2048 309 / 333; 64, d = 1024 120.7 / 112.1; 32 108.7 / 102.0): rings.
template <bool F32>
static int launch_direct_type(const DirectJob* jobs, int n, hipStream_t stream) {
  constexpr int EB = F32 ? 4 : 2;
  int64_t tiles64 = 0, tiles32 = 0, rows = 0, segs = 0, most = 0;   // most: rows of a product
  int steps = 0;
  bool lines = true;                                               // rows begin at 128-byte lines
  for (int q = 0; q < n; ++q) {
    const GemmArgs& g = jobs[q].g;
    const int64_t r = jobs[q].max_rows, s = g.offsets == nullptr ? 1 : (g.E < r ? g.E : r);
    tiles64 += (r / 64 + s) * ((g.N + 63) / 64);
    tiles32 += (r / 32 + s) * ((g.N + 31) / 32);
    rows += r;
    segs += s;
    if (r > most) most = r;
    const int st = g.Kd * EB / 64;
    if (st > steps) steps = st;
    lines = lines && (g.lda * EB) % 128 == 0 && (g.ldw * EB) % 128 == 0;
  }
  const bool few_waves = tiles32 * 4 < 16 * num_cus() && steps >= 128, short_k = steps <= 32 && tiles32 > 2 * num_cus();
  const bool ring = (lines && !(F32 && n == 1 && rows < 10 * segs)) || (F32 && rows >= 128 * segs);
  if (tiles64 >= num_cus() && rows >= 32 * segs) {
    if (F32 && (steps <= 24 || tiles64 < (steps <= 40 ? 14 : steps <= 64 ? 2 : 0) * num_cus()))
      return ring ? launch_direct_cfg<F32, 2, 2, 2>(jobs, n, stream) : launch_direct_cfg<F32, 2, 2, REGS>(jobs, n, stream);
    return launch_direct_cfg<F32, 4, 4, REGS>(jobs, n, stream);
  }
  if constexpr (F32) {
    if (few_waves) return ring ? launch_direct_cfg<F32, 2, 1, 0>(jobs, n, stream) : launch_direct_cfg<F32, 2, 1, REGS>(jobs, n, stream);
  } else {
    if (few_waves && most <= 16) return ring ? launch_direct_cfg<F32, 1, 1, 0>(jobs, n, stream) : launch_direct_cfg<F32, 1, 1, REGS>(jobs, n, stream);
    if (most <= 32) {
      if (!ring) return launch_direct_cfg<F32, 1, 2, REGS>(jobs, n, stream);
      return short_k ? launch_direct_cfg<F32, 1, 2, 3>(jobs, n, stream) : launch_direct_cfg<F32, 1, 2, 0>(jobs, n, stream);
    }
  }
  if (!ring) return launch_direct_cfg<F32, 2, 2, REGS>(jobs, n, stream);
  return short_k ? launch_direct_cfg<F32, 2, 2, 2>(jobs, n, stream) : launch_direct_cfg<F32, 2, 2, 0>(jobs, n, stream);
}

int launch_gemm_direct(const DirectJob* jobs, int n, int dtype, hipStream_t stream) {
  if (n < 1 || n > 2) return SCMOE_ERR_ARG;
  for (int q = 0; q < n; ++q)
    if (jobs[q].g.xrows != 0 || jobs[q].g.N < 1 || jobs[q].g.Kd < 1 || (jobs[q].g.Kd % 8) || (jobs[q].g.N % 8)) return SCMOE_ERR_ARG;
  return dtype == SCMOE_BF16 ? launch_direct_type<false>(jobs, n, stream) : launch_direct_type<true>(jobs, n, stream);
}

}  // namespace scmoe
