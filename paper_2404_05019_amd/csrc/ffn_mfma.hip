// Expert computation (ScMoE paper Eq. (1); experts are two-layer MLPs, Sec. 2.1) in bf16
// on the CDNA4 matrix cores: a grouped GEMM over variable-length expert segments.
//
//   C[r, n] = act( sum_k A[row(r), k] * W[e, n, k] + bias[e, n] ),  r in segment e
//
// Both operands are K-contiguous ([rows, K] activations, [N, K] weights), which is the
// layout v_mfma_f32_16x16x32_bf16 wants: each lane feeds 8 consecutive k of one row.
//
// Design (gfx950):
//  * Persistent workgroups; each takes BM x BN output tiles (one expert per tile) from a
//    schedule derived on the device from offsets[] (no host round trip), and requests the
//    first k-tiles of its next tile before it runs the epilogue of the current one.  The
//    tiles of the last, partly filled round are cut along K (see the split-K block below).
//  * Global -> LDS copies use the direct-to-LDS form of the global load (16 bytes per
//    lane, no VGPR staging).  Such a load writes 1 KiB of consecutive LDS per wave, so the
//    bank-conflict swizzle is applied on the global side: the lane that fills LDS slot
//    (row, c) fetches k-chunk  c ^ swz(row)  of that row.
//  * N LDS stages and double-buffered register fragments: global loads run N - 1/2 k-tiles
//    ahead (a stage is refilled in two groups, see k_tile), LDS reads one half-step (16 MFMAs)
//    ahead, issued one behind each MFMA; two workgroup barriers per k-tile, which order LDS
//    traffic only (lds_barrier).
//  * The MFMA is issued with the weight fragment as its first operand, so a lane ends up
//    holding 4 consecutive output columns of one row; the epilogue re-assembles rows in a
//    small per-wave LDS patch and stores whole 128-byte lines.
//  * Workgroup ids congruent mod 8 land on one XCD and share its L2: the tiles in flight on
//    an XCD are neighbours inside one expert (they share A and W panels), and the XCDs are
//    dealt neighbouring chunks, so that all of them read the same experts' weights at a time
//    (TileSchedule).
//  * Rows can be gathered on load through an index array (the dispatch permutation, paper
//    Sec. 2.2 "input encode"), and the second GEMM can scatter, scale and add on store
//    ("output decode"), which lets the layer skip both permuted copies.
#include "mfma_common.hpp"
#include "coef_gate.hpp"
#include "gate_mfma.hpp"
#include <algorithm>
#include <atomic>
#include <math.h>

namespace scmoe {

template <int BM_, int BN_, int BK_, int WM_, int WN_, int NS_>
struct TileCfg {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, NS = NS_;   // NS: LDS stages
  static constexpr int WAVES = WM * WN, THREADS = 64 * WAVES;
  static constexpr int TM = BM / WM, TN = BN / WN;       // wave tile
  static constexpr int MI = TM / 16, NJ = TN / 16;       // 16x16 MFMA tiles per wave
  static constexpr int RB = BK * 2;                      // bytes of one LDS row
  static constexpr int CPR = RB / 16;                    // 16-byte chunks per row
  static constexpr int RPL = 64 / CPR;                   // rows filled by one wave-wide load
  static constexpr int A_BYTES = BM * RB, B_BYTES = BN * RB, STAGE = A_BYTES + B_BYTES;
  static constexpr int A_PER_WAVE = BM / RPL / WAVES, B_PER_WAVE = BN / RPL / WAVES;
  static constexpr int STG_ROW = TN * 2;                  // bytes of one row of a wave's epilogue staging patch
  static constexpr int STG_ROWS = (WAVES == 8 && NS * STAGE + 32 * WAVES * STG_ROW <= 160 * 1024) ? 32 : 16; // rows staged at a time (LDS budget)
  static constexpr int STG_BYTES = STG_ROWS * STG_ROW;
  static constexpr int LDS_BYTES = NS * STAGE + WAVES * STG_BYTES;
  // workgroups of this shape that fit one CU (512 VGPRs per SIMD lane, 160 KiB LDS)
  static constexpr int WG_PER_CU = (160 * 1024 / LDS_BYTES) < (8 / WAVES) ? (160 * 1024 / LDS_BYTES) : (8 / WAVES);
  // Row tiles per raster group.  A first GEMM (N = F) has many column tiles and an XCD's 32
  // tiles in flight are best a 6 x 5 patch of a group; a second GEMM (N = d) has few (8 at
  // d = 2048), and groups of 4 x 8 tiles coincide with the chunks the XCDs are dealt.
  static constexpr int GM_FIRST = 6, GM_SECOND = 4;
  static_assert(BM % (RPL * WAVES) == 0 && BN % (RPL * WAVES) == 0, "loads must divide evenly");
  static_assert((TM == 128 || TM == 64) && TN == 64 && (BK == 32 || BK == 64) && NS >= 2 && NS <= 4, "tile shape");
  static_assert(LDS_BYTES * WG_PER_CU <= 160 * 1024 && WG_PER_CU >= 1, "LDS budget");
};

// DEC: output decode in the epilogue of a second GEMM.  0: none.  1: row r of the packed
// output goes to token scatter[r]: C[scatter[r]] = addend[scatter[r]] + row_scale[scatter[r]] * row
// (addend may be null: nothing is added).
// 2: rows stay where they are: C[r] = addend[r] + row_scale[2 r] * row (row_scale: pairs of
// coefficients per row, the first one is used; either pointer may be null).
// 3: joint second GEMM of the shared and the routed expert of a token (see GemmArgs::A2); 4: the same with
// addend rows.
// XSEG: the launch may carry the dense extra segment (GemmArgs::xrows).
// EG > 0: the last workgroups do a layer's gate (up to 16 EG experts), its encode and its coefficient gate first.
struct GateGemmArgs : GemmArgs { GateWork w; };
template <class CFG, bool ACT, bool OFF32, int DEC, bool XSEG, int EG = 0>
__global__ __launch_bounds__(CFG::THREADS, CFG::WG_PER_CU * CFG::WAVES / 4) void gemm_bf16_kernel(const std::conditional_t<(EG > 0), GateGemmArgs, GemmArgs> p) {
  constexpr int BM = CFG::BM, BN = CFG::BN, BK = CFG::BK, RB = CFG::RB, CPR = CFG::CPR;
  constexpr int MI = CFG::MI, NJ = CFG::NJ, STAGE = CFG::STAGE, A_BYTES = CFG::A_BYTES;
  constexpr int NS = CFG::NS;
  constexpr int KS32 = BK / 32;                                 // 32-k MFMA steps per k-tile
  constexpr int HS = 2 * KS32;                                  // half-steps per k-tile
  constexpr int LPW = CFG::A_PER_WAVE + CFG::B_PER_WAVE;        // direct loads per wave and k-tile
  constexpr bool DECODE = DEC != 0;
  constexpr bool CAT = DEC >= 3, ADD = DECODE && DEC != 3;
  constexpr bool ROTK = BM < 256 && !CAT;                       // (the large tiles are for calls it does not help)
  static_assert(!(ACT && DEC != 0) && !(XSEG && DEC != 0) && DEC >= 0 && DEC <= 4, "the output decode belongs to second GEMMs without the extra segment");
  static_assert(!CAT || (OFF32 && NS == 2), "operands change at an even k-tile, by their scalar bases");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  if constexpr (EG > 0) {
    const int g = gridDim.x - 1 - blockIdx.x;
    if (g < p.w.workgroups) {
      gate_mfma<true, CFG::WAVES, EG, GATE_ENC_LAST, CFG::LDS_BYTES>(smem, g, static_cast<const unsigned char*>(p.w.x), p.w.ldx, p.w.Wg, p.w.bias, p.w.T, p.w.d,
                                                                     p.w.E, p.w.k, p.w.normalize, p.w.idx, p.w.gw, nullptr, p.w.enc, p.w.marks, p.w.call,
                                                                     p.w.workgroups);
      __syncthreads();                       // (the LDS becomes the stages of the tiles)
    } else if (g - p.w.workgroups < p.w.coef_workgroups) {
      coef_gate_rows<true, true, CFG::WAVES>(reinterpret_cast<float*>(smem), g - p.w.workgroups, p.w.coef_workgroups, static_cast<const unsigned char*>(p.w.xc), p.w.ldxc * 2,
                                 p.w.Wcg, p.w.cg_mode, p.w.T, p.w.d, p.w.coef);
      __syncthreads();
    }
  }

  // ---- tile schedule ------------------------------------------------------------------------
  const int nk1 = p.Kd / BK;               // k-tiles of one product
  const int nk_all = CAT ? 2 * nk1 : nk1;
  TileSchedule<BM, BN, ACT ? CFG::GM_FIRST : CFG::GM_SECOND, CAT> sched(p.nt, p.E, p.offsets, p.xrows, nk_all, p.splitk_part != nullptr && (CAT ? 2 : 1) * p.Kd >= SPLITK_MIN_K, CFG::WAVES,
                                                                            blockIdx.x & 7, gridDim.x >> 3);
  const int nslots = sched.nslots;
  int it = blockIdx.x >> 3;                // work item: a tile, one K-part of a tile of the last round, or a finish item
  if (it >= sched.ngemm + sched.nfin) return;
  int nk = nk_all;                         // k-tiles of the current item
  int rot = 0;                             // the one it starts with (the walk wraps round)
  int kmid = 0;                            // CAT: its k-tile at which the shared expert's operands begin

  // ---- per-lane source addresses of the direct-to-LDS loads -------------------------------
  // First row of the tile that this wave's A load i fills (RPL rows): the first half of the
  // loads covers the first halves of the wave tiles (rows 0 .. TM/2-1 of each), the second half
  // the second halves.
  auto a_block = [&](int i) {
    constexpr int H = CFG::A_PER_WAVE / 2, HALF = CFG::TM / 2;
    const int q = (wave * H + i % H) * CFG::RPL;                // row among the rows of that half
    return (q / HALF) * CFG::TM + (i / H) * HALF + q % HALF;
  };
  // OFF32 (both operands span less than BUFFER_SPAN, checked on the host): an address is a
  // wave-uniform base plus a 32-bit per-lane offset that stays the same for a whole tile: one
  // register per load and no vector address arithmetic between the barrier of a k-tile and its next
  // MFMA.  A comes through a buffer descriptor, with the k-tile as its scalar offset: rows past the
  // segment lie outside the buffer, read zeros and cost no memory traffic (as repeats of the last row
  // 4096 tokens of 32 experts, d = 1024, F = 2048 190 us, so 186; W the same way took 24-46 scalar
  // registers out of the k loop: 8192 tokens, d = 384 92.6 -> 93.6).  Otherwise full 64-bit per-lane
  // pointers.
  const unsigned char* aptr[OFF32 ? 1 : CFG::A_PER_WAVE];
  const unsigned char* bptr[OFF32 ? 1 : CFG::B_PER_WAVE];
  uint32_t aoff[OFF32 ? CFG::A_PER_WAVE : 1], boff[OFF32 ? CFG::B_PER_WAVE : 1];
  const unsigned char* abase = nullptr;     // OFF32: p.A / the expert's W, advanced to the item's first k-tile
  const unsigned char* wbase = nullptr;
  const unsigned char* abase2 = nullptr;    // CAT: the same for the operands from k-tile kmid on
  const unsigned char* wbase2 = nullptr;
  auto set_ptrs = [&](int e, int row0, int row_end, int n0, int kb) {   // kb: first k-tile of the item
    // The dense extra segment (operands of its own) and the fused output decode have
    // instantiations of their own: no kernel carries code it does not run (the register
    // allocation of the k loop feels every scalar that is live across it).
    const bool xs = XSEG && e == p.E;
    const int64_t lda = xs ? p.xlda : p.lda, ldw = xs ? p.xldw : p.ldw;
    const int32_t* gather = xs ? p.xgather : p.gather;
    const unsigned char* We = (xs ? p.xW : p.W + static_cast<int64_t>(e) * p.N * ldw * 2) + static_cast<int64_t>(kb) * RB;
    abase = (xs ? p.xA : p.A) + static_cast<int64_t>(kb) * RB;
    wbase = We;
    if constexpr (CAT) {
      abase2 = p.A2 + static_cast<int64_t>(kb - nk1) * RB;
      wbase2 = p.W2 + static_cast<int64_t>(kb - nk1) * RB;
    }
#pragma unroll
    for (int i = 0; i < CFG::A_PER_WAVE; ++i) {
      const int row = a_block(i) + lane / CPR;
      const int kc = (lane % CPR) ^ swz<CPR>(row);
      int m = row0 + row;
      const bool past = m > row_end - 1;
      if (past) m = row_end - 1;                 // (64-bit pointers: rows past the segment re-read its last row)
      const int64_t src = gather ? gather[m] : m;
      if constexpr (OFF32) aoff[i] = past ? BUFFER_NOWHERE : static_cast<uint32_t>(src * lda * 2 + kc * 16);
      else aptr[i] = abase + src * lda * 2 + kc * 16;
    }
#pragma unroll
    for (int i = 0; i < CFG::B_PER_WAVE; ++i) {
      const int row = (wave * CFG::B_PER_WAVE + i) * CFG::RPL + lane / CPR;
      const int kc = (lane % CPR) ^ swz<CPR>(row);
      int n = n0 + row;
      if (n > p.N - 1) n = p.N - 1;
      if constexpr (OFF32) boff[i] = static_cast<uint32_t>(static_cast<int64_t>(n) * ldw * 2 + kc * 16);
      else bptr[i] = We + static_cast<int64_t>(n) * ldw * 2 + kc * 16;
    }
  };
  // The copies of a k-tile come in two groups: W and the first half of every wave tile's rows
  // (W_A0), and the second half of those rows (A1).
  constexpr int A1_LPW = CFG::A_PER_WAVE / 2;                   // loads per wave of the group A1
  auto issue_a = [&](int kt, int stage, auto half_c) {
    constexpr int h = decltype(half_c)::value;
    if (ROTK && (kt += rot) >= nk) kt -= nk;
    const unsigned char* ak = CAT && kt >= kmid ? abase2 : abase;
#pragma unroll
    for (int i = h * A1_LPW; i < (h + 1) * A1_LPW; ++i) {
      unsigned char* sa = smem + stage * STAGE + a_block(i) * RB;
      if constexpr (OFF32) {
        buffer_to_lds16(ak, sa, aoff[i], static_cast<uint32_t>(kt) * RB);
      } else {
        __builtin_amdgcn_global_load_lds(SCMOE_GLB_PTR(aptr[i] + static_cast<int64_t>(kt) * RB),
                                         SCMOE_LDS_PTR(sa), 16, 0, 0);
      }
    }
  };
  auto issue_w = [&](int kt, int stage) {
    if (ROTK && (kt += rot) >= nk) kt -= nk;
    unsigned char* sb = smem + stage * STAGE + A_BYTES + wave * CFG::B_PER_WAVE * 1024;
    const unsigned char* wk = (CAT && kt >= kmid ? wbase2 : wbase) + static_cast<int64_t>(kt) * RB;
    if constexpr (OFF32) asm volatile("" : "+s"(wk));           // the scalar sum stays scalar
#pragma unroll
    for (int i = 0; i < CFG::B_PER_WAVE; ++i) {
      if constexpr (OFF32) {
        asm volatile("" : "+v"(boff[i]));   // keeps the offset a 32-bit register of its own
        __builtin_amdgcn_global_load_lds(SCMOE_GLB_PTR(wk + boff[i]), SCMOE_LDS_PTR(sb + i * 1024), 16, 0, 0);
      } else {
        __builtin_amdgcn_global_load_lds(SCMOE_GLB_PTR(bptr[i] + static_cast<int64_t>(kt) * RB),
                                         SCMOE_LDS_PTR(sb + i * 1024), 16, 0, 0);
      }
    }
  };
  auto issue_wa0 = [&](int kt, int stage) {
    issue_w(kt, stage);
    issue_a(kt, stage, std::integral_constant<int, 0>{});
  };
  auto issue_a1 = [&](int kt, int stage) { issue_a(kt, stage, std::integral_constant<int, 1>{}); };
  auto issue_prologue = [&]() {
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      if (t < nk) {
        issue_wa0(t, t);
        issue_a1(t, t);
      }
    }
  };
  // wait until at most `tiles` of the newest k-tiles are still in flight (loads complete in
  // issue order, LPW loads per k-tile and wave)
  auto wait_vm = [&](auto n_c) {
    constexpr int n = decltype(n_c)::value;
    static_assert(n < 64, "vmcnt field");
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | 0x0F70);
  };
  // ... and `extra` more loads, at most
  auto wait_tiles = [&](int tiles, auto extra_c) {
    constexpr int x = decltype(extra_c)::value;
    if (NS > 3 && tiles >= 3) wait_vm(std::integral_constant<int, 3 * LPW + x < 63 ? 3 * LPW + x : 63>{});
    else if (NS > 2 && tiles >= 2) wait_vm(std::integral_constant<int, 2 * LPW + x < 63 ? 2 * LPW + x : 63>{});
    else if (tiles >= 1) wait_vm(std::integral_constant<int, LPW + x>{});
    else wait_vm(std::integral_constant<int, x>{});
  };

  // ---- fragment reads (the same for every tile) ---------------------------------------------
  // v_mfma_f32_16x16x32_bf16: an operand fragment is 16 rows x 32 k, lane l holding the 8
  // consecutive k of chunk l / 16 of row l % 16.  (Per flop it moves half the accumulator
  // data of the 32x32x16 form; with random operands a register-only loop of it sustains
  // 2.09 PFLOP/s at 2.05 GHz against 1.78 PFLOP/s at 1.78 GHz: the chip is power-limited.)
  // A wave's 128 x 64 tile is 8 x 4 such products per 32 k; it is walked in half-steps of
  // 16 MFMAs: the 4 weight fragments of the 32 k against row-subtiles 0-3, then against 4-7.
  const int wave_m = wave / CFG::WN, wave_n = wave % CFG::WN;
  const int l16 = lane & 15, lq = lane >> 4;
  // LDS byte address of (row l16, chunk lq) for each 32-k step of stage 0, swizzled (the
  // swizzle depends on row % 16 only).  Plain integers on top of an opaque base, so that the
  // address of any (stage, step, subtile) is one loop-invariant register plus an immediate.
  unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>(SCMOE_LDS_PTR(smem)));
  asm volatile("" : "+s"(lds0));
  unsigned xb[KS32], wb[KS32];
#pragma unroll
  for (int ks = 0; ks < KS32; ++ks) {
    const unsigned cs = static_cast<unsigned>(((ks * 4 + lq) ^ swz<CPR>(l16)) << 4);
    xb[ks] = lds0 + (wave_m * CFG::TM + l16) * RB + cs;
    wb[ks] = lds0 + A_BYTES + (wave_n * CFG::TN + l16) * RB + cs;
  }
  typedef const __attribute__((address_space(3))) bf16x8_t* lds_frag_ptr;

  f32x4_t acc[MI][NJ];          // MI = 8 row-subtiles, NJ = 4 column-subtiles of 16
  bf16x8_t wf[2][NJ];           // weight fragments of a 32-k step, double-buffered: step q of stage R
                                // uses buffer (R * KS32 + q) % 2, consecutive steps alternate
  bf16x8_t xf[2][MI / 2];       // activation fragments of a half-step, one buffer per half
  static_assert((NS * KS32) % 2 == 0, "the weight-fragment buffers alternate over the unrolled k loop");
  // Half-step hs of a k-tile multiplies the weight fragments of 32-k step hs % KS32 with the
  // activation fragments of that step of row-subtile half hs / KS32.  Reads for half-step hs of
  // stage R, in the order of first use:
  auto load_frags = [&](int R, int hs) {
    const int ks = hs % KS32, half = hs / KS32, st = R * STAGE, wbuf = (R * KS32 + ks) & 1, xbuf = hs & 1;
    if (half == 0) {
#pragma unroll
      for (int t = 0; t < (MI / 2 > NJ ? MI / 2 : NJ); ++t) {
        if (t < NJ) wf[wbuf][t] = *reinterpret_cast<lds_frag_ptr>(static_cast<uintptr_t>(wb[ks] + st + t * 16 * RB));
        if (t < MI / 2) xf[xbuf][t] = *reinterpret_cast<lds_frag_ptr>(static_cast<uintptr_t>(xb[ks] + st + t * 16 * RB));
      }
    } else {
#pragma unroll
      for (int t = 0; t < MI / 2; ++t)
        xf[xbuf][t] = *reinterpret_cast<lds_frag_ptr>(static_cast<uintptr_t>(xb[ks] + st + (MI / 2 + t) * 16 * RB));
    }
  };
  auto mfma_step = [&](int R, int hs) {
    const int ks = hs % KS32, half = hs / KS32, wbuf = (R * KS32 + ks) & 1, xbuf = hs & 1;
#pragma unroll
    for (int i = 0; i < MI / 2; ++i)
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj) {
        // there and back: only one operand changes from one instruction to the next, which the power limit
        // turns into clock (layer of 32768 tokens, d = 2048, F = 8192, E = 16 3786 -> 3752 us; 16384, d = 1024,
        // E = 8 563.5 -> 558.4)
        const int j = (i & 1) ? NJ - 1 - jj : jj;
        acc[half * (MI / 2) + i][j] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[wbuf][j], xf[xbuf][i], acc[half * (MI / 2) + i][j], 0, 0, 0);
      }
  };
  // issue order of one half-step: MFMA, ds_read, MFMA, ds_read, ... (the reads feed the NEXT one)
  auto interleave = [&](auto next_hs_c) {
    constexpr int reads = (decltype(next_hs_c)::value / KS32) ? MI / 2 : MI / 2 + NJ;
#pragma unroll
    for (int q = 0; q < reads; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, (MI / 2) * NJ - reads, 0);
  };

  int e, row0, row_end, n0, part;
  auto setup = [&](int item) {
    int l;
    sched.item(item, l, part);
    sched.locate(l, e, row0, row_end, n0);
    int kb;
    sched.k_range(e, part, nk_all, kb, nk, kmid);
    if (ROTK) rot = p.rotk ? static_cast<int>(static_cast<unsigned>(n0 / BN) * p.rotk % static_cast<unsigned>(nk)) : 0;
    set_ptrs(e, row0, row_end, n0, kb);
  };
  if (it < sched.ngemm) {
  setup(it);
  issue_prologue();
  // The arrival counters of the second GEMM's cut tiles (nothing is cut in this launch; workgroup 0 has a tile if
  // any has).  Here and not at the kernel's start, where the argument's load alone held every workgroup up: layer
  // of 8192 tokens, d = 384, F = 1536, E = 8 94.9 us, so 93.8.
  if (ACT && p.splitk_zero != nullptr && blockIdx.x == 0)
    for (int i = tid; i < SPLITK_PARTS; i += CFG::THREADS) p.splitk_zero[i] = 0;
  for (;;) {
    // The accumulators start from the bias (lane: columns 16 j + 4 lq ... of its column block;
    // for a split-K item only in part 0).  Loading it here and not in the epilogue matters:
    // a load in the epilogue would wait behind the next tile's first k-tiles, which are
    // requested before the epilogue and complete in issue order.
    // CAT: what the change of operands needs (the factors of the wave tile's rows, the shared
    // expert's bias) waits in the wave's epilogue patch, where it takes no registers.
    float* const mid_lds = reinterpret_cast<float*>(smem + NS * STAGE + wave * CFG::STG_BYTES);
    if constexpr (CAT) {
      asm volatile("" ::: "memory");      // (the patch was read as another type)
      if (kmid > 0) {
#pragma unroll
        for (int q = 0; q < CFG::TM / 64; ++q) {
          int r = row0 + wave_m * CFG::TM + q * 64 + lane;
          if (r > row_end - 1) r = row_end - 1;
          mid_lds[q * 64 + lane] = p.row_scale[r];
        }
        const int n = n0 + wave_n * CFG::TN + lane;
        mid_lds[CFG::TM + lane] = (p.bias2 != nullptr && n < p.N) ? p.bias2[n] : 0.0f;
      }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = n0 + wave_n * CFG::TN + j * 16 + 4 * lq;
      f32x4_t b = {0.0f, 0.0f, 0.0f, 0.0f};
      if constexpr (CAT) {
        const float* bias = kmid > 0 ? (p.bias ? p.bias + static_cast<int64_t>(e) * p.N : nullptr) : p.bias2;
        if (bias != nullptr && part <= 0 && n < p.N) b = *reinterpret_cast<const f32x4_t*>(bias + n);
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[i][j] = b;
        continue;
      }
      const bool xseg = XSEG && e == p.E;
      const float* bias = xseg ? p.xbias : p.bias + static_cast<int64_t>(e) * p.N;
      if ((xseg ? p.xbias : p.bias) != nullptr && part <= 0 && n < p.N)
        b = *reinterpret_cast<const f32x4_t*>(bias + n);
#pragma unroll
      for (int i = 0; i < MI; ++i) acc[i][j] = b;
    }

    // ---- main loop ---------------------------------------------------------------------------
    // LDS -> registers runs one half-step ahead, each ds_read slotted behind an MFMA.  After an epilogue
    // the stores of the previous tile share the counter with the loads, so everything is
    // waited for (the prologue loads had the whole epilogue to land).
    wait_vm(std::integral_constant<int, 0>{});
    lds_barrier();
    load_frags(0, 0);   // (stage 0, half-step 0)
    // One k-tile with its LDS stage known at compile time (the k loop is unrolled NS-fold),
    // so every LDS address is a loop-invariant register plus an immediate and no address
    // arithmetic has to share registers with fragments that are still in flight.
    // Two barriers per k-tile.  When half-step KS32 - 1 begins, this wave holds every weight
    // fragment of the k-tile and every activation fragment of the first row half in registers;
    // behind the first barrier that is so for all waves, and W and the first halves of the rows
    // (3/4 of the stage) are refilled with k-tile kt + NS while the second half is still being
    // multiplied.  The second barrier, ahead of the last half-step, does the same for the second
    // halves.  So a copy has NS - 1/2 k-tiles to arrive in, and a wait never drains the queue:
    // LPW (NS - 1) newer copies stay in flight.  (One group per k-tile, one k-tile of look-ahead and
    // a drained queue before: layer 3.69 -> 3.61 ms at 32768 tokens, d = 2048, F = 8192, E = 16; 0.579
    // -> 0.562 at 16384 tokens, d = 1024, F = 4096, E = 8.)
    auto k_tile = [&](auto stage_c, auto steady_c, int kt) {
      constexpr int stage = decltype(stage_c)::value;
      constexpr bool steady = decltype(steady_c)::value;   // k-tiles kt+1 .. kt+NS all exist
      constexpr int next = (stage + 1 == NS) ? 0 : stage + 1;
      using X0 = std::integral_constant<int, 0>;
      using XA1 = std::integral_constant<int, A1_LPW>;
      static_for<0, HS>([&](auto hs_c) {
        constexpr int hs = decltype(hs_c)::value;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (hs == KS32 - 1) {
          // the second row halves of this k-tile must have landed; in flight may be the k-tiles after it
          if constexpr (steady) wait_tiles(NS - 1, X0{});
          else wait_tiles(nk - 1 - kt < NS - 1 ? nk - 1 - kt : NS - 1, X0{});
          lds_barrier();
          if (steady || kt + NS < nk) issue_wa0(kt + NS, stage);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (hs == HS - 1) {
          if (steady || kt + 1 < nk) {
            // W and the first row halves of k-tile kt + 1 must have landed; in flight may be its
            // second halves and the k-tiles after it, of k-tile kt + NS the first group only
            if (steady || kt + NS < nk) wait_tiles(NS - 1, X0{});
            else wait_tiles(nk - 2 - kt, XA1{});
            lds_barrier();
            if (steady || kt + NS < nk) issue_a1(kt + NS, stage);
            __builtin_amdgcn_sched_barrier(0);
            load_frags(next, 0);
          }
          mfma_step(stage, hs);
          if constexpr (steady) interleave(std::integral_constant<int, 0>{});
        } else {
          load_frags(stage, hs + 1);
          mfma_step(stage, hs);
          interleave(std::integral_constant<int, hs + 1>{});
        }
      });
    };
    using std::integral_constant;
    using std::bool_constant;
    int kt = 0;
    // CAT, all k-tiles of the routed product done: the rows times their gate weights, plus the shared
    // expert's bias (a part of a cut tile may end before that point: then without the bias).
    auto change_operands = [&](bool with_bias) {
      f32x4_t b[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        b[j] = *reinterpret_cast<const f32x4_t*>(mid_lds + CFG::TM + j * 16 + 4 * lq);
        if (!with_bias) b[j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
      }
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const float f = mid_lds[i * 16 + l16];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[i][j][q] = fmaf(acc[i][j][q], f, b[j][q]);
      }
    };
    for (; kt + 2 * NS <= nk; kt += NS) {       // steady state: every load and read exists
      if constexpr (CAT) {
        if (kt == kmid && kt > 0) change_operands(true);
      }
      k_tile(integral_constant<int, 0>{}, bool_constant<true>{}, kt);
      k_tile(integral_constant<int, 1>{}, bool_constant<true>{}, kt + 1);
      if constexpr (NS > 2) k_tile(integral_constant<int, 2>{}, bool_constant<true>{}, kt + 2);
      if constexpr (NS > 3) k_tile(integral_constant<int, 3>{}, bool_constant<true>{}, kt + 3);
    }
    for (; kt < nk; kt += NS) {                 // the last k-tiles (fewer than 2 NS), guarded
      if constexpr (CAT) {
        if (kt == kmid && kt > 0) change_operands(true);
      }
      k_tile(integral_constant<int, 0>{}, bool_constant<false>{}, kt);
      if (kt + 1 < nk) k_tile(integral_constant<int, 1>{}, bool_constant<false>{}, kt + 1);
      if constexpr (NS > 2) {
        if (kt + 2 < nk) k_tile(integral_constant<int, 2>{}, bool_constant<false>{}, kt + 2);
      }
      if constexpr (NS > 3) {
        if (kt + 3 < nk) k_tile(integral_constant<int, 3>{}, bool_constant<false>{}, kt + 3);
      }
    }

    if constexpr (CAT) {
      if (kmid >= nk) change_operands(kmid == nk);
    }

    // ---- next tile: its first k-tiles are requested before this tile's epilogue -----------
    const int itn = sched.next(it);
    const bool more = itn < sched.ngemm;
    const int crow0 = row0, crow_end = row_end, cn0 = n0, cpart = part, cw = it;   // (a part is item cw < npart)
    unsigned char* const cC = (XSEG && e == p.E) ? p.xC : p.C;        // output of the current tile's segment
    const int64_t cldc = (XSEG && e == p.E) ? p.xldc : p.ldc;
    lds_barrier();                    // every wave holds its last fragments: LDS is free
    // Fused output decode: everything the epilogue needs from memory is requested here, ahead
    // of the next tile's first k-tiles (loads complete in issue order, and the epilogue has
    // nothing to overlap a round trip with): the token of each of the wave's 128 packed rows
    // (lane l: rows l and 64 + l; other lanes get them by a lane permute), their gate
    // weights, and the 16-byte pieces of the first slab's output rows that this lane will
    // add to (each slab then requests the next one's before it does its own work).
    constexpr int SLABS = MI / 2, PIECES = 32 / 8;     // 32-row slabs; a store instruction covers 8 rows
    int dtok[2] = {0, 0};
    float dscale[2] = {1.0f, 1.0f};
    uint4 dadd[PIECES];
    auto addend_loads = [&](int i) {                   // slab i's pieces of the rows to add to
      const int n = cn0 + wave_n * CFG::TN + (lane & 7) * 8;
#pragma unroll
      for (int g = 0; g < PIECES; ++g) {
        const int tok = __shfl(dtok[i >> 1], (i & 1) * 32 + g * 8 + (lane >> 3));
        dadd[g] = make_uint4(0u, 0u, 0u, 0u);
        if (n < p.N && p.addend != nullptr)
          dadd[g] = *reinterpret_cast<const uint4*>(p.addend + (static_cast<int64_t>(tok) * p.ldadd + n) * 2);
      }
    };
    auto decode_loads = [&]() {
      if constexpr (DECODE) {
#pragma unroll
        for (int q = 0; q < CFG::TM / 64; ++q) {
          int r = crow0 + wave_m * CFG::TM + q * 64 + lane;
          if (r > crow_end - 1) r = crow_end - 1;      // rows past the segment: its last row (never stored)
          dtok[q] = (DEC == 2) ? r : p.scatter[r];
        }
#pragma unroll
        for (int q = 0; q < CFG::TM / 64; ++q) {
          if (DEC == 1) dscale[q] = p.row_scale[dtok[q]];
          else if (DEC == 2) dscale[q] = p.row_scale ? p.row_scale[2 * static_cast<int64_t>(dtok[q])] : 1.0f;
        }
        if constexpr (ADD) addend_loads(0);
      }
    };
    constexpr bool dec = DECODE;
    if (dec && cpart < 0) decode_loads();
    if (more) {
      setup(itn);
      issue_prologue();
    }

    // ---- split-K items: leave the partial sums in scratch and count the part in; the finish
    // items at the end of the launch add the parts up.  The partial sums and the counter move
    // with relaxed device-scope accesses (sc1: past the caches that are not shared by the whole
    // device), ordered by a plain wait for the stores; device-scope fences would write back and
    // invalidate the whole L2 of the XCD on every use, which costs more than the split saves.
    const bool finish = cpart < 0;
    if (cpart >= 0) {
      constexpr int TILE = BM * BN;
      constexpr int FRAGS = MI * NJ;                                  // 16-byte pieces (accumulators) per lane
      const size_t slot0 = static_cast<size_t>(sched.xcd) * nslots;   // this XCD's scratch slots
      // accumulator (i, j) of wave w and lane l sits at float4 index (w * FRAGS + i * NJ + j) * 64 + l
      float* mine = p.splitk_part + (slot0 + cw) * TILE + ((wave * FRAGS) * 64 + lane) * 4;
      mfma_results_settle();
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) store16_device_scope(mine + ((i * NJ + j) * 64) * 4, acc[i][j]);
      wait_vm(std::integral_constant<int, 0>{});                      // this wave's stores have been performed
      lds_barrier();                                                  // ... and every wave's
      if (tid == 0)
        __hip_atomic_fetch_add(p.splitk_count + slot0 + cw / sched.S, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // ---- epilogue: activation, bf16; rows re-assembled in LDS, 16-byte stores ----------------
    // acc[i][j][v] is output row (lane % 16) of row-subtile i and column 4 * (lane / 16) + v of
    // column-subtile j.  A wave stages 32-row slabs (two row-subtiles) of its tile in its
    // private LDS patch and writes them out with TN/8 lanes per row, so that every store
    // instruction covers whole 128-byte lines.
    unsigned char* stg = smem + NS * STAGE + wave * CFG::STG_BYTES;
#pragma unroll
    for (int i = 0; i < MI / 2; ++i) {
      const int mbase = crow0 + wave_m * CFG::TM + i * 32;
      if (!finish || mbase >= crow_end) continue;   // wave-uniform: not the last part / slab past the segment
      float rscale[2] = {1.0f, 1.0f};             // fused decode: the gate weights of this lane's two rows
      uint4 add_cur[PIECES];
      if (dec) {
#pragma unroll
        for (int u = 0; u < 2; ++u) rscale[u] = __shfl(dscale[i >> 1], (i & 1) * 32 + u * 16 + l16);
        if constexpr (ADD) {
#pragma unroll
          for (int g = 0; g < PIECES; ++g) add_cur[g] = dadd[g];
          if (i + 1 < SLABS) addend_loads(i + 1);
        }
      }
#pragma unroll
      for (int h = 0; h < 32 / CFG::STG_ROWS; ++h) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int sr = u * 16 + l16 - h * CFG::STG_ROWS;   // this lane's row inside the staged rows
          const bool mine = sr >= 0 && sr < CFG::STG_ROWS;
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = acc[2 * i + u][j][q];
            if (ACT) {
#pragma unroll
              for (int q = 0; q < 4; ++q)
                v[q] = (p.gelu_mode == SCMOE_GELU_TANH) ? gelu_tanh_fast(v[q]) : gelu_erf_fast(v[q]);
            }
            if (dec && !CAT) {
#pragma unroll
              for (int q = 0; q < 4; ++q) v[q] *= rscale[u];
            }
            uint2 o;
            o.x = cvt_pk_bf16(v[0], v[1]);
            o.y = cvt_pk_bf16(v[2], v[3]);
            // columns 16 j + 4 lq ...: 16-byte chunk 2j + lq/2 of the row (swizzled like the
            // operand tiles), half lq % 2 of it
            if (mine)
              *reinterpret_cast<uint2*>(stg + sr * CFG::STG_ROW + (((2 * j + (lq >> 1)) ^ swz<8>(sr)) << 4) + (lq & 1) * 8) = o;
          }
        }
#pragma unroll
        for (int r0 = 0; r0 < CFG::STG_ROWS; r0 += 8) {
          const int r = r0 + (lane >> 3);       // 8 lanes of 16 bytes per 128-byte row
          const int c = lane & 7;
          uint4 o = *reinterpret_cast<const uint4*>(stg + r * CFG::STG_ROW + ((c ^ swz<8>(r)) << 4));
          const int m = mbase + h * CFG::STG_ROWS + r;
          const int n = cn0 + wave_n * CFG::TN + c * 8;
          const int g = (h * CFG::STG_ROWS + r0) / 8;          // which of the slab's 8-row pieces
          int64_t orow = m;
          if (dec) orow = __shfl(dtok[i >> 1], (i & 1) * 32 + g * 8 + (lane >> 3));   // (all lanes take part)
          if (m < crow_end && n < p.N) {
            if constexpr (ADD) {
              // output decode: this packed row belongs to token orow; add the row already there
              const uint4 a = add_cur[g];
              o.x = add_bf16x2(o.x, a.x);
              o.y = add_bf16x2(o.y, a.y);
              o.z = add_bf16x2(o.z, a.z);
              o.w = add_bf16x2(o.w, a.w);
            }
            if (p.stream_out) {
              // an output far larger than the caches: stored with the streaming hint, so that it
              // does not push the operand panels out of the L2
              typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
              const u32x4_t ov = {o.x, o.y, o.z, o.w};
              __builtin_nontemporal_store(ov, reinterpret_cast<u32x4_t*>(cC + (orow * cldc + n) * 2));
            } else {
              *reinterpret_cast<uint4*>(cC + (orow * cldc + n) * 2) = o;
            }
          }
        }
      }
    }
    it = itn;
    if (!more) break;
  }
  }

  // ---- finish items: one per wave tile of a tile that was cut along K ------------------------
  // The parts are added up in part order (the result does not depend on who arrived when) by a
  // workgroup that has nothing else left to do: each of its waves takes MI / WAVES row-subtiles
  // of the wave tile, so the 256 KiB of a tile's partial sums per part are read by all waves of
  // WAVES workgroups at once.  The parts were counted in long ago (they are the first items of
  // their workgroups, which have lower ids and started earlier); the count is checked anyway,
  // with a bounded wait, so that no wave can be left waiting for good.
  for (; it < sched.ngemm + sched.nfin; it += nslots) {
    constexpr int TILE = BM * BN, FRAGS = MI * NJ, FS = CFG::WAVES, RPW = MI > CFG::WAVES ? MI / CFG::WAVES : 1;
    static_assert((MI % CFG::WAVES == 0 || MI < CFG::WAVES) && NJ == 4, "row-subtiles of a wave tile are shared out among the waves");
    const int f = it - sched.ngemm;
    const int lt = f / FS, region = f - lt * FS;                      // cut tile (0 .. rem-1), wave tile of it
    const int S = sched.S;
    const size_t slot0 = static_cast<size_t>(sched.xcd) * nslots;
    int* cnt = p.splitk_count + slot0 + lt;
    int fe, frow0, frow_end, fn0;
    sched.locate(sched.full + lt, fe, frow0, frow_end, fn0);
    if (tid == 0) {
      for (int spin = 0; spin < (1 << 22); ++spin) {
        if ((__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xff) >= S) break;
        __builtin_amdgcn_s_sleep(16);
      }
    }
    lds_barrier();
    const bool xseg = XSEG && fe == p.E;
    unsigned char* const fC = xseg ? p.xC : p.C;
    const int64_t fldc = xseg ? p.xldc : p.ldc;
    const int rm = region / CFG::WN, rn = region - rm * CFG::WN;      // the wave tile's place in the tile
    const float* first = p.splitk_part + (slot0 + static_cast<size_t>(lt) * S) * TILE;
#pragma unroll
    for (int u = 0; u < RPW; ++u) {
      const int i = wave * RPW + u;                                   // row-subtile of the wave tile
      if (MI < CFG::WAVES && i >= MI) continue;                       // (wave-uniform) more waves than subtiles
      const int m = frow0 + rm * CFG::TM + i * 16 + l16;              // this lane's row
      if (frow0 + rm * CFG::TM + i * 16 >= frow_end) continue;        // (wave-uniform) subtile past the segment
      const int mc = m < frow_end ? m : frow_end - 1;
      // what the output decode needs of this row
      int64_t orow = mc;
      float rscale = 1.0f;
      if constexpr (DEC == 1) {
        orow = p.scatter[mc];
        rscale = p.row_scale[orow];
      } else if constexpr (CAT) {
        orow = p.scatter[mc];
      } else if constexpr (DEC == 2) {
        if (p.row_scale != nullptr) rscale = p.row_scale[2 * static_cast<int64_t>(mc)];
      }
      f32x4_t a[NJ];
      const float* src = first + ((region * FRAGS + i * NJ) * 64 + lane) * 4;
      for (int q0 = 0; q0 < S; q0 += 4) {           // four parts per round trip (parts past S - 1: S - 1 again, not added)
        f32x4_t t[16];
        const float* pq[4];
#pragma unroll
        for (int u4 = 0; u4 < 4; ++u4) pq[u4] = src + static_cast<size_t>(q0 + u4 < S ? q0 + u4 : S - 1) * TILE;
        load16x16_device_scope(pq[0], pq[1], pq[2], pq[3], t);
#pragma unroll
        for (int u4 = 0; u4 < 4; ++u4) {
          if (q0 + u4 < S) {                         // (wave-uniform)
#pragma unroll
            for (int j = 0; j < NJ; ++j) a[j] = (q0 + u4 == 0) ? t[u4 * NJ + j] : a[j] + t[u4 * NJ + j];
          }
        }
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int n = fn0 + rn * CFG::TN + j * 16 + 4 * lq;           // four consecutive columns
        float v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          v[c] = a[j][c];
          if (ACT) v[c] = (p.gelu_mode == SCMOE_GELU_TANH) ? gelu_tanh_fast(v[c]) : gelu_erf_fast(v[c]);
          if (DECODE && !CAT) v[c] *= rscale;
        }
        uint2 o;
        o.x = cvt_pk_bf16(v[0], v[1]);
        o.y = cvt_pk_bf16(v[2], v[3]);
        if (m < frow_end && n < p.N) {
          if constexpr (ADD) {
            if (p.addend != nullptr) {
              const uint2 ad = *reinterpret_cast<const uint2*>(p.addend + (orow * p.ldadd + n) * 2);
              o.x = add_bf16x2(o.x, ad.x);
              o.y = add_bf16x2(o.y, ad.y);
            }
          }
          *reinterpret_cast<uint2*>(fC + (orow * fldc + n) * 2) = o;
        }
      }
    }
    // the last of a tile's finish items leaves the counter at zero for the next launch
    lds_barrier();
    if (tid == 0) {
      const int old = __hip_atomic_fetch_add(cnt, 0x100, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((old >> 8) == FS - 1) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ---- host side --------------------------------------------------------------------------------

using CfgA = TileCfg<256, 256, 64, 2, 4, 2>;   // 8 waves, 128 KiB LDS, one workgroup per CU
using CfgB = TileCfg<256, 256, 32, 2, 4, 4>;   // 8 waves, 4 stages, 128 KiB LDS
using CfgT = TileCfg<128, 128, 64, 2, 2, 3>;   // 4 waves of 64 x 64, 104 KiB LDS, one workgroup per CU: fewer 128 x 128 tiles than CUs
using CfgV = TileCfg<256, 128, 64, 4, 2, 3>;   // 8 waves of 64 x 64, 160 KiB LDS, one workgroup per CU: second GEMMs of one round of such tiles, of most of a second, or with a long K
using CfgS = TileCfg<64, 128, 64, 1, 2, 3>;    // 2 waves of 64 x 64, 76 KiB LDS, two workgroups per CU: second GEMMs of up to 64 rows per segment
using CfgU = TileCfg<128, 128, 64, 2, 2, 2>;   // 4 waves of 64 x 64, 72 KiB LDS, two workgroups per CU: few rows per expert, small problems

// Tile configuration in use: 0 unless scmoe_set_gemm_variant has set another.  The one
// process-wide setting of the library: an atomic, read once per launch.
static std::atomic<int> g_variant{0};
constexpr int NUM_VARIANTS = 4;

static int gemm_variant() { return g_variant.load(std::memory_order_relaxed); }

int set_gemm_variant(int v) {
  if (v < 0 || v >= NUM_VARIANTS) return SCMOE_ERR_ARG;
  g_variant.store(v, std::memory_order_relaxed);
  return SCMOE_OK;
}

bool ffn_mfma_supported(int d, int F) { return d > 0 && F > 0 && (d % 64) == 0 && (F % 64) == 0; }

// which output decode a launch asks for (see gemm_bf16_kernel)
static int decode_kind(const GemmArgs& a) {
  return a.A2 != nullptr ? (a.addend != nullptr ? 4 : 3) : a.scatter != nullptr ? 1 : (a.row_scale != nullptr || a.addend != nullptr) ? 2 : 0;
}

template <class CFG, bool ACT, bool OFF32, int DEC, bool XSEG>
static int launch_gemm_impl(GemmArgs a, int max_rows, hipStream_t stream) {
  // the dynamic-LDS limit is a per-device attribute of the kernel: raise it once per device
  static std::atomic<bool> attr_set[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = -1;
  if (dev < 0 || !attr_set[dev].load(std::memory_order_acquire)) {
    hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_kernel<CFG, ACT, OFF32, DEC, XSEG>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, CFG::LDS_BYTES);
    if (err != hipSuccess) return hip_fail(err);
    if (dev >= 0) attr_set[dev].store(true, std::memory_order_release);
  }
  // only a second GEMM decodes, and not together with the dense extra segment
  if ((ACT && (a.scatter != nullptr || a.addend != nullptr)) || (!XSEG && a.xrows != 0)) return SCMOE_ERR_ARG;
  if (DEC != decode_kind(a) || (DEC != 0 && DEC != 2 && (a.scatter == nullptr || a.row_scale == nullptr))) return SCMOE_ERR_ARG;
  if (DEC >= 3 && (a.W2 == nullptr || a.Kd % (2 * CFG::BK) != 0)) return SCMOE_ERR_ARG;
  // upper bound on row tiles: sum_e ceil(c_e / BM) <= max_rows / BM + E
  const int mtb = max_rows / CFG::BM + a.E + (a.xrows + CFG::BM - 1) / CFG::BM;
  a.nt = (a.N + CFG::BN - 1) / CFG::BN;
  // Large outputs are streamed past the caches (measured: -0.6 to -1 % layer time at the large and
  // medium workloads).  The hidden rows of a first GEMM are read back by the second one right
  // away: below 256 MiB (the size of the memory-side cache) they are left to the caches (the
  // small workload loses 4 % otherwise); a second GEMM's rows are final and stream from 64 MiB on.
  a.stream_out = (static_cast<int64_t>(max_rows) + a.xrows) * a.N * 2 >= (int64_t(ACT ? 256 : 64) << 20);
  int slots = (mtb * a.nt + 7) / 8;                            // tiles per XCD, upper bound
  const int resident = (num_cus() / 8) * CFG::WG_PER_CU;       // workgroups one XCD holds at once
  if (slots > resident) {
    slots = resident;
  } else if (a.splitk_part != nullptr && a.Kd >= SPLITK_MIN_K) {
    // Far fewer tiles than workgroups the chip can hold: launch the workgroups anyway, so
    // that the schedule cuts every tile along K (as many slots as the split-K scratch has room
    // for).  From a quarter of the capacity on it no longer pays (measured: tiles cut in two
    // cost the small workload 6 %).
    const int room = SPLITK_PARTS / 8;
    const int want = resident < room ? resident : room;
    if (want >= 4 * slots) slots = want;
  }
  // the split-K scratch is laid out for 8 * slots partial tiles of this shape
  if (8 * slots > SPLITK_PARTS ||
      static_cast<size_t>(8) * slots * CFG::BM * CFG::BN * 4 > SPLITK_WS_BYTES - SPLITK_COUNT_BYTES) {
    a.splitk_part = nullptr;
    a.splitk_count = nullptr;
  }
  hipLaunchKernelGGL((gemm_bf16_kernel<CFG, ACT, OFF32, DEC, XSEG>), dim3(8 * slots), dim3(CFG::THREADS), CFG::LDS_BYTES,
                     stream, a);
  return launch_status();
}

// a_rows: rows of the activation matrix that can be addressed (through `gather` any of them).
template <class CFG, bool ACT>
static int launch_gemm(const GemmArgs& a, int max_rows, int64_t a_rows, hipStream_t stream) {
  const int64_t lim = BUFFER_SPAN;
  const bool off32 = a.Kd < BUFFER_K && a_rows * a.lda * 2 < lim && static_cast<int64_t>(a.N) * a.ldw * 2 < lim &&
                     static_cast<int64_t>(a.xrows) * a.xlda * 2 < lim && static_cast<int64_t>(a.N) * a.xldw * 2 < lim;
  if constexpr (ACT) {
    return off32 ? launch_gemm_impl<CFG, true, true, 0, true>(a, max_rows, stream)
                 : launch_gemm_impl<CFG, true, false, 0, true>(a, max_rows, stream);
  } else {
    if (a.xrows > 0)
      return off32 ? launch_gemm_impl<CFG, false, true, 0, true>(a, max_rows, stream)
                   : launch_gemm_impl<CFG, false, false, 0, true>(a, max_rows, stream);
    switch (decode_kind(a)) {
      case 1:
        return off32 ? launch_gemm_impl<CFG, false, true, 1, false>(a, max_rows, stream)
                     : launch_gemm_impl<CFG, false, false, 1, false>(a, max_rows, stream);
      case 2:
        return off32 ? launch_gemm_impl<CFG, false, true, 2, false>(a, max_rows, stream)
                     : launch_gemm_impl<CFG, false, false, 2, false>(a, max_rows, stream);
      case 3:
      case 4: return SCMOE_ERR_ARG;        // (launch_joint_second)
      default:
        return off32 ? launch_gemm_impl<CFG, false, true, 0, false>(a, max_rows, stream)
                     : launch_gemm_impl<CFG, false, false, 0, false>(a, max_rows, stream);
    }
  }
}

// Row tiles of that height of the segments of so many rows in all: as many as there are segments where those average less
// than 7/8 of one.
static int64_t row_tiles(int64_t rows, int64_t E, int edge) { return 8 * rows <= 7 * edge * E ? E : rows / edge + E / 2; }

// ... of a balanced load: with its mean half a standard deviation higher in every segment.
static int64_t balanced_row_tiles(int64_t rows, int64_t E, int edge) {
  const double mean = static_cast<double>(rows) / E;
  return E * static_cast<int64_t>(ceil((mean + 0.5 * sqrt(mean)) / edge));
}

// ... and from above, where the load is balanced or is not.
static int64_t most_row_tiles(int64_t rows, int64_t E, int edge) {
  return E == 1 ? (rows + edge - 1) / edge : std::max(row_tiles(rows, E, edge), balanced_row_tiles(rows, E, edge));
}

// Whether a launch takes the 256 x 256 tiles (variant 0): a first GEMM or not, no other chain beside it, rows in E segments
// and in the extra one.
static bool takes_large_tiles(bool first, bool alone, int64_t max_rows, int64_t E, int64_t xrows, int64_t N) {
  const int64_t segs = E + (xrows > 0 ? 1 : 0), rows = max_rows + xrows, cus = num_cus();
  const int64_t nt = (N + CfgA::BN - 1) / CfgA::BN, extra = (xrows + CfgA::BM - 1) / CfgA::BM;
  // At N <= 128 half of a 256-column tile would be padding (layer call, us, large tiles / two
  // workgroups of 128 x 128: 32000 tokens, d = 64, F = 128, E = 8 50.7 / 39.5, E = 32 79 / 68; top-2 of
  // 16 experts, d = 128, F = 1024 161 / 148).
  // A first GEMM whose large tiles leave the second of two rounds partly empty, at up to 320 rows a segment: a
  // segment's last 256-row tile is mostly padding, and smaller tiles fill the last round.  From more than one round to
  // 1.6, and up to two where segments just exceed a tile and pay for another one (layer us, large / small tiles, rounds:
  // 4000, d = 640, F = 1728, E = 24 116.7 / 107.3 (1.1); 1302 x 4 rows, d = 512, F = 2048, E = 32 129.1 / 120.7 (1.2); 2500, d = 768,
  // F = 3072, E = 16 143.5 / 134.9 (1.2); 4096 x 2, E = 32, d = 1024, F = 2048 179.8 / 175.0 and 4096, E = 16, F = 4096 173.1 / 167.8
  // (1.5); 2000 x 4, d = 512, F = 2048, E = 32, 250 rows a segment 137.6 / 135.4 (1.7); but 2500, d = 2048, F = 2048, E = 16 168.8 /
  // 180.6 (0.8), 1302 x 4, d = 512, F = 1344, E = 32 96.2 / 98.8 (0.9), 2500, d = 1024, F = 4096, E = 16, 156 rows 176.3 / 182.6 (1.6);
  // three rounds, 8192, E = 32, d = 1024, F = 4096 251.9 / 256.1; 400 rows a segment, 6400, E = 16 169.7 / 180.5).
  const int64_t large = (row_tiles(max_rows, E, CfgA::BM) + extra) * nt;
  const bool few_rows = rows <= 128 * segs;
  const bool short_first = first && rows <= 320 * segs && large > cus &&
                           (5 * large <= 8 * cus || (max_rows >= 240 * E && large <= 2 * cus));
  // A first GEMM of expert segments alone whose large tiles fill four fifths of the CUs or more, once, and are 85 % full in rows and
  // columns (layer us, small / large tiles: top-1, 8192 tokens, d = 384, F = 1536, E = 8 62.5 / 58.6; 6000, d = 512, F = 2048 68.6 / 63.7;
  // fewer, at 0.75 of the CUs, top-1, 15212, d = 320, F = 640, E = 8 47 / 53 and 7567, top-2, d = 384, F = 768, E = 8 94 / 98; half a last
  // column tile, 10613, d = 128, F = 320 47 / 52; 78 % full, 5000, E = 12 65.6 / 66.4).  Of 315 drawn calls of two thirds of the CUs,
  // 85 % full in rows, 32 are slower by more than 1.5 %, up to 16 %, of the 116 left three, up to 4 %.
  // Not beside a chain on another stream, which could not share a CU with them (118 / 122).
  const int64_t most = most_row_tiles(max_rows, E, CfgA::BM) * nt;
  if (first && alone && E > 1 && xrows == 0 && !few_rows && N > CfgU::BN && 5 * most >= 4 * cus && most <= cus &&
      20 * max_rows * N >= 17 * CfgA::BM * row_tiles(max_rows, E, CfgA::BM) * CfgA::BN * nt)
    return true;
  return N > CfgU::BN && (max_rows / CfgA::BM + E + extra) * nt >= cus && !(few_rows && first) && !short_first;
}

template <bool ACT>
static int launch_variant(const GemmArgs& a, int max_rows, int64_t a_rows, hipStream_t stream) {
  switch (gemm_variant()) {
    case 1: return launch_gemm<CfgB, ACT>(a, max_rows, a_rows, stream);
    case 2: return launch_gemm<CfgU, ACT>(a, max_rows, a_rows, stream);
    case 3: return launch_gemm<CfgT, ACT>(a, max_rows, a_rows, stream);
    default: break;
  }
  // Variant 0 picks by size.
  const int64_t segs = a.E + (a.xrows > 0 ? 1 : 0), rows = static_cast<int64_t>(max_rows) + a.xrows;
  auto tiles_of = [&](int64_t edge) {     // upper bound on the tiles of that edge
    return (max_rows / edge + a.E + (a.xrows + edge - 1) / edge) * ((a.N + edge - 1) / edge);
  };
  // Segments of 128 rows or fewer on average: the launch is bound by streaming the weights, and
  // 256-row tiles would be mostly padding.  128 x 128 tiles, two workgroups per CU, and the
  // column tiles start their walk over K at different places (rotk): in step, with rows a power
  // of two apart, they would all be at the same few memory channels.  Measured, layer call at
  // d = 2048, F = 8192, E = 16: 500 tokens 0.383 -> 0.331 ms, 1000 tokens 0.451 -> 0.364; at 2000
  // tokens (125 rows per expert) equal to the large tiles, above that those win.  At other widths and
  // expert counts only against the smaller tiles before these: 500 tokens, d = 1024, F = 2048, E = 64
  // 0.216 -> 0.191; 3000, d = 1024, F = 4096, E = 32 0.294 -> 0.257.
  const bool few_rows = rows <= 128 * segs;
  GemmArgs g = a;
  g.rotk = few_rows ? 5 : 0;
  if (takes_large_tiles(ACT, !a.beside, max_rows, a.E, a.xrows, a.N)) return launch_gemm<CfgA, ACT>(g, max_rows, a_rows, stream);
  // A second GEMM of up to 53 rows per expert (above, more and more experts pass 64): half of a 128-row stage would be padding,
  // and three stages of 64 rows keep half as much again of the weights in flight (layer us, d = 2048, F = 8192, E = 16: 500 tokens
  // 294 / 278, 800 tokens 327 / 318; 300, d = 1024, F = 4096 108.6 / 90.4; top-1 without shared expert, 500, d = 1024 92.1 / 90.0; a
  // first GEMM, with its many column tiles, gains nothing: 500 tokens 296 / 297, 800 tokens 327 / 341).  With an expert in each:
  //  * more than 3/8 of a tile per CU (fewer are better off with four waves a workgroup: top-4, 64 tokens, d = 1280, F = 2560,
  //    E = 8 83 / 91; top-1, 126, d = 1472, F = 3904, E = 4 54 / 57), or few enough to be cut along a long K where the 128-row
  //    tiles are not, a quarter of one per CU being their limit (top-4, 43, d = 1600, F = 6400, E = 4 102 / 84; top-1, 181,
  //    d = 1664, F = 4416 77 / 70; with the shared expert 182, d = 1536, F = 6144 100 / 86, but 39, top-4, d = 1472, F = 3904 85 / 87);
  //  * up to one, with two tiles for some experts, or from 5/4 to 2: between, some CUs have a second tile (224 tokens, top-2,
  //    d = 1728, F = 4608, E = 16 150 / 166; skewed, 265, d = 1344, F = 3584 103 / 116; 600, d = 1536, F = 4096, E = 12 124 / 126);
  //  * no other chain's second GEMM beside it (top-3, 99 tokens, d = 1600, F = 6400, E = 8 on two streams 141 / 172).
  // Of 450 drawn calls of up to 64 rows about 220 are taken, four of them slower by more than 1.5 %, at most 7.  The 256-row tiles
  // above come first, whatever the segments: from (rows / 256 + experts) x column tiles of one per CU on (600 tokens, d = 2048, E = 32).
  const int64_t cus = num_cus(), s_nt = (a.N + CfgS::BN - 1) / CfgS::BN, s_segs = a.E + (a.xrows + CfgS::BM - 1) / CfgS::BM;
  const int64_t s_tiles = s_segs * s_nt, s_more = (s_segs + max_rows / (2 * CfgS::BM)) * s_nt, s_most = (s_segs + max_rows / CfgS::BM) * s_nt;
  const bool s_rows = 6 * static_cast<int64_t>(max_rows) <= 5 * CfgS::BM * static_cast<int64_t>(a.E) && rows <= 96 * segs;
  const bool s_fit = 8 * s_tiles > 3 * cus && s_tiles <= 2 * cus && (s_more <= cus || 4 * s_tiles > 5 * cus);
  const bool s_cut = a.splitk_part != nullptr && 2 * a.Kd >= (a.xrows > 0 ? 4 : 3) * SPLITK_MIN_K && 4 * tiles_of(CfgT::BM) > cus && 2 * s_most <= cus;
  if (!ACT && s_rows && (s_fit || s_cut) && !(a.beside && a.scatter == nullptr)) return launch_gemm<CfgS, ACT>(g, max_rows, a_rows, stream);
  // Not even one 128 x 128 tile per CU, and a second GEMM (long K, short epilogue): every
  // workgroup is alone on its CU, and three LDS stages keep more in flight (small workload: 18.4
  // against 27.8 us with two waves and 32-deep k-tiles; 2000 tokens, d = 512: 79.6 against 95.9 us
  // of layer time with two workgroups per CU, whose free slots would cut the tiles along K).
  if (!ACT && tiles_of(CfgT::BM) <= num_cus()) return launch_gemm<CfgT, ACT>(g, max_rows, a_rows, stream);
  // A second GEMM of more rows: 256 x 128 tiles, eight waves of 64 x 64 and three stages, one workgroup per CU: 0.82 us a
  // k-tile of a full chip, where two workgroups of 128 x 128 take 0.7 to 1.0 for the same outputs (kernel us, 128 x 128 /
  // 256 x 128: 3001 tokens, top-2, d = 768, F = 3072, E = 12 60.6 / 51.0; layer us 6000, d = 1024, F = 4096, E = 8 274 / 253; 1500,
  // d = 1536 152 / 131).  Where they were measured to gain (layer or call us in the same order):
  //  * 16 k-tiles and more (below, three stages are hardly filled: 6780, d = 320, F = 640, E = 2 50 / 59);
  //  * more of the smaller tiles than CUs, by a tenth below 44 k-tiles (those have a CU each up to there: 8000, d = 192, E = 16,
  //    skewed 49.9 / 53.2; 17279, d = 192, F = 768, E = 16, skewed 53 / 56; but 1525, top-2, d = 1024, F = 4096, E = 8 159 / 132);
  //  * not with the second round of them partly empty: more than one, counted from above, up to 1.75 (1.06, 16384, d = 512, F = 2048,
  //    E = 8 127.0 / 132.1; 1.5, 10708, d = 768, F = 2048, E = 32 162 / 175; 1.64, skewed, 18538, d = 576, F = 1536, E = 12 200 / 221), or
  //    from 44 k-tiles on, which gain more, by the average up to 1.3 (1.25, 8192, d = 1024, F = 4096, E = 16 216.9 / 220.9; but
  //    1.6, 7007, d = 1792, F = 4800, E = 12 619 / 596; 7522, top-1 without shared expert, d = 896, F = 3584, E = 4 271 / 253), unless
  //    experts fit one of the smaller row tiles: half of the wide ones is padding then (1204, d = 1984, F = 3968, E = 16 196 / 213;
  //    top-2, 1641, d = 1088, F = 4352, E = 32 250 / 271; of 48 such calls the 40 beyond one round lose 3 to 20 %, the eight within gain 3 to 9 %).
  // Of 600 drawn calls that the average alone takes 100 are slower by more than 1.5 %, up to 19 %; of the 300 left 17, up to 6 %.
  const int64_t v_extra = (a.xrows + CfgV::BM - 1) / CfgV::BM, v_nt = (a.N + CfgV::BN - 1) / CfgV::BN;
  const int64_t square = (max_rows / CfgU::BM + (a.xrows + CfgU::BM - 1) / CfgU::BM) * static_cast<int64_t>((a.N + CfgU::BN - 1) / CfgU::BN);
  const int64_t wide = (row_tiles(max_rows, a.E, CfgV::BM) + v_extra) * v_nt, v_most = (most_row_tiles(max_rows, a.E, CfgV::BM) + v_extra) * v_nt;
  const bool v_long = a.Kd >= 44 * CfgV::BK, v_full = 8 * static_cast<int64_t>(max_rows) > 7 * CfgU::BM * static_cast<int64_t>(a.E);
  if (!ACT && !few_rows && a.N > CfgV::BN && a.Kd >= 16 * CfgV::BK && 10 * square >= (v_long ? 10 : 11) * cus &&
      (32 * wide + 4 * a.E * v_nt <= 33 * cus || 10 * wide >= 13 * cus) && ((v_long && v_full) || v_most <= cus || 4 * v_most > 7 * cus))
    return launch_gemm<CfgV, ACT>(g, max_rows, a_rows, stream);
  // Otherwise two workgroups per CU, whose epilogues and waits fall on each other's arithmetic
  // (layer time, us, against two waves and 32-deep k-tiles: 700 tokens, d = 768: 97 -> 90; 1500
  // tokens, top-2, d = 768, E = 16: 86 -> 79; 3000 tokens, d = 1024, E = 32: 278 -> 245).
  return launch_gemm<CfgU, ACT>(g, max_rows, a_rows, stream);
}

// The joint second GEMM of a top-1 layer (GemmArgs::A2), rows: tokens.
static int launch_joint_second(const GemmArgs& a, int rows, hipStream_t stream) {
  return a.addend != nullptr ? launch_gemm_impl<CfgA, false, true, 4, false>(a, rows, stream)
                             : launch_gemm_impl<CfgA, false, true, 3, false>(a, rows, stream);
}

__global__ void zero_ints(int* p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

size_t ffn_mfma_scratch_bytes() { return SPLITK_WS_BYTES; }
int ffn_mfma_counter_ints() { return SPLITK_PARTS; }

// Split-K scratch of a call: arrival counters first (every launch leaves them at zero again),
// then the partial tiles.  Without scratch the last round of tiles is not split.
struct SplitK { float* parts = nullptr; int* counters = nullptr; };
// clear: the counters that the first GEMM's launch has to clear (it cuts no tile itself: d is short), which
// saves a launch of 4.7 us (top-2 of 32 experts, 4096 tokens, d = 1024, F = 2048 in four calls 180 -> 175).
static int prepare_splitk(const FfnArgs& a, SplitK& sk, hipStream_t stream, int** clear = nullptr) {
  if (clear != nullptr) *clear = nullptr;
  if (a.scratch == nullptr || a.scratch_bytes < SPLITK_WS_BYTES) return SCMOE_OK;
  if (a.d < SPLITK_MIN_K && a.F < SPLITK_MIN_K) return SCMOE_OK;      // no product long enough to be cut
  sk.counters = static_cast<int*>(a.scratch);
  sk.parts = reinterpret_cast<float*>(static_cast<unsigned char*>(a.scratch) + SPLITK_COUNT_BYTES);
  if (a.scratch_zeroed) return SCMOE_OK;
  if (clear != nullptr && a.d < SPLITK_MIN_K) {
    *clear = sk.counters;
    return SCMOE_OK;
  }
  hipLaunchKernelGGL(zero_ints, dim3(1), dim3(256), 0, stream, sk.counters, SPLITK_PARTS);
  return launch_status();
}

// hidden = act(x . W1^T + b1)
static GemmArgs first_gemm(const FfnArgs& a, const SplitK& sk) {
  GemmArgs g{};
  g.A = static_cast<const unsigned char*>(a.x);
  g.lda = a.ldx;
  g.gather = a.gather;
  g.offsets = a.offsets;
  g.W = static_cast<const unsigned char*>(a.W1);
  g.ldw = a.ldw1;
  g.bias = a.b1;
  g.C = static_cast<unsigned char*>(a.hidden);
  g.ldc = a.ldh;
  g.E = a.E;
  g.N = a.F;
  g.Kd = a.d;
  g.gelu_mode = a.gelu_mode;
  g.beside = a.beside;
  g.splitk_part = sk.parts;
  g.splitk_count = sk.counters;
  return g;
}

// y = hidden . W2^T + b2, optionally decoded on store
static GemmArgs second_gemm(const FfnArgs& a, const SplitK& sk) {
  GemmArgs g{};
  g.A = static_cast<const unsigned char*>(a.hidden);
  g.lda = a.ldh;
  g.gather = nullptr;
  g.offsets = a.offsets;
  g.W = static_cast<const unsigned char*>(a.W2);
  g.ldw = a.ldw2;
  g.bias = a.b2;
  g.C = static_cast<unsigned char*>(a.y);
  g.ldc = a.ldy;
  g.E = a.E;
  g.N = a.d;
  g.Kd = a.F;
  g.gelu_mode = a.gelu_mode;
  g.scatter = a.scatter;
  g.row_scale = a.row_scale;
  g.addend = static_cast<const unsigned char*>(a.addend);
  g.ldadd = a.ldadd;
  g.beside = a.beside;
  g.splitk_part = sk.parts;
  g.splitk_count = sk.counters;
  return g;
}

// Only the second GEMM of a call may depend on work of another stream (a fused output decode
// adds to rows that the shared expert writes there): the first GEMM runs beside it.
static int wait_before_second(const FfnArgs& a, hipStream_t stream) {
  if (a.before_second == nullptr) return SCMOE_OK;
  const hipError_t e = hipStreamWaitEvent(stream, a.before_second, 0);
  return e == hipSuccess ? SCMOE_OK : hip_fail(e);
}

// A call is one for the direct kernel in fp32, at widths that are no multiples of 64, and
//  * with at most 64 rows in all, or segments that average 16 rows or fewer (a 128- or 256-row
//    tile would be mostly padding: 8 tokens at the large widths 173 -> 129 us of layer time), or
//  * when it is small: then a launch is mostly the tiled kernel's start and end.  Up to 5e8
//    multiply-adds a product (us, tiled / direct, layer calls, rows x d x F: 300 tokens, d = 256,
//    0.8e8 46 / 29; 400, d = 512, 4.2e8 55 / 48; 200, d = 768, 4.7e8 66 / 64; 150, d = 1024, 6.3e8
//    68 / 75) and 2.2e6 outputs of all products together: the direct kernel needs a workgroup for
//    64 x 64 outputs, however short K is (tokens, d, F: 4000, 64, 128 29.2 / 25.9; 16000 32.9 / 35.6;
//    2000, 64, 512 32.6 / 31.5; 8000 39.9 / 49.1; 4000, 128, 128 31.0 / 29.4; 16000 36.0 / 43.3; 1000,
//    256, 512 34.4 / 33.0; 2000 34.6 / 40.2; 1000, 384, 768 38.3 / 43.2).  Not counted where neither
//    width fills a 128-column tile (32000, 64, 64 46.9 / 41.8).
//    Both chains of a layer decide by their mean and their sum, so that they can share launches.
bool ffn_is_tiled(int dtype, int d, int F, int max_rows, int E, int64_t mean_rows, int64_t all_rows) {
  if (dtype != SCMOE_BF16 || !ffn_mfma_supported(d, F)) return false;
  if (max_rows <= 64 || (max_rows <= 16 * static_cast<int64_t>(E) && max_rows <= 1024)) return false;
  if (gemm_variant() != 0) return true;                 // a tile configuration has been asked for
  if (static_cast<double>(mean_rows) * d * F > 5e8) return true;
  return (d >= 128 || F >= 128) && static_cast<double>(all_rows) * (d + F) > 2.2e6;
}

// Where both second GEMMs of a top-1 layer run as one product.  What it saves: the shared expert's rows
// written and read again, a launch, the decode's loads, an epilogue per row, and the idle end of one launch.
// What it costs: the shared expert's product too now has partly filled row tiles, at least one per expert.
// rows: packed rows at most.  Layer us, two launches / one (T, d, F, E; balanced load unless noted):
//  * Half a tile of F / 64 k-tiles for every expert and column tile, where the experts fill one: up to 16
//    k-tiles (21 us) for every CU here.  16384, 1024, 4096, 8 572.5 / 561.1 (4 k-tiles); 30000, 768, 3072, 8
//    659 / 588 (2); 16384, 1280, 5120, 4 843 / 779 (3); 12000, 1536, 4096, 8 with a residual 629 / 606 (6);
//    6000, 2048, 5504, 8 642.2 / 641.3 (11); 16384, 1024, 4096, 32 640.5 / 637.7 (16); 20000, 2048, 4096, 16
//    skewed 1000 / 977 (16); 16384, 1024, 2048, 64 463 / 456 (16); with 32 and F = 8192, E = 16 4096, 2048
//    681 / 673, but 8192, 2048 1021 / 1039; 16384, 2048 1900 / 1931; 32768, 2048 3722 / 3752.
//  * Experts of fewer than 256 rows have a tile each, so the shared expert's product gets E - rows / 256 row tiles
//    more than it has alone: up to 0.4 tiles per CU.  d = 1024, F = 2048, E = 64: 1100 tokens 220 / 257, 4200 268 /
//    297, 8192 309 / 326, 9600 351.6 / 352.9, 11520 (0.3 tiles per CU) 369 / 361, 12800 383 / 367; F = 1024 9600 208.3 /
//    210.6; d = 2048, F = 2048, E = 32: 600 221 / 266, 4096 296 / 298, 5120 (0.375) 345 / 309, 6400 338 / 316; E =
//    24: 2100 219 / 221, 4096 259 / 251; d = 1024, F = 1024, E = 48: 6000 164 / 159.  (0.45 pays at F = 1024, E = 48, 4800
//    156 / 152; a skewed load the host does not know: 8192, 2048, 2048, 32 340 / 354.)
// Not excluded: a capacity that drops three quarters of the tokens and more, where the shared expert's tiles fit
// the chip at once and the routed launch alone would be short (16384, 1024, 4096, 8: 4096 rows 340 / 361; 8192 rows
// 408 / 403; 8192, 2048, 2048, 8: 2048 rows 215 / 220, 4096 243 / 232).
// Below one 256 x 256 tile per CU the smaller tiles are faster, which have no such form.
bool ffn_joint_second_fits(int T, int rows, int d, int F, int E, int64_t ldh, int64_t ldw2) {
  const int64_t nt = (d + CfgA::BN - 1) / CfgA::BN, lim = BUFFER_SPAN, cus = num_cus();
  if (gemm_variant() != 0 || F % (2 * CfgA::BK) != 0 || F >= BUFFER_K || (T + 1) * ldh * 2 >= lim || (d + 1) * ldw2 * 2 >= lim) return false;
  if ((T / CfgA::BM + E) * nt < cus) return false;
  return E * nt * (F / CfgA::BK) <= 2 * 16 * cus && 5 * nt * (CfgA::BM * static_cast<int64_t>(E) - rows) <= 2 * CfgA::BM * cus;
}

// What a second GEMM of so many 256 x 128 tiles takes, in us: rounds of tiles, 0.82 us a k-tile and 4 us of epilogue and
// tile change each, and from K = SPLITK_MIN_K on a last round of few tiles cut along K (18 us to sum the parts).
// Measured / this: 256 tiles, K = 4096 63 / 61; 290 91 / 88; 200, K = 1536 28 / 29; 282, K = 2048 54 / 56; 306 65 / 60.
static double second_gemm_us(int64_t tiles, int F) {
  const int64_t slots = num_cus() / 8, n = (tiles + 7) / 8, full = n / slots, rem = n % slots;
  const double tile = 0.82 * F / CfgV::BK + 4.0;
  const int64_t parts = F >= SPLITK_MIN_K && rem > 0 ? (slots / rem < SPLITK_MAX ? slots / rem : SPLITK_MAX) : 1;
  return 5.0 + full * tile + (rem == 0 ? 0.0 : parts > 1 ? 0.82 * F / CfgV::BK / parts + 18.0 : tile);
}

bool ffn_second_in_one_launch(int T, int rows, int d, int F, int E) {
  const int64_t all = static_cast<int64_t>(T) + rows, segs = static_cast<int64_t>(E) + 1;
  if (all <= 64 * segs) return ((T + CfgS::BM - 1) / CfgS::BM + static_cast<int64_t>(E)) * ((d + CfgS::BN - 1) / CfgS::BN) <= 2 * num_cus();
  if (all <= 128 * segs) return true;
  if (d <= CfgV::BN) return false;
  const int64_t nt = (d + CfgV::BN - 1) / CfgV::BN, shared = (T + CfgV::BM - 1) / CfgV::BM * nt;
  const int64_t routed = most_row_tiles(rows, E, CfgV::BM) * nt;
  const double combine = 2.0 + 6.0 * T * d / 5.5e6;      // y_perm and s read, y written
  // Up to 15/8 rounds, counted from above: with a third one the single launch loses (two / one, layer us, tiles per CU by the
  // average: 20387 tokens, d = 320, F = 1280, E = 16 151 / 170 (1.96); 14602, d = 512, F = 1344, E = 24 176 / 191 (1.98); 10491, d = 640,
  // F = 2560, E = 32 258 / 278 (1.89); 2117, d = 2048, F = 4096, E = 8 232 / 238 (1.31, from above 1.56); nothing gained at 8192,
  // d = 1024, F = 4096, E = 8).  Of 271 drawn layers 251 are taken, four of them slower by more than 1.5 %, at most 6 (skewed).
  // And not for the fewest tiles: there either form cuts all of them into as many parts as it may, and one- and two-stream
  // calls agree bit for bit.
  if (8 * (shared + routed) > 15 * num_cus() || 8 * (shared + routed) <= num_cus()) return false;
  return second_gemm_us(shared + routed, F) + combine < second_gemm_us(shared, F) + second_gemm_us(routed, F);
}

// The shared expert's first GEMM with a layer's gate, encode and coefficient gate on the side: the tiles go to the first
// workgroups of every XCD, the gate's tokens to the last ones of the launch.
template <class CFG, int EG>
static int launch_first_with_gate(GemmArgs a, GateWork w, hipStream_t stream) {
  static std::atomic<bool> attr_set[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = -1;
  if (dev < 0 || !attr_set[dev].load(std::memory_order_acquire)) {
    hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_kernel<CFG, true, true, 0, true, EG>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, CFG::LDS_BYTES);
    if (err != hipSuccess) return hip_fail(err);
    if (dev >= 0) attr_set[dev].store(true, std::memory_order_release);
  }
  a.nt = (a.N + CFG::BN - 1) / CFG::BN;
  const int64_t tiles = (a.xrows + CFG::BM - 1) / CFG::BM * static_cast<int64_t>(a.nt);     // (no more than CUs: too little to be stored with the streaming hint)
  const int resident = num_cus() * CFG::WG_PER_CU;
  w.workgroups = (w.T + 16 * CFG::WAVES - 1) / (16 * CFG::WAVES);
  w.coef_workgroups = 0;
  if (w.cg_mode != SCMOE_CG_NONE) {
    w.coef_workgroups = (w.T + 4 * CFG::WAVES - 1) / (4 * CFG::WAVES);      // four tokens a wave, where there is room
    const int room = resident - w.workgroups;
    if (w.coef_workgroups > room) w.coef_workgroups = room;
    if (w.coef_workgroups < 1) return SCMOE_ERR_ARG;
  }
  // An XCD's tiles go to as many of its first workgroups, and the gate's workgroups follow: the slowest of those encodes, and
  // with a tile behind that the launch takes 44 us instead of 26 (7883 tokens, d = 512, F = 1344, E = 8, 186 tiles: on 248
  // workgroups the layer took 112 us, so 97).
  const int64_t all = (tiles + 7) / 8 * 8 + w.workgroups + w.coef_workgroups;
  const int grid = all < resident ? static_cast<int>((all + 7) / 8 * 8) : resident;
  if (w.workgroups + w.coef_workgroups > grid) return SCMOE_ERR_ARG;
  GateGemmArgs g;
  static_cast<GemmArgs&>(g) = a;
  g.w = w;
  hipLaunchKernelGGL((gemm_bf16_kernel<CFG, true, true, 0, true, EG>), dim3(grid), dim3(CFG::THREADS), CFG::LDS_BYTES, stream, g);
  return launch_status();
}

// Whether a layer's gate and encode go on the side of the shared expert's first GEMM, which then is a launch of its own
// ahead of the routed experts'.  What that saves are the launches of gate and encode (14 to 30 us, in which the matrix cores
// idle) and of the coefficient gate; what it costs is
//  * the encode by one workgroup where that ends after the tiles do: a wave walks its share of the choices, 64 a turn, and
//    has as many turns as the tiles have k-tiles, or three times as many with 256-row tiles, whose k-tile is that much
//    longer (layer us, apart / on the side: top-2, 5161 tokens, d = 256, F = 704, E = 8, 41 turns 51 / 68; top-4, 2304, d = 384,
//    F = 768, E = 4, 36 turns 57 / 67; 7809, d = 384, F = 1024, E = 8, 62 turns 145 / 162);
//  * a partly filled round of tiles more, so only where both launches together have no more rounds (tiles per CU, rounded up)
//    than the joint one.  The routed launch is counted from above: a balanced load with the mean half a standard deviation
//    higher, and at 256 rows a tile a skewed one, with a last tile of their own for three quarters of the experts; the joint
//    one from below at 256 rows a tile: balanced (the round cost 12 of 14 such layers 2 to 12 %: 1828, d = 960, F = 3840, E = 8 90 / 94;
//    top-2, 6950, d = 768, F = 1536 with a coefficient gate 140 / 150; top-4, 2003, d = 512, F = 1344, E = 8 70 / 78), and with a
//    quarter of the rows dropped where a capacity may, unless a coefficient gate's launch is saved as well, which is worth as much
//    as the round (1500, d = 1536, F = 4096, E = 8 130 / 142; 3001, top-2, d = 768,
//    F = 3072, E = 12 144 / 153; skewed 2733, d = 1920, F = 3840, E = 16 270 / 305; skewed with drops 8205, d = 384, F = 1024, E = 4
//    58 / 63; but taken: 500, d = 2048, F = 8192, E = 16 307 / 279; 600, d = 1024, F = 4096, E = 16 106 / 96; 8192, d = 384, F = 1536, E = 8
//    81 / 77; 6000, d = 512, F = 2048 91 / 84; with a coefficient gate top-2, 456, d = 768, F = 2048, E = 16 61 / 52).
// Of 1800 drawn layers that fit, about 1100 are taken; ten of those are slower than apart by more than 1.5 %, skewed loads whose
// rounds the host cannot count (top-3, 825 tokens, d = 1536, F = 4096, E = 16 184 / 206; 1980, d = 1856, F = 7424, E = 2 236 / 267).
// Not at widths whose tiles are done before the encode is (16000, d = 128 59 / 66; 8000, d = 192, E = 8 and 16 52 / 52 and 56 / 56),
// with 256-row tiles not below d = 384, and only up to 16 experts, for which alone the launch is built.
bool ffn_gate_on_the_side(const GateWork& g, int rows, int F, int64_t ldw1) {
  const int64_t lim = BUFFER_SPAN, cus = num_cus(), items = static_cast<int64_t>(g.T) * g.k;
  if (gemm_variant() != 0 || !aligned16(g.Wg) || g.d < 256 || g.d >= 4096 || g.E > 16 || items > 32768) return false;
  if (static_cast<int64_t>(g.T) * g.ldxc * 2 >= lim || static_cast<int64_t>(F) * ldw1 * 2 >= lim) return false;
  const int edge = takes_large_tiles(true, true, rows, g.E, g.T, F) ? 256 : 128;
  const int64_t nt = (F + edge - 1) / edge, shared = (g.T + edge - 1) / edge * nt, gate = (g.T + edge / 2 - 1) / (edge / 2);
  if (gate > cus || (shared + 7) / 8 * 8 + (edge == 256 ? gate : 0) > cus || (edge == 256 && g.d < 384)) return false;     // (and room for the coefficient gate)
  const int64_t turns = ((items + 63) / 64 + edge / 32 - 1) / (edge / 32);
  if (64 * turns > (edge == 256 ? 3 : 1) * g.d) return false;
  int64_t least = row_tiles(rows, g.E, edge), most = most_row_tiles(rows, g.E, edge);
  if (edge == 256) {
    most = std::max(most, static_cast<int64_t>(rows / 256 + 3 * g.E / 4));
    least = std::min(least, balanced_row_tiles(rows, g.E, edge));
    if (g.enc.capacity < g.T && g.cg_mode == SCMOE_CG_NONE) least = std::min(least, static_cast<int64_t>(rows * int64_t(3) / 1024 + g.E / 2));
  }
  return (shared + cus - 1) / cus + (most * nt + cus - 1) / cus <= (shared + least * nt + cus - 1) / cus;
}

static int launch_first_with_gate(const GemmArgs& a, int max_rows, int E, const GateWork& w, hipStream_t stream) {
  return takes_large_tiles(true, true, max_rows, E, a.xrows, a.N) ? launch_first_with_gate<CfgA, 1>(a, w, stream) : launch_first_with_gate<CfgU, 1>(a, w, stream);
}

static bool is_tiled(const FfnArgs& a, int dtype) {
  if (a.path != FFN_AUTO) return a.path == FFN_TILED;
  return ffn_is_tiled(dtype, a.d, a.F, a.max_rows, a.E, a.max_rows, a.max_rows);
}

// The two products of a call as jobs of the direct kernel.
static DirectJob direct_job(GemmArgs g, bool act, const FfnArgs& a) {
  g.rotk = a.slots ? 0 : 3;
  return DirectJob{g, act, a.max_rows};
}
static DirectJob direct_first(const FfnArgs& a) { return direct_job(first_gemm(a, SplitK{}), true, a); }
static DirectJob direct_second(const FfnArgs& a) { return direct_job(second_gemm(a, SplitK{}), false, a); }

int ffn_forward(const FfnArgs& a, int dtype, hipStream_t stream) {
  if (a.max_rows <= 0) return wait_before_second(a, stream);      // (nothing kept: the wait is the caller's join)
  if (!is_tiled(a, dtype)) {
    const DirectJob first = direct_first(a), second = direct_second(a);
    int st = launch_gemm_direct(&first, 1, dtype, stream);
    if (st == SCMOE_OK) st = wait_before_second(a, stream);
    return st == SCMOE_OK ? launch_gemm_direct(&second, 1, dtype, stream) : st;
  }
  SplitK sk;
  int* clear = nullptr;
  int st = prepare_splitk(a, sk, stream, &clear);
  if (st != SCMOE_OK) return st;
  GemmArgs first = first_gemm(a, sk);
  first.splitk_zero = clear;
  st = launch_variant<true>(first, a.max_rows, a.gather ? a.x_rows : a.max_rows, stream);
  if (st != SCMOE_OK) return st;
  st = wait_before_second(a, stream);
  if (st != SCMOE_OK) return st;
  return launch_variant<false>(second_gemm(a, sk), a.max_rows, a.max_rows, stream);
}

int ffn_forward_pair(const FfnArgs& se, const FfnArgs& rt, int dtype, hipStream_t stream) {
  if (se.d != rt.d || se.F != rt.F || se.E != 1 || (se.gather != nullptr) != (rt.joint_offsets != nullptr) || se.gelu_mode != rt.gelu_mode) return SCMOE_ERR_ARG;
  if (se.max_rows <= 0) return ffn_forward(rt, dtype, stream);
  if (rt.max_rows <= 0) return ffn_forward(se, dtype, stream);
  const bool ts = is_tiled(se, dtype), tr = is_tiled(rt, dtype);
  if (rt.joint_offsets != nullptr && (!ts || !tr || se.ldh != rt.ldh || se.ldw2 != rt.ldw2)) return SCMOE_ERR_ARG;
  if (!ts && !tr && rt.addend == nullptr) {
    const DirectJob first[2] = {direct_first(rt), direct_first(se)}, second[2] = {direct_second(rt), direct_second(se)};
    const int st = launch_gemm_direct(first, 2, dtype, stream);
    return st == SCMOE_OK ? launch_gemm_direct(second, 2, dtype, stream) : st;
  }
  if (!ts || !tr) {
    const int st0 = ffn_forward(se, dtype, stream);      // the shared expert first: rt may add to its rows
    return st0 == SCMOE_OK ? ffn_forward(rt, dtype, stream) : st0;
  }
  SplitK sks, skr;
  int st = prepare_splitk(se, sks, stream);
  if (st != SCMOE_OK) return st;
  st = prepare_splitk(rt, skr, stream);
  if (st != SCMOE_OK) return st;
  auto with_shared = [&](GemmArgs g, const GemmArgs& x) {      // x as the dense extra segment of g's launch
    g.xrows = se.max_rows;
    g.xA = x.A;
    g.xlda = x.lda;
    g.xW = x.W;
    g.xldw = x.ldw;
    g.xbias = x.bias;
    g.xgather = x.gather;
    g.xC = x.C;
    g.xldc = x.ldc;
    return g;
  };
  const GemmArgs s2 = second_gemm(se, sks), r2 = second_gemm(rt, skr);
  if (se.gate != nullptr) {
    GemmArgs none = first_gemm(rt, SplitK{});      // (no routed tiles)
    none.E = 0;
    st = launch_first_with_gate(with_shared(none, first_gemm(se, SplitK{})), rt.max_rows, rt.E, *se.gate, stream);
    if (st == SCMOE_OK) st = launch_variant<true>(first_gemm(rt, skr), rt.max_rows, rt.gather ? rt.x_rows : rt.max_rows, stream);
  } else {
    st = launch_variant<true>(with_shared(first_gemm(rt, skr), first_gemm(se, sks)), rt.max_rows, rt.gather ? rt.x_rows : rt.max_rows, stream);
  }
  if (st != SCMOE_OK) return st;
  if (rt.joint_offsets != nullptr) {
    GemmArgs g = r2;
    g.offsets = rt.joint_offsets;
    g.E = rt.E + 1;
    g.A2 = s2.A;
    g.W2 = s2.W;
    g.bias2 = s2.bias;
    return launch_joint_second(g, se.max_rows, stream);
  }
  // Neither decodes (more than one expert per token): one launch, whose tiles fill the chip better
  // (3001 tokens, top-2, d = 768, F = 3072, E = 12: 193 -> 167 us of layer time).
  if (decode_kind(s2) == 0 && decode_kind(r2) == 0) return launch_variant<false>(with_shared(r2, s2), rt.max_rows, rt.max_rows, stream);
  st = launch_variant<false>(s2, se.max_rows, se.max_rows, stream);
  if (st != SCMOE_OK) return st;
  return launch_variant<false>(r2, rt.max_rows, rt.max_rows, stream);
}

}  // namespace scmoe
