// Gate routing on the matrix cores (ScMoE paper Eq. (2)-(4)) as a piece of device code that a workgroup of any launch can
// run, with the input encode (Sec. 2.2) of calls whose gate and encode share a launch.
#pragma once
#include "common.hpp"
#include "mfma_common.hpp"

namespace scmoe {

// A choice, written at device scope (past the caches that are not shared by the whole device) if AGENT.
template <bool AGENT>
__device__ __forceinline__ void store_choice(int32_t* p, int v) {
  if constexpr (AGENT) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

// Top-k selection and gate weights of one token from its E <= NE logits `l` in LDS (Eq. (2)-(3));
// also returns the maximum and the sum of exp(l - max) for the caller's softmax output.  One lane
// walks a token's logits, so the walk is kept out of the LDS: all logits are read at once into
// registers, and every pass over them is unrolled (instead of reading them one after the other,
// each compare waiting for its read: top-2, 4096 tokens, d = 1024, E = 64 47.6 -> 43.0 us, E = 32
// 25.6 -> 23.4).
template <int NE, bool AGENT>
__device__ __forceinline__ void route_token_n(const float* l, int E, int k, int normalize, bool write, int64_t t,
                                              int32_t* __restrict__ expert_idx, float* __restrict__ gate_w,
                                              float& m_out, float& sum_out) {
  float v[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) v[e] = l[e < E ? e : E - 1];
  // the j-th choice: largest logit among the experts not chosen yet, lowest index among
  // equals, a NaN only if nothing else is left
  int sel[SCMOE_MAX_TOPK];
  float sv[SCMOE_MAX_TOPK];
  unsigned long long taken = 0ull;
#pragma unroll
  for (int j = 0; j < SCMOE_MAX_TOPK; ++j) {
    int best = -1;
    float bv = 0.0f;
    if (j < k) {
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const bool free = e < E && !((taken >> e) & 1ull);
        const bool take = free && (best < 0 || v[e] > bv || (bv != bv && v[e] == v[e]));
        best = take ? e : best;
        bv = take ? v[e] : bv;
      }
      taken |= 1ull << best;
    }
    sel[j] = best;
    sv[j] = bv;
  }
  float m = -INFINITY;
#pragma unroll
  for (int e = 0; e < NE; ++e)
    if (e < E && v[e] > m) m = v[e];
  float sum = 0.0f;
#pragma unroll
  for (int e = 0; e < NE; ++e)
    if (e < E) sum += expf(v[e] - m);
  m_out = m;
  sum_out = sum;
  if (write) {
    // normalize: softmax over the selected logits only, taken relative to the first
    // (largest) one, whose term is exactly 1
    float z[SCMOE_MAX_TOPK];
    float zsum = 0.0f;
#pragma unroll
    for (int j = 0; j < SCMOE_MAX_TOPK; ++j) {
      z[j] = 0.0f;
      if (j < k) {
        z[j] = (j == 0) ? 1.0f : expf(sv[j] - sv[0]);
        zsum += z[j];
      }
    }
#pragma unroll
    for (int j = 0; j < SCMOE_MAX_TOPK; ++j) {
      if (j < k) {
        store_choice<AGENT>(expert_idx + t * k + j, sel[j]);
        gate_w[t * k + j] = normalize ? z[j] / zsum : expf(sv[j] - m) / sum;
      }
    }
  }
}

// EMAX: the most experts the caller's kernel can have.
template <int EMAX, bool AGENT = false>
__device__ __forceinline__ void route_token(const float* l, int E, int k, int normalize, bool write, int64_t t,
                                            int32_t* __restrict__ expert_idx, float* __restrict__ gate_w,
                                            float& m_out, float& sum_out) {
  static_assert(SCMOE_MAX_EXPERTS == 64 && EMAX <= 64, "sizes below");
  if (EMAX <= 8 || E <= 8) route_token_n<8, AGENT>(l, E, k, normalize, write, t, expert_idx, gate_w, m_out, sum_out);
  else if (EMAX <= 16 || E <= 16) route_token_n<16, AGENT>(l, E, k, normalize, write, t, expert_idx, gate_w, m_out, sum_out);
  else if (EMAX <= 32 || E <= 32) route_token_n<32, AGENT>(l, E, k, normalize, write, t, expert_idx, gate_w, m_out, sum_out);
  else route_token_n<64, AGENT>(l, E, k, normalize, write, t, expert_idx, gate_w, m_out, sum_out);
}

// The chains on the matrix cores.  The fp32
// matrix instruction v_mfma_f32_16x16x4_f32 adds its four products to the accumulator one
// after the other in ascending k, each step rounded like a fused multiply-add (checked bit for
// bit against fmaf chains, subnormal sums and cancellation included), so one instruction
// advances the 16 x 16 chains of 16 tokens and 16 experts by four features: the same bits as
// the kernels below at a quarter of a dependent instruction per feature and chain.  With more
// than 16 experts a wave keeps EG = 2 or 4 accumulators, one per group of 16 experts, and
// every step issues EG independent instructions on the same x operand; where there are fewer waves than SIMDs, GW = 2 or
// 4 waves share 16 tokens instead, each with a group of its own, and the chain is as short as with 16 experts.
// A wave owns 16 tokens.  Nothing passes through registers on the way in: x rows and W_g are
// copied global -> LDS directly (so the compiler never waits for a register load, which with
// such copies in flight would drain all of them), x into a ring of XS stages per wave (a
// stage: 128 bytes of each of the 16 rows, two copies of 1 KiB), W_g in tiles of 256 / EG
// features into a ring of buffers shared by the workgroup (its natural [feature][expert] order
// is already the operand order: lane (c, kq) of step s reads expert c of feature 4 s + kq).
// Operands are read from LDS a few steps ahead of the matrix instructions that use them.  Waits
// are explicit: copies complete in issue order, so "all but the newest n" names a stage.
constexpr int GM_STAGE = 2048;           // bytes per stage: 16 rows x 128 bytes
constexpr int GM_WBUF = 16 * 1024;       // bytes per W_g buffer: a tile of 256 features of 16 experts, 128 of 32, 64 of 64

// LDS reads and waits of the matrix-core gate kernel's main loop, written out (see there).
// The result register of a read is not valid before an lds_wait that names it.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(SCMOE_LDS_PTR(p)));
}
template <int OFF>
__device__ __forceinline__ void lds_read_b32(uint32_t& r, uint32_t addr) {
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
}
// a bf16 into the upper half of r (whose lower half stays as it is: zero), i.e. the fp32 value
template <bool BF16, int OFF>
__device__ __forceinline__ void lds_read_x(uint32_t& r, uint32_t addr) {
  if constexpr (BF16) asm volatile("ds_read_u16_d16_hi %0, %1 offset:%2" : "+v"(r) : "v"(addr), "n"(OFF));
  else asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
}
// the x operand of step S inside a stage: which 16-byte column of a 64-byte copy, and its byte offset
// from there (for the lane's row and feature)
template <bool BF16>
constexpr int gm_x_col(int S) { return BF16 ? (S >> 1) & 3 : S & 3; }
template <bool BF16>
constexpr int gm_x_off(int S) { return BF16 ? (S >> 3) * 1024 + (S & 1) * 8 : (S >> 2) * 1024; }
// until at most N of the LDS reads issued so far are outstanding; x and w are valid afterwards
template <int N, int EG>
__device__ __forceinline__ void lds_wait(uint32_t& x, uint32_t (&w)[EG]) {
  static_assert(N >= 0 && N < 15 && (EG == 1 || EG == 2 || EG == 4), "lgkmcnt field");
  if constexpr (EG == 1) asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(x), "+v"(w[0]) : "n"(N));
  else if constexpr (EG == 2) asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(x), "+v"(w[0]), "+v"(w[1]) : "n"(N));
  else asm volatile("s_waitcnt lgkmcnt(%5)" : "+v"(x), "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]) : "n"(N));
}

// Shape of the kernel for EG groups of 16 experts per wave, GW waves that share 16 tokens (E <= 16 EG GW; one of EG and
// GW is 1), NW waves per workgroup and ROOM bytes of LDS.
template <bool BF16, int NW, int EG, int ROOM = 160 * 1024, int GW = 1>
struct GateMfmaCfg {
  static constexpr int G = EG * GW;                   // groups in all
  static constexpr int EB = BF16 ? 2 : 4;
  static constexpr int SF = 128 / EB;                 // features per stage of x
  static constexpr int SS = SF / 4;                   // steps (of four features) per stage
  static constexpr int KC = 256 / G;                  // features per W_g tile: at most 16 KiB
  static constexpr int IPT = KC / SF;                 // stages per W_g tile
  static constexpr int WB = G == 1 ? 2 : G == 2 ? 3 : 4;               // W_g buffers: tile j + WB - 1 is requested when tile j begins
  static constexpr int XS0 = NW == 16 ? 3 : EG == 1 ? (NW == 8 ? 7 : 8) : EG == 2 ? 6 : 5, XS1 = (ROOM - WB * GM_WBUF) / (NW * GM_STAGE);
  static constexpr int XS = XS0 < XS1 ? XS0 : XS1;                     // x ring stages per wave
  static constexpr int P = EG == 1 ? SS / 2 : EG == 2 ? 4 : 2;         // steps the operand reads run ahead of their use
  static constexpr int LGS = 16 * G + 1;              // row stride of the logit exchange buffer
  static constexpr int TOK = 16 * NW / GW;
  static_assert((EG == 1 || GW == 1) && NW % GW == 0, "groups");
  static constexpr int LDS = WB * GM_WBUF + NW * XS * GM_STAGE;
  static_assert(IPT >= 1 && SS % P == 0 && P <= SS / 2, "steps per stage and per tile");
  static_assert((P - 1) * (1 + EG) < 15, "LDS reads a wait can count");
  static_assert(XS >= 3 && 2 * (XS - 2) < 64, "ring depth");
  static_assert(TOK * (LGS + 2) * 4 <= WB * GM_WBUF, "the logits, their maxima and sums fit the W_g buffers");
  static_assert(WB >= 2 && LDS <= ROOM, "LDS");
};

// The input encode of a call whose tokens all belong to this workgroup: thread i has item i = j T + t (the
// order of dispatch_onepass, whose results these are), at most 64 NW of them.  lds: (NW + 1) * 64 ints.
template <int NW>
__device__ __forceinline__ void dispatch_own(const int32_t* expert_idx, int T, int k, int E, const DispatchOut& o, int* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = threadIdx.x;
  for (int z = i; z < o.ch.nzero; z += 64 * NW) {
    if (o.ch.zero_a != nullptr) o.ch.zero_a[z] = 0;
    if (o.ch.zero_b != nullptr) o.ch.zero_b[z] = 0;
  }
  if (o.ch.pair != nullptr && i == 0) {
    o.ch.pair[0] = 0;
    o.ch.pair[1] = o.ch.pair_hi;
  }
  const int n = T * k, j = i / T, t = i - j * T;
  int e = -1;
  if (i < n) e = expert_idx[t * k + j];
  if (e >= E) e = -1;
  // items of the wave whose expert is `lane`, and the lanes that hold this lane's expert
  unsigned long long mine = __ballot(e >= 0), same = mine;
  for (int b = 0; (1 << b) < E; ++b) {
    const unsigned long long bal = __ballot(e >= 0 && ((e >> b) & 1));
    mine &= ((lane >> b) & 1) ? bal : ~bal;
    same &= ((e >> b) & 1) ? bal : ~bal;
  }
  const int rank = __popcll(same & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
  lds[wave * 64 + lane] = __popcll(mine);
  __syncthreads();
  if (wave == 0) {
    int run = 0;                                          // items of expert `lane` in the waves before
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int c = lds[w * 64 + lane];
      lds[w * 64 + lane] = run;
      run += c;
    }
    const int c = lane < E ? (run < o.capacity ? run : o.capacity) : 0;
    int incl = c;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int up = __shfl_up(incl, off, 64);
      if (lane >= off) incl += up;
    }
    lds[NW * 64 + lane] = incl - c;
    if (lane < E) {
      o.counts[lane] = c;
      o.offsets[lane] = incl - c;
      if (lane == E - 1) o.offsets[E] = incl;
    }
  }
  __syncthreads();
  if (i < n) {
    int out = -1;
    if (e >= 0) {
      const int slot = lds[wave * 64 + e] + rank;
      if (slot < o.capacity) {
        out = lds[NW * 64 + e] + slot;
        o.src_token[out] = t;
      }
    }
    o.dst_row[t * k + j] = out;
  }
}

// The input encode of a whole call by one workgroup: the items in order, an equal share of consecutive 64-item vectors
// to every wave, counted and ranked inside their vectors on one walk, placed on a second one, with the results of
// dispatch_onepass.  The choices come from other workgroups of this launch and are read at device scope.
// Up to 16 experts.  lds: (NW + 1) * 64 ints, then two bytes an item, in whole vectors.
template <int NW>
__device__ __forceinline__ void dispatch_all(const int32_t* expert_idx, int T, int k, int E, const DispatchOut& o, int* lds) {
  constexpr int ROUND = 8, NB = 4;                        // vectors whose loads are in flight together; bits of an expert index
  for (int z = threadIdx.x; z < o.ch.nzero; z += 64 * NW) {
    if (o.ch.zero_a != nullptr) o.ch.zero_a[z] = 0;
    if (o.ch.zero_b != nullptr) o.ch.zero_b[z] = 0;
  }
  if (o.ch.pair != nullptr && threadIdx.x == 0) {
    o.ch.pair[0] = 0;
    o.ch.pair[1] = o.ch.pair_hi;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = T * k, nvec = (n + 63) >> 6, per = (nvec + NW - 1) / NW;
  const int va = wave * per, vz = va + per < nvec ? va + per : nvec;
  unsigned char* const choice = reinterpret_cast<unsigned char*>(lds + (NW + 1) * 64);     // expert of item i; 255: none
  unsigned char* const ahead = choice + nvec * 64;        // lanes before it in its vector with the same expert
  const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  // (the loops are kept short: one workgroup runs them once, and its instructions come from memory)
#pragma unroll 1
  for (int v0 = va; v0 < vz; v0 += ROUND) {
    int ev[ROUND];
#pragma unroll
    for (int u = 0; u < ROUND; ++u) {
      const int i = (v0 + u) * 64 + lane, c = i < n ? i : n - 1;
      const int j = (c >= T) + (c >= 2 * T) + (c >= 3 * T);
      ev[u] = __hip_atomic_load(expert_idx + (c - j * T) * k + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int u = 0; u < ROUND; ++u) {
      const int i = (v0 + u) * 64 + lane;
      if (v0 + u < vz) choice[i] = static_cast<unsigned char>(i < n && ev[u] >= 0 && ev[u] < E ? ev[u] : 255);
    }
  }
  int cnt = 0;                                            // items of expert `lane`
#pragma unroll 1
  for (int v = va; v < vz; ++v) {
    const int e = choice[v * 64 + lane];
    unsigned long long mine = __ballot(e != 255), same = mine;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const bool bit = (e >> b) & 1;
      const unsigned long long bal = __ballot(bit);
      mine &= ((lane >> b) & 1) ? bal : ~bal;
      same &= bit ? bal : ~bal;
    }
    cnt += __popcll(mine);
    ahead[v * 64 + lane] = static_cast<unsigned char>(__popcll(same & below));
  }
  lds[wave * 64 + lane] = cnt;
  __syncthreads();
  if (wave == 0) {
    int run = 0;                                          // items of expert `lane` in the waves before
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int c = lds[w * 64 + lane];
      lds[w * 64 + lane] = run;
      run += c;
    }
    const int c = lane < E ? (run < o.capacity ? run : o.capacity) : 0;
    int incl = c;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int up = __shfl_up(incl, off, 64);
      if (lane >= off) incl += up;
    }
    lds[NW * 64 + lane] = incl - c;
    if (lane < E) {
      o.counts[lane] = c;
      o.offsets[lane] = incl - c;
      if (lane == E - 1) o.offsets[E] = incl;
    }
  }
  __syncthreads();
  int base = lds[wave * 64 + lane];                       // items of expert `lane` before the vector
  const int seg = lds[NW * 64 + lane];
#pragma unroll 1
  for (int v = va; v < vz; ++v) {
    const int i = v * 64 + lane, e = choice[i];
    const int slot = __shfl(base, e & 63) + ahead[i], first = __shfl(seg, e & 63);
    unsigned long long mine = __ballot(e != 255);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const unsigned long long bal = __ballot((e >> b) & 1);
      mine &= ((lane >> b) & 1) ? bal : ~bal;
    }
    base += __popcll(mine);
    if (i < n) {
      const int out = e != 255 && slot < o.capacity ? first + slot : -1;
      const int j = (i >= T) + (i >= 2 * T) + (i >= 3 * T), t = i - j * T;
      if (out >= 0) o.src_token[out] = t;
      o.dst_row[t * k + j] = out;
    }
  }
}

// Marks workgroup `mine` of `all` as done and says whether all are (called by one whole wave; its earlier stores have been
// performed).  The last one to be marked sees all marks; others may as well.  A mark is the number of the call (call_number),
// another one for every call, because the memory is the caller's and not cleared: whatever lies there counts as a mark only if
// it is that number, which for other data has a probability of 2^-64 a mark and which no other call of the process has.
// A replayed graph has the same number again, so whoever saw all marks clears them.
__device__ __forceinline__ bool all_arrived(unsigned long long* marks, unsigned long long call, int mine, int all) {
  const int lane = threadIdx.x & 63;
  if (lane == 0) __hip_atomic_store(marks + mine, call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  bool there = true;
  for (int i = lane; i < all; i += 64) there = there && __hip_atomic_load(marks + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == call;
  return __all(there);
}

// What a gate workgroup does beside the choices of its tokens: nothing; the input encode of a call whose tokens are all
// its own (dispatch_own); count itself in, and the last of the launch's gate workgroups does the encode (dispatch_all).
enum { GATE_ONLY = 0, GATE_ENC_OWN = 1, GATE_ENC_LAST = 2 };

// The workgroup's part of the gate: tokens 16 NW / GW block and on.  gm: ROOM bytes of LDS, 1024-byte aligned.
template <bool BF16, int NW, int EG, int MODE, int ROOM = 160 * 1024, int GW = 1>
__device__ __forceinline__ void gate_mfma(
    unsigned char* gm, int block, const unsigned char* __restrict__ x, int64_t ldx, const float* __restrict__ Wg,
    const float* __restrict__ bias, int T, int d, int E, int k, int normalize,
    int32_t* __restrict__ expert_idx, float* __restrict__ gate_w, float* __restrict__ probs, const DispatchOut& enc,
    unsigned long long* marks, unsigned long long call, int workgroups) {
  using C = GateMfmaCfg<BF16, NW, EG, ROOM, GW>;
  constexpr int EB = C::EB, SS = C::SS, KC = C::KC, IPT = C::IPT, WB = C::WB, XS = C::XS, P = C::P;
  constexpr int TOK = C::TOK, LGS = C::LGS;
  constexpr bool AGENT = MODE == GATE_ENC_LAST;           // the choices are read by another workgroup of this launch
  // gm: [WB W_g buffers][NW rings]; afterwards [logits][their maxima][sums]
  float* const row_max = reinterpret_cast<float*>(gm) + TOK * LGS;
  float* const row_sum = row_max + TOK;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, kq = lane >> 4;
  const int t0 = block * TOK;
  const int NS = d / 4;                                   // steps in all
  const int NI = (NS + SS - 1) / SS;                      // stages in all
  unsigned char* const ring = gm + WB * GM_WBUF + wave * (XS * GM_STAGE);

  // ---- copies --------------------------------------------------------------------------------
  // x: lane p of a copy fetches 16 bytes of row p / 4, at a 16-byte column of the 64 bytes the copy
  // covers, and they land at ring position p.  Four lanes share the 64 bytes of a row: a copy whose
  // neighbouring lanes read different rows takes the compute unit's address path up to four times as
  // long (18 against 63 B/ns from the caches; four waves' copies would fill it at the rate the chain
  // has now).  The column is p % 4
  // XOR (row / 4) % 4, which spreads the operand reads over all banks.  Columns past the row's end
  // re-read its last 16 bytes (never consumed), and so do whole stages past the end, which keeps
  // the number of copies per stage fixed for the waits below.
  const int crow = lane >> 2, ccol = (lane & 3) ^ ((lane >> 4) & 3);
  const int tgroup = wave / GW, egroup = wave % GW;       // 16 tokens; 16 experts (GW > 1)
  int trow = t0 + tgroup * 16 + crow;
  if (trow > T - 1) trow = T - 1;
  const unsigned char* const xrow = x + static_cast<int64_t>(trow) * ldx * EB;
  const int row_last = d * EB - 16;
  auto issue_x = [&](int i, int slot) {
    unsigned char* dst = ring + slot * GM_STAGE;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int off = i * 128 + h * 64 + ccol * 16;
      if (off > row_last) off = row_last;
      __builtin_amdgcn_global_load_lds(SCMOE_GLB_PTR(xrow + off), SCMOE_LDS_PTR(dst + h * 1024), 16, 0, 0);
    }
  };
  // W_g tile j is the bytes [4 KC E j, 4 KC E (j + 1)) of the matrix (whole rows), copied 1 KiB at
  // a time by the waves in turn; the last copy of a tile may reach into the next tile, and past
  // the end of the matrix a copy re-reads its last 16 bytes (never consumed).
  const unsigned char* const wg = reinterpret_cast<const unsigned char*>(Wg);
  const int64_t w_last = static_cast<int64_t>(d) * E * 4 - 16;
  const int w_copies = (E + C::G - 1) / C::G;                 // = ceil(4 KC E / 1024)
  auto issue_w = [&](int j, int buf) {
    unsigned char* dst = gm + buf * GM_WBUF;
    for (int u = wave; u < w_copies; u += NW) {
      int64_t off = static_cast<int64_t>(j) * (4 * KC) * E + u * 1024 + lane * 16;
      if (off > w_last) off = w_last;
      __builtin_amdgcn_global_load_lds(SCMOE_GLB_PTR(wg + off), SCMOE_LDS_PTR(dst + u * 1024), 16, 0, 0);
    }
  };
  auto wait_vm = [&](auto n_c) {
    constexpr int n = decltype(n_c)::value;
    static_assert(n < 64, "vmcnt field");
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | 0x0F70);
    asm volatile("" ::: "memory");
  };
  // Copies that may still be on their way when stage i + 1 is needed: those of the XS - 2 stages
  // after it.  At the end of a W_g tile the next tile must be in as well; it was requested
  // (WB - 1) IPT stages of x ago (copies complete in issue order).
  using InFlight = std::integral_constant<int, 2 * (XS - 2)>;
  using InFlightTileEnd = std::integral_constant<int, (XS - 2 < (WB - 1) * IPT) ? 2 * (XS - 2) : 2 * (WB - 1) * IPT>;

  // ---- operands ------------------------------------------------------------------------------
  // x: token c16's 16 bytes of 16-byte column q sit at ring position 4 c16 + (q ^ (c16 / 4)); W_g:
  // feature row f of the tile starts at byte 4 E f.  Lanes past the last expert read what lies there
  // (in bounds: the rings follow the tiles; their rows of the product are never looked at).
  int xl[4], wl[SS];
#pragma unroll
  for (int q = 0; q < 4; ++q) xl[q] = (c16 * 4 + (q ^ (c16 >> 2))) * 16 + kq * EB;
#pragma unroll
  for (int s = 0; s < SS; ++s) wl[s] = ((4 * s + kq) * E + c16) * 4 + 64 * egroup;     // of step s of a stage
  // Operand registers hold what the matrix instruction takes: fp32 bits (a bf16 in the upper half).
  // P steps are in registers or on their way at any time: step s uses slot s % P.
  uint32_t xr[P], wr[P][EG];
  f32x4_t acc[EG];
#pragma unroll
  for (int g = 0; g < EG; ++g) acc[g] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  // experts are the rows of the product (first operand), tokens its columns: lane (c16, kq)
  // ends with token c16 and experts 16 g + 4 kq .. 16 g + 4 kq + 3 of every group g
  auto chain_step = [&](int slot_r) {
#pragma unroll
    for (int g = 0; g < EG; ++g)
      acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wr[slot_r][g]), __uint_as_float(xr[slot_r]), acc[g], 0, 0, 0);
  };
  // step S of the stage at xs, whose W_g rows start at ws (plain reads: the compiler waits for them)
  auto read_step = [&](int slot_r, const unsigned char* xs, const unsigned char* ws, int S) {
    const unsigned char* const xp = xs + xl[gm_x_col<BF16>(S)] + gm_x_off<BF16>(S);
    if (BF16) xr[slot_r] = static_cast<uint32_t>(*reinterpret_cast<const uint16_t*>(xp)) << 16;
    else xr[slot_r] = *reinterpret_cast<const uint32_t*>(xp);
#pragma unroll
    for (int g = 0; g < EG; ++g) wr[slot_r][g] = *reinterpret_cast<const uint32_t*>(ws + wl[S] + 64 * g);
  };

#pragma unroll
  for (int j = 0; j < WB - 1; ++j)
    if (j * KC < d) issue_w(j, j);
#pragma unroll
  for (int i = 0; i < XS - 1; ++i) issue_x(i, i);
  wait_vm(InFlight{});                                    // the first W_g tiles and stage 0 are in LDS
  lds_barrier();
#pragma unroll
  for (int s = 0; s < P; ++s) read_step(s, ring, gm, s);
  int slot = 0, slot_free = XS - 1;                       // ring slots of stage i and of stage i - 1
  int wbuf = 0, wbuf_free = WB - 1;                       // buffers of W_g tile j and of tile j - 1
  int i = 0;
  auto next_slot = [&]() {
    slot_free = slot;
    slot = (slot + 1 == XS) ? 0 : slot + 1;
  };
  auto next_wbuf = [&]() {
    wbuf_free = wbuf;
    wbuf = (wbuf + 1 == WB) ? 0 : wbuf + 1;
  };

  // Whole W_g tiles: IPT stages in straight-line code.  A dependent matrix instruction issues
  // only when the one before it has finished, and the wave issues in order, so the reads of the
  // operands P steps ahead and the copies are placed between the matrix instructions, where they cost
  // nothing.  Not so vector instructions: one between two dependent matrix instructions makes the
  // step 55 to 67 cycles long, without any it is 33 (a probe of this loop on one wave).  So the
  // addresses of the operands are worked out for half a stage at a time, and all that is added
  // to them is a constant (us, with one per step / so, 500 tokens: d = 2048,
  // E = 16 19.1 / 16.0, E = 32 35.9 / 28.2, E = 64 66.6 / 50.7; d = 4096, E = 16 34.3 / 28.6; 8 tokens the same).
  // The operand reads and their waits are written out here (lds_read_*, lds_wait): with
  // global -> LDS copies in flight every wait the compiler generates is a wait for everything,
  // i.e. for the reads issued just before.  LDS reads complete in order: a step's operands were
  // read P steps earlier, (P - 1) (1 + EG) reads ago.
  const int NTF = NS / (IPT * SS);
  uint32_t xa[4], wa[SS];                                  // operand addresses: x columns of a stage, W_g of its steps
  auto addresses = [&](uint32_t& a, const unsigned char* base, int off) {
    asm volatile("v_add_u32 %0, %1, %2" : "=v"(a) : "s"(lds_addr(base)), "v"(off));
  };
#pragma unroll
  for (int c = 0; c < 4; ++c) addresses(xa[c], ring, xl[c]);
  for (int j = 0; j < NTF; ++j) {
    if ((j + WB - 1) * KC < d) issue_w(j + WB - 1, wbuf_free);   // that buffer was released by the last barrier
    const unsigned char* const wt = gm + wbuf * GM_WBUF;
    next_wbuf();
    const unsigned char* const wt_next = gm + wbuf * GM_WBUF;
    static_for<0, IPT>([&](auto q_c) {
      constexpr int q = decltype(q_c)::value;
      issue_x(i + XS - 1, slot_free);
      next_slot();
#pragma unroll
      for (int s = P; s < SS; ++s) addresses(wa[s], wt + q * (SS * 16) * E, wl[s]);
      static_for<0, SS>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value, s2 = s + P;
        if constexpr (s == SS - P) {                      // the reads of the next stage begin with this step
          if (q == IPT - 1) {
            wait_vm(InFlightTileEnd{});                   // stage i + 1 and this wave's share of the next W_g tile are in LDS
            lds_barrier();                                // every wave has read its last operands of this tile; all shares of the next are in
          } else {
            wait_vm(InFlight{});                          // stage i + 1 is in LDS
          }
          // (after the last stage: stale but in-bounds LDS, unused)
#pragma unroll
          for (int c = 0; c < 4; ++c) addresses(xa[c], ring + slot * GM_STAGE, xl[c]);
#pragma unroll
          for (int c = 0; c < P; ++c) addresses(wa[c], q == IPT - 1 ? wt_next : wt + (q + 1) * (SS * 16) * E, wl[c]);
        }
        lds_wait<(P - 1) * (1 + EG)>(xr[s % P], wr[s % P]);
        chain_step(s % P);
        lds_read_x<BF16, gm_x_off<BF16>(s2 % SS)>(xr[s % P], xa[gm_x_col<BF16>(s2 % SS)]);
        static_for<0, EG>([&](auto g_c) { lds_read_b32<64 * decltype(g_c)::value>(wr[s % P][decltype(g_c)::value], wa[s2 % SS]); });
      });
      ++i;
    });
    // the operands just read are carried into the next round in registers the compiler may
    // copy: they have to be there before it does
    static_for<0, P>([&](auto s_c) { lds_wait<0>(xr[decltype(s_c)::value], wr[decltype(s_c)::value]); });
  }
  // The rest of a last, partial tile, stage by stage, with plain reads (the last stage may be short).
  while (i < NI) {
    const int q = i % IPT;
    if (q == 0 && (i / IPT + WB - 1) * KC < d) issue_w(i / IPT + WB - 1, wbuf_free);
    issue_x(i + XS - 1, slot_free);
    const int steps = NS - i * SS;                        // at least 2; SS or more unless this is the last stage
    const unsigned char* const xs = ring + slot * GM_STAGE;
    next_slot();
    const unsigned char* const xs_next = ring + slot * GM_STAGE;
    const unsigned char* const wt = gm + wbuf * GM_WBUF;
    const unsigned char* const wt_next = gm + (wbuf + 1 == WB ? 0 : wbuf + 1) * GM_WBUF;
    if (q == IPT - 1) next_wbuf();
    static_for<0, SS>([&](auto s_c) {
      constexpr int s = decltype(s_c)::value, s2 = s + P;
      if constexpr (s == SS - P) {
        if (q == IPT - 1 && i + 1 < NI) {
          wait_vm(InFlightTileEnd{});
          lds_barrier();
        } else {
          wait_vm(InFlight{});
        }
      }
      if (s < steps) chain_step(s % P);
      if (s2 < SS) read_step(s % P, xs, wt + q * (SS * 16) * E, s2);
      else read_step(s % P, xs_next, q == IPT - 1 ? wt_next : wt + (q + 1) * (SS * 16) * E, s2 - SS);
    });
    ++i;
  }
  wait_vm(std::integral_constant<int, 0>{});              // no copy may land after the workgroup has given up its LDS
  auto encode = [&]() {
    if constexpr (MODE == GATE_ENC_OWN) {
      __syncthreads();                                    // the choices are written, the buffers free
      dispatch_own<NW>(expert_idx, T, k, E, enc, reinterpret_cast<int*>(gm));
    } else if constexpr (MODE == GATE_ENC_LAST) {
      wait_vm(std::integral_constant<int, 0>{});          // this wave's choices are where every workgroup sees them
      __syncthreads();                                    // ... and every wave's
      int* const last = reinterpret_cast<int*>(gm + C::LDS) - 1;
      if (wave == 0) {
        const bool all = all_arrived(marks, call, block, workgroups);
        if (lane == 0) *last = all;
      }
      __syncthreads();
      if (*last != 0) {                                   // (two workgroups may find all the others done: they write the same)
        for (int i = tid; i < workgroups; i += 64 * NW) __hip_atomic_store(marks + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        dispatch_all<NW>(expert_idx, T, k, E, enc, reinterpret_cast<int*>(gm));
      }
    }
  };
  if (EG == 1 && GW == 1 && k == 1 && probs == nullptr) {
    // Top-1 without the probability output is routed in registers: a lane folds its four logits,
    // then the four lanes of a token (16 lanes apart, in ascending expert order) fold theirs.
    // Same rule and same operations in the same order as route_token, hence the same bits: the
    // largest logit wins, the lowest index among equals, a NaN only against another NaN; the
    // softmax denominator is summed expert after expert, handed from lane to lane.
    // (written with selects, on copies of the accumulators pinned to vector registers: the
    // same logic as nested branches on the accumulator tuple came out of the compiler with two
    // of the four logits overwritten by the first one)
    float v[4];
    float bv = 0.0f, mx = -INFINITY;
    int bi = -1;                                          // (no expert yet)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int e = 4 * kq + r;
      const bool valid = e < E;
      float a = acc[0][r];
      asm volatile("" : "+v"(a));
      if (bias != nullptr) a = __fadd_rn(a, bias[valid ? e : 0]);
      v[r] = a;
      const bool take = valid && (bi < 0 || a > bv || (bv != bv && a == a));
      bi = take ? e : bi;
      bv = take ? a : bv;
      mx = (valid && a > mx) ? a : mx;
    }
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float pv = __shfl_xor(bv, off), pm = __shfl_xor(mx, off);
      const int pi = __shfl_xor(bi, off);
      if (pi >= 0) {
        if (bi < 0) { bi = pi; bv = pv; }
        else {
          const bool mine_first = bi < pi;
          const float lo = mine_first ? bv : pv, hi = mine_first ? pv : bv;
          const int lo_i = mine_first ? bi : pi, hi_i = mine_first ? pi : bi;
          const bool take_hi = hi > lo || (lo != lo && hi == hi);
          bv = take_hi ? hi : lo;
          bi = take_hi ? hi_i : lo_i;
        }
      }
      if (pm > mx) mx = pm;
    }
    float w = 1.0f;                                       // normalize: the one selected logit's softmax over itself
    if (!normalize) {
      float t[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) t[r] = expf(v[r] - mx);
      float sum = 0.0f;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float sg = sum;                                   // (meaningful in the lanes that hold group g)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * g + r < E) sg += t[r];
        sum = __shfl(sg, c16 + 16 * g);
      }
      w = expf(bv - mx) / sum;
    }
    const int t = t0 + wave * 16 + c16;
    if (kq == 0 && t < T) {
      store_choice<AGENT>(expert_idx + t, bi);
      gate_w[t] = w;
    }
    encode();
    return;
  }
  lds_barrier();                                          // the W_g buffers are free: reuse them for the logits
  float* lg = reinterpret_cast<float*>(gm);
#pragma unroll
  for (int g = 0; g < EG; ++g) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int e = 16 * (g + egroup) + 4 * kq + r;
      if (e < E) {
        float v = acc[g][r];
        if (bias != nullptr) v = __fadd_rn(v, bias[e]);
        lg[(tgroup * 16 + c16) * LGS + e] = v;
      }
    }
  }
  __syncthreads();
  if (tid < TOK)
    route_token<16 * C::G, AGENT>(lg + tid * LGS, E, k, normalize, t0 + tid < T, t0 + tid, expert_idx, gate_w, row_max[tid], row_sum[tid]);
  if (probs != nullptr) {
    __syncthreads();
    const int ntok = (T - t0 < TOK) ? T - t0 : TOK;
    for (int c = tid; c < ntok * E; c += 64 * NW) {
      const int tok = c / E, e = c - tok * E;
      probs[static_cast<int64_t>(t0) * E + c] = expf(lg[tok * LGS + e] - row_max[tok]) / row_sum[tok];
    }
  }
  encode();
}

}  // namespace scmoe
