// The persistent tile schedule of the grouped GEMM.  No device header is needed, so that what it
// hands out can be checked on the host.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define SCMOE_SCHED_FN __host__ __device__ __forceinline__
#else
#define SCMOE_SCHED_FN inline
#endif

namespace scmoe {

constexpr int SPLITK_MAX = 8;    // most parts one tile is cut into

// Persistent tile schedule.  Row tiles are counted from offsets[] on the device (no host
// round trip).  Workgroup ids congruent mod 8 run on one XCD.  The tiles form up to two
// ranges: the dense extra segment (if any) and the E segments of offsets[], segment after
// segment, each segment in the raster order "a group of up to GM row tiles x all column
// tiles" (so a group never mixes two experts' weights).  XCD x owns the x-th eighth of the
// extra segment's range; the other range is dealt to the XCDs in chunks of RR tiles, XCD
// after XCD, and only the rest that does not fill a round of chunks is cut into eighths (so
// every XCD gets the same amount of both kinds of work, and at any time all XCDs read the
// weights of the same one or two experts, which the memory-side cache then serves).  The
// workgroups of an XCD take the tiles of its share round-robin, so the tiles in flight on one
// XCD are neighbours and share A and W panels in its L2.
template <int BM, int BN, int GM, bool CAT = false>
struct TileSchedule {
  int mt_seg, nt, E, xt, xrows;   // row tiles of the offsets[] segments / of the extra segment
  const int32_t* offsets;
  int nslots;
  int a0, na, rr, b0;             // this XCD's share: tiles a0 .. a0+na-1 of the extra segment's
                                  // range; of the other range rr tiles out of the dealt chunks,
                                  // then tiles from b0 on of the undealt rest
  static constexpr int RR = 32;
  // Work items of this XCD.  Its `full` tiles fill whole rounds of nslots workgroups; the `rem`
  // tiles of the last, partly filled round are each cut along K into S parts (S > 1 only with
  // scratch for the partial sums), so that the round keeps (nearly) all workgroups busy.
  // Item order: first the rem * S parts (part w % S of local tile full + w / S), then the full
  // tiles (local tile = item - parts), then rem * FS finish items, one per FS-th of a cut tile,
  // which add the parts up and write the result.  A workgroup takes items slot, slot + nslots,
  // ...: a part is always the first item of its workgroup, a finish item the last, so the
  // partial sums are long written when they are read (the kernel still checks the arrival count).
  int full, rem, S, npart, ngemm, nfin, xcd;
  // CAT (joint second GEMM): the last segment's tiles are half as long as the others; na of them are
  // this XCD's share and follow its nr other tiles.
  int nr = 0, hole = 0;           // items hole .. hole + rem - 1 do not exist (see next)
  int cur_e = 0, cur_base = 0;    // where the last search through offsets[] ended (see locate)

  // nt column tiles; xr rows of the dense extra segment; nk k-tiles; fs finish items a cut tile;
  // workgroup i runs on XCD i mod 8, ns workgroups on each
  SCMOE_SCHED_FN TileSchedule(int nt_, int E_, const int32_t* offs, int xr, int nk, bool can_split, int FS, int xcd_, int ns)
      : mt_seg(0), nt(nt_), E(E_), xt((xr + BM - 1) / BM), xrows(xr), offsets(offs), nslots(ns), xcd(xcd_) {
    if constexpr (CAT) {
      xrows = offsets[E] - offsets[E - 1];
      xt = (xrows + BM - 1) / BM;
      --E;
    }
    for (int q = 0; q < E; ++q) mt_seg += (offsets[q + 1] - offsets[q] + BM - 1) / BM;
    auto share = [&](int total, int& first) {
      const int chunk = (total + 7) >> 3;
      first = xcd * chunk;
      const int last = (xcd + 1) * chunk < total ? (xcd + 1) * chunk : total;
      return last > first ? last - first : 0;
    };
    na = share(xt * nt, a0);
    const int routed = mt_seg * nt;
    rr = (routed / (8 * RR)) * RR;
    int n = share(routed - 8 * rr, b0);
    b0 += 8 * rr;
    n += CAT ? rr : na + rr;
    nr = n;
    full = (n / nslots) * nslots;
    rem = n - full;
    S = 1;
    if (can_split && rem > 0) {
      S = nslots / rem;
      if (S > SPLITK_MAX) S = SPLITK_MAX;
      if (S > nk) S = nk;
      if (S < 1) S = 1;
    }
    if constexpr (CAT) {
      // In units of a short tile (half the k-tiles): uncut, the last round is two units long for the
      // workgroups with a full tile, and the others do up to two short ones meanwhile; cut, the
      // parts come first and the short tiles follow the full ones.  The sum of the parts costs
      // about as much as 20 k-tiles.
      const int idle = nslots - rem;
      const int over = na > 2 * idle ? (na - 2 * idle + nslots - 1) / nslots : 0;
      if (S > 1 && (2 + over) * (nk / 2) <= nk / S + 20 + (na + nslots - 1) / nslots * (nk / 2)) S = 1;
      if (S == 1) {
        const bool second = rem > 0 && na > idle;
        hole = second ? full + nslots : 0;
        npart = 0;
        ngemm = full + na + (second ? 2 * rem : rem);
        nfin = 0;
        return;
      }
    }
    npart = S > 1 ? rem * S : 0;
    ngemm = S > 1 ? npart + full + (CAT ? na : 0) : n;
    nfin = S > 1 ? rem * FS : 0;
  }
  // the item after `it` of the same workgroup
  SCMOE_SCHED_FN int next(int it) const {
    it += nslots;
    if (CAT && hole > 0 && it >= hole && it < hole + rem) it += nslots;
    return it;
  }
  // GEMM item (it < ngemm) -> local tile index and part (part < 0: the whole tile)
  SCMOE_SCHED_FN void item(int it, int& l, int& part) const {
    if (it < npart) {
      l = full + it / S;
      part = it - (it / S) * S;
    } else {
      l = it - npart;
      if (CAT && hole > 0 && it >= hole) l -= rem;    // (past the items that do not exist)
      if (CAT && npart > 0 && l >= full) l += rem;    // (past the tiles that are cut)
      part = -1;
    }
  }
  // k-tiles kb .. kb + n - 1 of the nk of a tile are the item's (part of a tile of segment e; part < 0:
  // the whole tile).  CAT: the second half of the nk belongs to the shared expert's product, which
  // begins kmid k-tiles into the item; tiles of the last segment have that half alone, and tiles are cut at
  // even k-tiles.
  SCMOE_SCHED_FN void k_range(int e, int part, int nk, int& kb, int& n, int& kmid) const {
    kb = 0;
    n = nk;
    kmid = 0;
    if constexpr (CAT) {
      const int half = nk / 2;
      if (part >= 0) {
        kb = part * half / S * 2;
        n = (part + 1) * half / S * 2 - kb;
      } else if (e == E) {
        kb = half;
        n = half;
      }
      kmid = half - kb;
    } else if (part >= 0) {
      kb = part * nk / S;
      n = (part + 1) * nk / S - kb;
    }
  }
  // raster order inside a range of mt row tiles: tile l -> row tile, first column
  // (the fewest groups of at most GM row tiles, of sizes that differ by one at most: the first
  // `big` groups have one row tile more than the others)
  SCMOE_SCHED_FN void raster(int l, int mt, int& m, int& n0) const {
    const int ng = (mt + GM - 1) / GM;
    const int base = mt / ng, big = mt - base * ng;
    const int lbig = big * (base + 1) * nt;          // tiles in the larger groups
    int grows, first, r;
    if (l < lbig) {
      grows = base + 1;
      const int g = l / (grows * nt);
      first = g * grows;
      r = l - g * grows * nt;
    } else {
      grows = base;
      const int g = (l - lbig) / (grows * nt);
      first = big * (base + 1) + g * grows;
      r = (l - lbig) - g * grows * nt;
    }
    m = first + r % grows;
    n0 = (r / grows) * BN;
  }
  // local tile l -> expert e (E: the dense extra segment), packed rows [row0, row_end)
  // (row0 + BM may exceed row_end), column n0
  // The tiles of a workgroup come in ascending order, so the search through offsets[] goes on
  // from the expert of the previous tile (cur_e, with cur_base tiles in the experts before
  // it) instead of from expert 0: a dependent scalar load per expert passed, 2 us per tile
  // at 16 experts when started from 0 every time.
  SCMOE_SCHED_FN void locate(int l, int& e, int& row0, int& row_end, int& n0) {
    int mt;
    if constexpr (CAT) {
      if (l >= nr) {
        raster(a0 + l - nr, xt, mt, n0);
        e = E;
        row0 = offsets[E] + mt * BM;
        row_end = offsets[E] + xrows;
        return;
      }
    } else if (l < na) {
      raster(a0 + l, xt, mt, n0);
      e = E;
      row0 = mt * BM;
      row_end = xrows;
      return;
    }
    // Segment after segment, each in its own raster order: a raster group never holds rows
    // of two experts, so the workgroups that run side by side share one expert's weights.
    int t = CAT ? l : l - na;
    t = (t < rr) ? ((t / RR) * 8 + xcd) * RR + t % RR : b0 + t - rr;
    row0 = 0;
    row_end = 1;
    n0 = 0;
    if (t < cur_base) {        // not expected; start over
      cur_e = 0;
      cur_base = 0;
    }
    int base = cur_base;
    for (e = cur_e; e < E; ++e) {
      const int s = offsets[e];
      const int c = offsets[e + 1] - s;
      const int ntile = (c + BM - 1) / BM;
      if (t - base < ntile * nt) {
        raster(t - base, ntile, mt, n0);
        row0 = s + mt * BM;
        row_end = s + c;
        cur_e = e;
        cur_base = base;
        break;
      }
      base += ntile * nt;
    }
    if (e == E) e = E - 1;   // not reachable for a tile of this XCD's share
  }
};

}  // namespace scmoe
