// Walks the grouped GEMM's tile schedule as its workgroups do and checks that every tile is done
// exactly once: input lines "CAT BM nt nk split fs slots xrows E offsets[0..E]" (E = 0: no segment but the extra one; CAT: joint second GEMM, whose
// offsets hold the tokens without a routed row as the last of the E segments); for each a line "LONGEST
// TOTAL", the k-tiles of the workgroup with the most and of all, or what is wrong.
#include <stdio.h>

#include <map>
#include <tuple>
#include <vector>

#include "tile_schedule.hpp"

template <int BM, bool CAT>
static void walk(int nt, int nk, bool split, int fs, int slots, int xrows, int E, const std::vector<int32_t>& off) {
  constexpr int BN = 128;
  std::map<std::tuple<int, int, int>, std::vector<int>> seen;      // (segment, row, column) -> k-tiles done
  std::map<std::tuple<int, int, int>, int> finished, parts;
  long total = 0, longest = 0;
  for (int xcd = 0; xcd < 8; ++xcd)
    for (int slot = 0; slot < slots; ++slot) {
      scmoe::TileSchedule<BM, BN, 4, CAT> s(nt, E, off.data(), xrows, nk, split, fs, xcd, slots);
      if (s.npart > slots || (s.S > 1 && s.S > nk)) { printf("parts do not fit\n"); return; }
      long mine = 0;
      int it = slot;
      for (; it < s.ngemm; it = s.next(it)) {
        int l, part, e, r0, r1, n0;
        s.item(it, l, part);
        s.locate(l, e, r0, r1, n0);
        int kb, n, kmid;
        s.k_range(e, part, nk, kb, n, kmid);
        if (part >= 0) {
          if (it != slot || (CAT && e == E - 1)) { printf("a part is not the first item\n"); return; }
          ++parts[{e, r0, n0}];
        }
        if (CAT && (kmid != nk / 2 - kb || (part >= 0 && (kb % 2 || n % 2)))) { printf("operands change at the wrong k-tile\n"); return; }
        if (kb < 0 || kb + n > nk) { printf("k-tiles out of range\n"); return; }
        const int lo = e < E ? off[e] : 0, hi = e < E ? off[e + 1] : xrows;
        if (r0 < lo || r0 >= hi || r1 != hi || (r0 - lo) % BM || n0 < 0 || n0 >= nt * BN || n0 % BN || n < 1) { printf("a tile that is none\n"); return; }
        auto& v = seen[{e, r0, n0}];
        v.resize(nk);
        for (int k = 0; k < n; ++k) ++v[kb + k];
        mine += n;
      }
      for (; it < s.ngemm + s.nfin; it += slots) {
        int e, r0, r1, n0;
        s.locate(s.full + (it - s.ngemm) / fs, e, r0, r1, n0);
        ++finished[{e, r0, n0}];
      }
      total += mine;
      if (mine > longest) longest = mine;
    }
  size_t want = 0;
  for (int e = 0; e <= E; ++e) {
    const int rows = e < E ? off[e + 1] - off[e] : xrows;
    want += static_cast<size_t>((rows + BM - 1) / BM) * nt;
  }
  if (seen.size() != want) { printf("%zu tiles of %zu\n", seen.size(), want); return; }
  for (auto& t : seen) {
    const bool last = CAT && std::get<0>(t.first) == E - 1;
    for (int k = 0; k < nk; ++k)
      if (t.second[k] != (last && k < nk / 2 ? 0 : 1)) { printf("a k-tile done %d times\n", t.second[k]); return; }
    if (finished[t.first] != (parts.count(t.first) ? fs : 0)) { printf("a cut tile finished %d times\n", finished[t.first]); return; }
  }
  printf("%ld %ld\n", longest, total);
}

int main() {
  int cat, bm, nt, nk, split, fs, slots, xrows, E;
  while (scanf("%d %d %d %d %d %d %d %d %d", &cat, &bm, &nt, &nk, &split, &fs, &slots, &xrows, &E) == 9) {
    std::vector<int32_t> off(E + 1);
    for (auto& o : off)
      if (scanf("%d", &o) != 1) return 1;
    auto f = cat ? (bm == 256 ? walk<256, true> : walk<128, true>) : bm == 256 ? walk<256, false> : bm == 128 ? walk<128, false> : walk<64, false>;
    if (bm != 256 && bm != 128 && (cat || bm != 64)) return 1;
    f(nt, nk, split != 0, fs, slots, xrows, E, off);
  }
  return 0;
}
