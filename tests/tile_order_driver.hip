// Host-side check of the tile orders' further forms: tokens first, and contractions cut into slabs.  Built and run by
// tests/test_tile_order_cpu.py; no GPU is needed.  Every tile of every slab must be handed out exactly once, the tiles of a
// slab in one piece, and tokens first must keep a vocab tile's tiles of a panel together.
#include <cstdio>
#include <vector>
#include "../paper_2602_05885_amd/csrc/gemm_core.h"
using namespace pg;

int main() {
  int fails = 0;
  for (int tiles_m = 1; tiles_m <= 40; ++tiles_m)
    for (int tiles_n = 1; tiles_n <= 40; ++tiles_n) {
      const int total = tiles_m * tiles_n;
      std::vector<int> seen(total, 0);
      for (int b = 0; b < total + 64; ++b) {
        int tm = -1, tn = -1;
        if (!map_tile(b, tiles_m, tiles_n, tm, tn, true)) continue;
        if (tm < 0 || tm >= tiles_m || tn < 0 || tn >= tiles_n) { ++fails; continue; }
        ++seen[tm * tiles_n + tn];
        int tm1, tn1;      // the XCD's next tile: the same vocab tile until its panel is through
        if (map_tile(b + 8, tiles_m, tiles_n, tm1, tn1, true) && (tn + 1) % SB_N != 0 && tn + 1 < tiles_n) fails += tm1 != tm || tn1 != tn + 1;
      }
      for (int v : seen) fails += v != 1;
      for (int slabs : {1, 2, 3, 7, 24}) {
        std::vector<int> out((size_t)total * slabs, 0);
        for (int b = 0; b < total * slabs + 64; ++b) {
          int tm = -1, tn = -1, slab = -1;
          if (!map_tile_interleaved(b, tiles_m, tiles_n, slabs, slab, tm, tn)) continue;
          if (slab < 0 || slab >= slabs || tm < 0 || tm >= tiles_m || tn < 0 || tn >= tiles_n) { ++fails; continue; }
          ++out[(size_t)slab * total + tm * tiles_n + tn];
        }
        for (int v : out) fails += v != 1;
      }
    }
  for (int rows = 1; rows <= 256; ++rows)      // the forward's short tiles cover their rows
    for (int tiles_t = 1; tiles_t <= 4; ++tiles_t) {
      const int nj = fwd_nj(rows, tiles_t);
      fails += (nj != 4 && nj != 6 && nj != 8) || nj * 32 < (rows + BK - 1) / BK * BK;
    }
  // Entries dealt by workgroup index and tickets behind them: together every entry of every share once.
  for (int grid : {8, 64, 256})
    for (int total = 1; total <= 1200; total += 7)
      for (int order = 0; order < 2; ++order)
        for (int rounds = 1; rounds <= 2; ++rounds) {
          if (grid < 256 && total > grid * 4) continue;
          TileQueue Q{};
          Q.total = total; Q.interleaved = order; Q.dealt = rounds * (grid >> 3);
          long long handed = 0;
          for (int b = 0; b < grid; ++b)
            for (int r = 0; r < rounds; ++r) handed += (b >> 3) + r * (grid >> 3) < Q.share(b & 7);
          for (int y = 0; y < 8; ++y) handed += imax(Q.share(y) - Q.dealt, 0);
          fails += handed != total;
          if (total <= grid && rounds == 1)
            for (int y = 0; y < 8; ++y) fails += Q.share(y) > Q.dealt;      // nothing is left for the counters
        }
  // The forward's two entries each: with few more tiles than workgroups, as few workgroups as that takes have any.
  for (int grid : {8, 64, 256})
    for (int total = grid + 1; total <= grid + grid * 9 / 16; ++total) {
      TileQueue Q{};
      Q.total = total;
      Q.deal(grid, 2);
      std::vector<int> seen((size_t)total + 64, 0);
      int busy = 0;
      for (int b = 0; b < grid; ++b) {
        busy += Q.entry(b, 0) >= 0;
        for (int r = 0; r < 2; ++r) {
          const int e = Q.entry(b, r);
          int tm, tn;
          if (e >= 0 && map_tile(e, total, 1, tm, tn)) ++seen[tm];
          else fails += e >= 0;
        }
      }
      for (int t = 0; t < total; ++t) fails += seen[t] != 1;
      fails += busy > (total + 1) / 2 + 8;
    }
  printf("tile order driver: (%d failures)\n", fails);
  return fails != 0;
}
