// Host-side check of the tile orders' further forms: tokens first, and contractions cut into slabs.  Built and run by
// tests/test_tile_order_cpu.py; no GPU is needed.  Every tile of every slab must be handed out exactly once, the tiles of a
// slab in one piece, tokens first must keep a vocab tile's tiles of a panel together, and the queue must hand out every entry once.
#include <cstdio>
#include <vector>
#include "../paper_2602_05885_amd/csrc/gemm_core.h"
using namespace pg;

// A launch of the persistent kernels' protocol on the host: the queue's own arithmetic (deal, entry, resolve), host counters, and the
// workgroups' steps in a random order.  A step is what happens between two accesses to the counters: a workgroup draws a ticket while
// it works on a tile and resolves it later.  forward: two entries each in advance (of more tiles than workgroups), a third claimed under
// the first.  homes: the XCD a workgroup runs on is the one of its index (0), another one (1), the same for all (2).
// Returns how many entries were not handed out exactly once, plus those that do not exist.
static int run_launch(int grid, int total, int order, int forward, int homes, unsigned seed) {
  unsigned cnt[8] = {};
  std::vector<int> given((size_t)8 * (total + 8), 0);
  auto drawn = [&](int y) { return cnt[y]; };
  auto draw = [&](int y) { return cnt[y]++; };
  struct Workgroup {
    TileQueue q{};
    int cur = -1, nxt = -1, state = 0;       // 0 starts, 1 works on cur, 2 has drawn a ticket, 3 has left
    bool two = false, dealt = false;
    unsigned ticket = 0;
  };
  std::vector<Workgroup> w(grid);
  std::vector<int> live(grid);
  int wrong = 0;
  for (int b = 0; b < grid; ++b) {
    live[b] = b;
    TileQueue& q = w[b].q;
    q.total = total; q.interleaved = order;
    w[b].two = forward && total > grid;
    q.deal(grid, w[b].two ? 2 : 1, forward != 2);
    q.home = homes == 0 ? b & 7 : homes == 1 ? (b * 5 + 3) >> 2 & 7 : 2;
    w[b].dealt = total <= (forward ? 2 : 1) * grid;       // nothing beside the dealt entries
  }
  auto take = [&](int e) {
    if (e < 0 || (e >> 3) >= w[0].q.share(e & 7)) ++wrong;
    else ++given[(size_t)(e & 7) * (total + 8) + (e >> 3)];
  };
  while (!live.empty()) {
    seed = seed * 1664525u + 1013904223u;
    const size_t at = (seed >> 8) % live.size();
    const int b = live[at];
    Workgroup& g = w[b];
    if (g.state == 0) {
      g.cur = g.q.entry(b, 0);
      g.nxt = g.two ? g.q.entry(b, 1) : -1;
      if (!g.dealt && (g.cur < 0 || (forward && g.nxt < 0))) {
        if (g.cur < 0) g.cur = g.q.resolve(draw(g.q.home), true, drawn, draw);
        if (forward) g.nxt = g.q.resolve(draw(g.q.home), true, drawn, draw);
      }
      g.state = g.cur < 0 ? 3 : 1;
    } else if (g.state == 1) {
      take(g.cur);
      const bool more = forward ? g.nxt >= 0 : !g.dealt;
      if (more) g.ticket = draw(g.q.home);
      g.state = more ? 2 : 3;
    } else {
      const int e = g.q.resolve(g.ticket, true, drawn, draw);
      g.cur = forward ? g.nxt : e;
      g.nxt = forward ? e : -1;
      g.state = g.cur < 0 ? 3 : 1;
    }
    if (g.state == 3) { live[at] = live.back(); live.pop_back(); }
  }
  for (int y = 0; y < 8; ++y)
    for (int i = 0; i < w[0].q.share(y); ++i) wrong += given[(size_t)y * (total + 8) + i] != 1;
  return wrong;
}

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
  // Entries dealt by workgroup index, tickets behind them, stolen ones: every entry once, in whatever order the workgroups get on.
  unsigned seed = 1;
  for (int grid : {8, 64, 256})
    for (int order = 0; order < 2; ++order)
      for (int forward = 0; forward < 3; ++forward)      // (2: two tiles each for everybody)
        for (int homes = 0; homes < 3; ++homes)
          for (int total = 1; total <= 5 * grid; total += 1 + (grid > 8) * (int)((seed >> 8) % 23)) {
            seed = seed * 1664525u + 1013904223u;
            const int wrong = run_launch(grid, total, order, forward, homes, seed);
            if (wrong && fails < 20) printf("grid %d total %d order %d forward %d homes %d: %d wrong\n", grid, total, order, forward, homes, wrong);
            fails += wrong;
          }
  // The forward's two entries each: with few more tiles than workgroups, as few workgroups as that takes have any, where it asks for that.
  for (int grid : {8, 64, 256})
    for (int total = grid + 1; total <= grid + grid * 9 / 16; ++total) {
      TileQueue Q{};
      Q.total = total;
      Q.deal(grid, 2, true);
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
