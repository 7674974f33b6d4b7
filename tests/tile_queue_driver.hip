// Host-side check of the tile orders and of the per-XCD queue shares of the persistent kernels.  Built and
// run by tests/test_tile_queue_cpu.py; no GPU is needed (nothing here calls the HIP runtime).
// For every tile count swept and both orders: the entries i < share(y) of the 8 XCDs, decoded with the
// order's map, hand out every tile (tm, tn) exactly once; entries at and beyond share(y) map to no tile;
// 32 consecutive entries of one XCD form a block of at most 4 x 8 neighbouring tiles (what the L2 sharing
// relies on); tiles of 320 rows stay within the range of their loads; the parts of a dH
// launch (dh_form) stay inside the accumulator and are the least of its model; dw_split's parts are no shorter than its least; token blocks cut the live tiles without a gap or an overlap; and the kept tiles fit their region.
#include <cstdio>
#include <vector>
#include "../paper_2602_05885_amd/csrc/gemm_core.h"
#include "../paper_2602_05885_amd/csrc/kernels.h"
using namespace pg;

static int fails = 0;
#define CHECK(cond, ...) do { if (!(cond)) { if (fails < 20) { printf("FAIL line %d: ", __LINE__); printf(__VA_ARGS__); printf("\n"); } ++fails; } } while (0)

static void sweep(int tiles_m, int tiles_n, int interleaved) {
  TileQueue Q{};
  Q.total = tiles_m * tiles_n; Q.interleaved = interleaved;
  std::vector<int> seen((size_t)Q.total, 0);
  int sum = 0;
  for (int y = 0; y < 8; ++y) {
    const int n = Q.share(y);
    sum += n;
    for (int i = 0; i < n + 3; ++i) {
      int tm = -1, tn = -1;
      const int b = TileQueue::encode(y, i);
      const bool ok = interleaved ? map_tile_interleaved(b, tiles_m, tiles_n, tm, tn) : map_tile(b, tiles_m, tiles_n, tm, tn);
      if (i >= n) { CHECK(!ok, "%dx%d order %d: entry %d of XCD %d beyond its share %d maps to a tile", tiles_m, tiles_n, interleaved, i, y, n); continue; }
      CHECK(ok && tm >= 0 && tm < tiles_m && tn >= 0 && tn < tiles_n, "%dx%d order %d: entry %d of XCD %d -> (%d, %d)", tiles_m, tiles_n, interleaved, i, y, tm, tn);
      if (ok && tm >= 0 && tm < tiles_m && tn >= 0 && tn < tiles_n) ++seen[(size_t)tm * tiles_n + tn];
    }
  }
  CHECK(sum == Q.total, "%dx%d order %d: shares add up to %d of %d", tiles_m, tiles_n, interleaved, sum, Q.total);
  for (int t = 0; t < Q.total; ++t) CHECK(seen[t] == 1, "%dx%d order %d: tile %d handed out %d times", tiles_m, tiles_n, interleaved, t, seen[t]);
  // blocks: entries 32 r .. 32 r + 31 of an XCD span at most 4 tile rows and 8 tile columns
  for (int y = 0; y < 8; ++y)
    for (int i0 = 0; i0 + 32 <= Q.share(y); i0 += 32) {
      int m0 = 1 << 30, m1 = -1, n0 = 1 << 30, n1 = -1;
      for (int i = i0; i < i0 + 32; ++i) {
        int tm, tn;
        if (interleaved) map_tile_interleaved(TileQueue::encode(y, i), tiles_m, tiles_n, tm, tn);
        else map_tile(TileQueue::encode(y, i), tiles_m, tiles_n, tm, tn);
        m0 = imin(m0, tm); m1 = imax(m1, tm); n0 = imin(n0, tn); n1 = imax(n1, tn);
      }
      // a block of the contiguous order may straddle two blocks of the flattened order (its range need not
      // start on a multiple of 32), and ragged edges make blocks narrower and longer: bound the area instead
      if (interleaved && tiles_m % 4 == 0 && tiles_n % 8 == 0 && i0 + 32 <= (Q.total / 256) * 32)
        CHECK(m1 - m0 < 4 && n1 - n0 < 8, "%dx%d: block %d of XCD %d spans %d x %d tiles", tiles_m, tiles_n, i0 / 32, y, m1 - m0 + 1, n1 - n0 + 1);
    }
}

// The parts of dh_parts, tried one after the other.
static int least_parts_of(long long tiles, int n_pad, int acc_rows, int stages) {
  int few = 1;             // up to eight: the least modelled rounds, the fewest parts among equals
  long long least = 0;
  for (int q = 1; q <= 8 && (q == 1 || ((long long)q * n_pad <= acc_rows && q * 8 <= stages)); ++q) {
    const long long cost = (tiles * q + 255) / 256 * ((stages + q - 1) / q + 24);
    if (q == 1 || cost < least) { few = q; least = cost; }
  }
  int best = few;          // of few tiles: the least rounds and slabs
  for (int q = few; q <= 64; ++q) {
    if (q > few && (q * tiles > 256 || (long long)q * n_pad > acc_rows || q * 4 > stages)) break;
    const long long cost = (tiles * q + 255) / 256 * 256 * ((stages + q - 1) / q + 24) + tiles * q * 16;
    if (q == few || cost < least) { best = q; least = cost; }
  }
  return best;
}

// Every form of a dH launch: the slabs fit the accumulator, the parts are what the rule says and long enough, fp32 products side by side fit one round, the
// parts' stages follow on each other, and every tile of every slab is handed out once.
static void sweep_dh_forms() {
  int most = 0, wide = 0, wide_many = 0, three = 0, in_turn_fit = 0;
  for (int n_pad : {256, 512, 768, 1024, 1536, 2048, 3072, 5120, 8192, 12288, 16640, 32768, 65536})
    for (int acc_rows : {n_pad, 2 * n_pad, 3 * n_pad + 100, 9 * n_pad, 32768, 60 * 256 + 77})
      for (int n : {64, 256, 320, 576, 1024, 1088, 1600, 2560, 4096, 5120, 8192})
        for (int stages : {1, 4, 8, 31, 44, 63, 104, 356, 1023, 2376})
          for (int f32 = 0; f32 < 2; ++f32)
            for (int wide_ok = 0; wide_ok < 2; ++wide_ok) {
              if (acc_rows < n_pad) continue;
              const DhForm f = dh_form(n_pad, acc_rows, n, stages, f32, wide_ok);
              const int slabs = f.ks * f.products, tiles_m = n_pad / 256, tiles_n = store_tiles_n(n, f.wide);
              const long long tiles = (long long)tiles_m * tiles_n;
#define AT "dh_form(%d, %d, %d, %d, %d, %d) = %d parts, %d products, wide %d: "
#define FORM n_pad, acc_rows, n, stages, f32, wide_ok, f.ks, f.products, f.wide
              CHECK((long long)slabs * n_pad <= acc_rows, AT "beyond the accumulator", FORM);
              CHECK(f.ks >= 1 && f.ks <= DH_PARTS_MAX && f.ks <= imax(SPLIT_MAX, stages / DH_MIN_STAGES) && (f.ks == 1 || f.ks * DH_MIN_STAGES <= stages), AT "parts too short", FORM);
              CHECK(f.ks <= SPLIT_MAX || tiles * slabs <= 256, AT "more than one round", FORM);
              CHECK(f.products == 1 || (f.products == 3 && f32 && tiles * slabs <= 256), AT "products", FORM);
              CHECK(!f.wide || (wide_ok && !f32), AT "wide", FORM);
              CHECK(f.ks == (f.products == 3 ? least_parts_of(3 * tiles, n_pad, acc_rows / 3, stages) : least_parts_of(tiles, n_pad, acc_rows, stages)), AT "not the least", FORM);
              if (f32) {         // products in turn or side by side: the shorter one
                const int k1 = least_parts_of(tiles, n_pad, acc_rows, stages), k3 = least_parts_of(3 * tiles, n_pad, acc_rows / 3, stages);
                const bool fit = 3 * k3 * tiles <= 256 && 3ll * k3 * n_pad <= acc_rows;
                const long long in_turn = (tiles * k1 + 255) / 256 * 256 * (3ll * ((stages + k1 - 1) / k1) + 36) + tiles * k1 * 16;
                const long long beside = 256ll * ((stages + k3 - 1) / k3 + 24) + 3 * tiles * k3 * 16;
                CHECK(f.products == (fit && beside < in_turn ? 3 : 1), AT "%lld in turn, %lld side by side", FORM, in_turn, beside);
                in_turn_fit += fit && f.products == 1;
              }
              int at = 0;        // the parts of gemm_store_tile
              for (int p = 0; p < f.ks; ++p) {
                const int s0 = (int)((unsigned)p * (unsigned)stages / (unsigned)f.ks), s1 = (int)((unsigned)(p + 1) * (unsigned)stages / (unsigned)f.ks);
                CHECK(s0 == at && s1 >= s0, AT "part %d is stages %d .. %d", FORM, p, s0, s1);
                at = s1;
              }
              CHECK(at == stages, AT "the parts end at stage %d", FORM, at);
              most = imax(most, f.ks); wide += f.wide; wide_many += f.wide && f.ks > SPLIT_MAX; three += f.products == 3;
              if (slabs == 1 || (n_pad + n + stages + f32) % 3) continue;       // (the orders of one slab: sweep())
              TileQueue Q{};
              Q.total = (int)tiles * slabs; Q.interleaved = 1;
              std::vector<int> seen((size_t)Q.total, 0);
              for (int y = 0; y < 8; ++y)
                for (int i = 0; i < Q.share(y); ++i) {
                  int slab = -1, tm = -1, tn = -1;
                  if (map_tile_interleaved(TileQueue::encode(y, i), tiles_m, tiles_n, slabs, slab, tm, tn) && slab >= 0 && slab < slabs && tm >= 0 && tm < tiles_m && tn >= 0 && tn < tiles_n)
                    ++seen[((size_t)slab * tiles_m + tm) * tiles_n + tn];
                }
              for (int t = 0; t < Q.total; ++t) CHECK(seen[t] == 1, AT "tile %d handed out %d times", FORM, t, seen[t]);
            }
  CHECK(most == DH_PARTS_MAX && wide > 0 && wide_many > 0 && three > 0 && in_turn_fit > 0,
        "the sweep reaches %d parts, %d wide forms (%d of many parts), %d of three products, %d of one where three fit", most, wide, wide_many, three, in_turn_fit);
}

// The forms of a list (n_pad acc_rows n stages f32 wide_ok a line), for the tests' restatement of the rule.
static int print_forms() {
  int n_pad, acc_rows, n, stages, f32, wide_ok;
  while (scanf("%d %d %d %d %d %d", &n_pad, &acc_rows, &n, &stages, &f32, &wide_ok) == 6) {
    const DhForm f = dh_form(n_pad, acc_rows, n, stages, f32, wide_ok);
    printf("%d %d %d\n", f.ks, f.products, f.wide);
  }
  return 0;
}

int main(int argc, char**) {
  if (argc > 1) return print_forms();
  for (int tm = 1; tm <= 70; ++tm)
    for (int tn = 1; tn <= 45; ++tn)
      for (int order = 0; order < 2; ++order) sweep(tm, tn, order);
  for (int order = 0; order < 2; ++order) {     // the shapes the 14B head produces
    sweep(594, 128, order); sweep(89, 20, order); sweep(128, 20, order); sweep(60, 20, order); sweep(594, 512, order);
  }
  sweep_dh_forms();
  // Wide tiles only where 320 rows of the operand lie below 4 GiB; what the calls accept has 256 of them there.
  int wide_near = 0, wide_far = 0;
  for (long long V : {25600ll, 2000000ll, 6710000ll, 6711000ll, 7000000ll, 8388000ll}) {
    const long long ld = pad_ld((V + 255) / 256 * 256);
    if (ld * 2 * 256 >= 1ll << 32) { CHECK(false, "V = %lld is not accepted", V); continue; }
    for (int d : {320, 640, 1600, 5120})
      for (int rows : {256, 2048, 8192, 20224, 65536})
        for (int chunk : {4, 512, 16384}) {
          const int acc_rows = imax(rows, imin(8 * rows, 32768)), stages = 4 * chunk;
          const DhForm f = dh_form(rows, acc_rows, d, stages, 0, wide_fits(ld));
          (ld * 2 * WIDE_ROWS < 1ll << 32 ? wide_near : wide_far) += f.wide;
          CHECK(f.wide == (wide_fits(ld) && dh_form(rows, acc_rows, d, stages, 0, true).wide), "dh_form(%d, %d, %d, %d)", rows, acc_rows, d, stages);
        }
  }
  CHECK(wide_near > 0 && wide_far == 0, "wide tiles: %d within their range, %d beyond", wide_near, wide_far);
  for (int stages = 0; stages <= 300; ++stages)
    for (int cap = 1; cap <= DW_SPLIT_MAX; ++cap) {
      const int ks = dw_split(stages, cap);
      CHECK(ks >= 1 && ks <= cap && (ks == 1 || stages / ks >= DW_MIN_STAGES) && (ks == cap || (ks + 1) * DW_MIN_STAGES > stages),
            "dw_split(%d, %d) = %d", stages, cap, ks);
      int at = 0;       // the parts of gemm_store_tile
      for (int p = 0; p < ks; ++p) {
        const int s0 = (int)((long long)p * stages / ks), s1 = (int)((long long)(p + 1) * stages / ks);
        CHECK(s0 == at && s1 >= s0 && (ks == 1 || s1 - s0 >= DW_MIN_STAGES), "part %d of %d: stages %d .. %d of %d", p, ks, s0, s1, stages);
        at = s1;
      }
      CHECK(at == stages, "%d parts end at stage %d of %d", ks, at, stages);
    }
  for (int host_tiles = 1; host_tiles <= 80; ++host_tiles)        // what the host launches: blocks for all of its tiles
    for (int cap_t = 0; cap_t <= 40; ++cap_t) {
      const int nblocks = cap_t ? (host_tiles + cap_t - 1) / cap_t : 1;
      for (int live = 0; live <= host_tiles; ++live) {
        int at = 0;
        for (int b = 0; b < nblocks; ++b) {
          int t0 = -1, nt = -1;
          token_block(TokenBlocks{cap_t, b}, live, t0, nt);
          CHECK(t0 == at && nt >= 0 && (!cap_t || nt <= cap_t) && (nt == cap_t || t0 + nt == live),
                "block %d of %d (cap %d): tiles %d + %d of %d", b, nblocks, cap_t, t0, nt, live);
          at = t0 + nt;
        }
        CHECK(at == live, "%d blocks of %d end at tile %d of %d", nblocks, cap_t, at, live);
      }
    }
  float region = 0.f;
  for (int cap : {0, 1, 47, 48, 594, 38016, 39936})
    for (int tiles_v : {1, 2, 75, 594, 2000})
      for (int live = 0; live <= 200; ++live) {
        const int n = kept_vocab_tiles(Kept{&region, cap}, tiles_v, live);
        CHECK(n >= 0 && n <= tiles_v && (long long)n * live <= cap && (live == 0 ? n == 0 : n == tiles_v || (long long)(n + 1) * live > cap),
              "kept_vocab_tiles(%d, %d, %d) = %d", cap, tiles_v, live, n);
        CHECK(kept_vocab_tiles(Kept{nullptr, cap}, tiles_v, live) == 0, "nothing is kept without a region");
      }
  printf(fails ? "tile queue driver: %d FAILED\n" : "tile queue driver: every tile handed out exactly once (%d failures)\n", fails);
  return fails != 0;
}
