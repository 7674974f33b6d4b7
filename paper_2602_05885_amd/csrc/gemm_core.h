// 256x256x64 bf16 MFMA tile engine for gfx950 (CDNA4), shared by the three contractions
// of the policy-gradient head (dW and dH also in tiles of 320x256x64, see mainloop):
//   logits^T = W H^T        (forward statistics, and the backward's recompute)
//   dW       = dS^T H
//   dH       = dS W
// Every contraction is brought to the form C[m,n] = sum_k A[m,k] B[n,k] with both
// operands k-contiguous in memory, so one main loop serves all of them.
//
// Shape of the engine (each choice measured on MI355X):
//   * 8 wavefronts per workgroup as 4 (m) x 2 (n), two per SIMD, each owning a 64 x 128 block
//     = 4 x 8 MFMA 16x16x32 tiles (128 fp32 accumulators per lane; 80 x 128 = 5 x 8 tiles, 160
//     accumulators, in the wide form).  Two wavefronts per SIMD
//     hide each other's LDS and barrier latency; one wavefront per SIMD with a 128 x 128 block
//     was 30 % slower with compiler-scheduled code.
//   * v_mfma_f32_16x16x32_bf16 rather than 32x32x16: same LDS traffic per flop, half the
//     accumulator traffic; the chip is power-limited under MFMA load and sustains a higher
//     clock with it (+6 % end to end, +13 % on a pure MFMA stream).
//   * operand slabs go global -> LDS directly (buffer_load ... lds, 16 B per lane), two
//     64-deep stages of 64 KiB (72 wide).
//   * a wavefront that issues a burst of such loads is held at the issue stage while the
//     texture-address unit works through them (16 cycles per 1 KiB load, 64 loads per stage), and
//     its MFMAs wait behind them.  The loads are therefore trickled out one per 64-cycle step over
//     the whole stage, which a two-barrier stage schedule makes legal: the A slab of a stage is
//     dead once the register-resident A fragments have been read (barrier X after step 4, 5 wide), the
//     B slab once the last streamed B fragment has been read (barrier Y, two steps before the end
//     of the stage).  Measured +10..13 % over issuing a stage's loads in one burst.
//   * inside a stage the LDS->register traffic is software-pipelined by hand (A fragments
//     resident, B fragments streamed two steps ahead, the first fragments of the next stage
//     fetched behind barrier Y under the last two steps' MFMAs) and pinned with sched_barrier.
//   * the M side of the MFMA is the "vocab-like" operand, so a lane's accumulators of one
//     MFMA tile share one n (token): row statistics over the vocabulary reduce inside a lane
//     first, then across the four 16-lane groups, then across wavefronts through LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pg {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int BM = 256;           // tile rows   (A rows)
constexpr int BN = 256;           // tile cols   (B rows)
constexpr int BK = 64;            // k-slab per pipeline stage
constexpr int WM = 4, WN = 2;     // wavefront grid
constexpr int NW = WM * WN;
constexpr int NTHREADS = NW * 64;
constexpr int WROWS = BM / WM;    // 64 rows per wavefront
constexpr int WCOLS = BN / WN;    // 128 cols per wavefront
constexpr int GM = WROWS / 16;    // 4 MFMA tiles along m
constexpr int GN = WCOLS / 16;    // 8 MFMA tiles along n
constexpr int SLAB_BYTES = BM * BK * 2;          // one operand slab: 256 rows x 128 B
constexpr int STAGE_BYTES = 2 * SLAB_BYTES;      // A slab + B slab
constexpr int CHUNKS = 32 / NW;                  // direct loads per wavefront per slab (1 KiB each)
// Epilogue staging rows (256 bf16 + pad).  The pad makes the lanes of a half-wavefront hit distinct
// banks: rows written 16 at a time with 8-byte elements want a row pitch of 4 banks (mod 64),
// rows written 8 at a time with 32 bytes per row want 8 banks.
constexpr int EPI_STRIDE = 528;                  // 132 dwords
constexpr int EPI_STRIDE_T = 544;                // 136 dwords
constexpr int GEMM_LDS_BYTES = 256 * EPI_STRIDE_T; // 136 KiB >= the 128 KiB double-buffered main loop
constexpr int GW = 5;             // MFMA tiles along m per wavefront in wide tiles
constexpr int WIDE_ROWS = 64 * GW, WIDE_LDS_BYTES = 2 * (WIDE_ROWS * BK * 2 + SLAB_BYTES);
static_assert(GEMM_LDS_BYTES >= 2 * STAGE_BYTES, "LDS budget");
static_assert(GM == 4 && GN == 8, "the main loop's schedule is written for 4 x 8 MFMA tiles per wavefront");

// ---- control block written by the row-compaction kernel, the dH form by the combine (device memory) ----
struct Ctl {
  int n_active;   // number of compacted rows
  int n_pad;      // n_active rounded up to a multiple of 256
  float norm;     // loss normaliser
  unsigned step[8]; // of the workgroups of every XCD in a forward (InStep), zero at launch
  int dh_slabs;   // slabs of the dH accumulator: the scatter adds that many
  int dh_ks, dh_products, dh_wide;      // of the dH launches (DhForm)
};

// ---- workgroup -> tile mapping -------------------------------------------------
// Workgroups are dealt round-robin to the 8 XCDs, each with a private L2.  The flattened tile
// order (panels of n-tiles; inside a panel, groups of 4 m-tiles, so 32 consecutive tiles form
// a 4 x 8 block whose A slabs are shared by 8 and B slabs by 4 workgroups) is cut into 8 equal
// contiguous ranges, one per XCD: the 32 workgroups resident on an XCD work on one such block
// out of that XCD's L2, and every XCD gets the same number of tiles to within one.
constexpr int SB_M = 4, SB_N = 8;

__host__ __device__ inline int grid_for_tiles(int tiles_m, int tiles_n) {
  const int total = tiles_m * tiles_n;
  return ((total + 7) / 8) * 8;
}

// (host-callable too, like the queue's share() below: a host test sweeps them over tile counts and checks
// that every tile is handed out exactly once)
__host__ __device__ constexpr int imin(int a, int b) { return a < b ? a : b; }
__host__ __device__ constexpr int imax(int a, int b) { return a > b ? a : b; }

// Entry t of the flattened order: panels of `width` n-tiles, inside a panel groups of SB_M m-tiles with m running fastest, or
// (n_first) one m-tile after the other.  A block of 32 is 4 x 8 tiles either way; what differs is which operand is asked for by
// workgroups that start close in time, and so is still in the 4 MiB L2 when the last of them gets to it.
__host__ __device__ inline void flat_tile(int t, int tiles_m, int tiles_n, int width, bool n_first, int& tm, int& tn) {
  const int panel_tiles = width * tiles_m;
  const int p = t / panel_tiles;
  const int w = imin(width, tiles_n - p * width);
  const int idx = t - p * panel_tiles;
  if (n_first) {
    tm = idx / w;
    tn = p * width + (idx - tm * w);
    return;
  }
  const int mg = idx / (SB_M * w);
  const int rig = imin(SB_M, tiles_m - mg * SB_M);
  const int rem = idx - mg * SB_M * w;
  tm = mg * SB_M + rem % rig;
  tn = p * width + rem / rig;
}

// (a panel is SB_N token tiles wide)
__host__ __device__ inline bool map_tile(int bid, int tiles_m, int tiles_n, int& tm, int& tn, bool n_first = false) {
  const int total = tiles_m * tiles_n;   // may be smaller than what the grid was sized for
  const int per = (total + 7) / 8;
  const int xcd = bid & 7, q = bid >> 3;
  const int t = xcd * per + q;
  if (q >= per || t >= total) return false;
  flat_tile(t, tiles_m, tiles_n, SB_N, n_first, tm, tn);
  return true;
}

// The same flattened order dealt to the XCDs in units of 32 consecutive tiles (one 4 x 8 block):
// the eight XCDs then work on eight neighbouring blocks of one n-panel at the same time and the
// panel's B slabs are fetched from HBM once for all of them (they meet in the memory-side cache).
// The last (< 256) tiles are split evenly.  Pays when the n-panel (B rows x K) is too large to
// stay cached while an XCD walks the whole M extent on its own: measured +1..3 % on the dW and
// dH contractions, -1.5 % on the logits contraction (whose token panels do stay cached).
// d <= 8192 is one panel: with panels of 8, dW and dH of d = 4096, 2869 rows took 1.4 to 2.3 % longer, of d = 5120, 12000 rows 2.0 % (loss calls of
// 2869 rows 8.85 -> 8.99 ms, 4100 rows 12.95 -> 13.03, 32768 rows of d = 5120 the same).
// A contraction cut into `slabs` parts has the tiles of one part after those of the other (parts share no operand): dH of
// 675 rows, d = 5120, 3.5 -> 2.8 GB read, 630 -> 570 us.
constexpr int STORE_PANEL = 32;
__host__ __device__ inline bool map_tile_interleaved(int bid, int tiles_m, int tiles_n, int slabs, int& slab, int& tm, int& tn) {
  const int per_slab = tiles_m * tiles_n, total = per_slab * slabs;
  const int full = (total / 256) * 256;
  const int xcd = bid & 7, q = bid >> 3;
  int t;
  if (q < full / 8) {
    t = ((q >> 5) * 8 + xcd) * 32 + (q & 31);
  } else {
    const int rem = total - full, per = (rem + 7) / 8, qq = q - full / 8;
    t = full + xcd * per + qq;
    if (qq >= per || t >= total) return false;
  }
  slab = 0;
  if (slabs > 1) {
    slab = t / per_slab;
    t -= slab * per_slab;
  }
  flat_tile(t, tiles_m, tiles_n, STORE_PANEL, false, tm, tn);
  return true;
}
__host__ __device__ inline bool map_tile_interleaved(int bid, int tiles_m, int tiles_n, int& tm, int& tn) {
  int slab;
  return map_tile_interleaved(bid, tiles_m, tiles_n, 1, slab, tm, tn);
}

// Split-K factor of the dH contraction.  Its row extent is the padded number of active tokens, known only on
// the device, and its contraction (a vocab chunk) is long: with few rows one tile per compute unit leaves most
// of the chip idle, with a few more the second round of tiles is nearly empty.  The contraction length is
// therefore cut into ks parts that run side by side.  Part p accumulates into its own slab of n_pad rows of
// the [acc_rows, d] accumulator (so ks n_pad <= acc_rows), and the final scatter adds the slabs in order.
// ks minimises the modelled time of the launch, in stages: rounds of 256 tiles, each as long as a part plus
// SPLIT_TILE_STAGES for what a tile costs beside its main loop (cold start, accumulator read and write, the
// slab's extra pass in the scatter).  Measured at V = 151936 (one chunk, 2376 stages), dH launch alone:
//   768 rows, d = 5120 (60 tiles)     one part 1466 us, 4 parts 579 us
//   3072 rows, d = 4096 (192 tiles)   one part 3167 us, 4 parts 2479 us
// (Up to 8 parts; dh_parts has more for few tiles.)
// The values that it goes by (k_stages: those of the first chunk, for all chunks) are the same for every launch of a call, so the decomposition, and with it the
// summation order, is fixed for given inputs.  A wavefront of the combine settles it, beside the rows' epilogue, and leaves it in Ctl for the dH launches and the
// scatter.
constexpr int SPLIT_MAX = 8, SPLIT_MIN_STAGES = 8, SPLIT_TILE_STAGES = 24, DH_PARTS_MAX = 64;
struct Parts { int ks, stages; };       // parts, and stages of the longest

// The numbers of parts, 1 .. MAX, are tried side by side, one in each lane (whole wavefronts only; on the host one after the other): the least cost(parts,
// stages), the fewest among equals.  (A division by a variable is a sequence of 25 instructions: one number after the other the search took longer than the
// combine that it is to run beside.)
constexpr unsigned long long NO_PARTS = ~0ull >> 6;
#ifdef __HIP_DEVICE_COMPILE__
template <int CTRL> __device__ __forceinline__ unsigned long long least_of_pair(unsigned long long x) {
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)x, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(x >> 32), CTRL, 0xf, 0xf, true);
  const unsigned long long y = (unsigned long long)hi << 32 | lo;
  return y < x ? y : x;
}
__device__ __forceinline__ unsigned long long of_lane(unsigned long long x, int lane) {
  return (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(x >> 32), lane) << 32 | (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, lane);
}
#endif
template <int MAX, class Cost>
__host__ __device__ inline Parts least_parts(int k_stages, Cost&& cost) {
  static_assert(MAX == 8 || MAX == 64, "lanes");
#ifdef __HIP_DEVICE_COMPILE__
  const int ks = (int)(threadIdx.x & 63) + 1, stages = (k_stages + ks - 1) / ks;
  unsigned long long key = cost(ks, stages) << 6 | (unsigned)(ks - 1);
  key = least_of_pair<0xB1>(key);          // lane ^ 1
  key = least_of_pair<0x4E>(key);          // lane ^ 2
  key = least_of_pair<0x141>(key);         // mirrored among 8
  unsigned long long least = of_lane(key, 0);
  if (MAX > 8) {
    key = least_of_pair<0x140>(key);       // mirrored among 16
    least = of_lane(key, 0);
#pragma unroll
    for (int lane = 16; lane < 64; lane += 16) {
      const unsigned long long k = of_lane(key, lane);
      least = k < least ? k : least;
    }
  }
  const int at = (int)(least & 63);
  return Parts{at + 1, __builtin_amdgcn_readlane(stages, at)};
#else
  unsigned long long least = ~0ull;
  for (int ks = 1; ks <= MAX; ++ks) {
    const unsigned long long key = cost(ks, (k_stages + ks - 1) / ks) << 6 | (unsigned)(ks - 1);
    least = key < least ? key : least;
  }
  const int ks = (int)(least & 63) + 1;
  return Parts{ks, (k_stages + ks - 1) / ks};
#endif
}
__host__ __device__ inline Parts dh_split(int n_pad, int acc_rows, int tiles_n, int k_stages) {
  if (n_pad <= 0 || 2ll * n_pad > acc_rows || 2 * SPLIT_MIN_STAGES > k_stages) return Parts{1, k_stages};
  const long long tiles = (long long)(n_pad / 256) * tiles_n;
  return least_parts<SPLIT_MAX>(k_stages, [&](int ks, int stages) -> unsigned long long {
    if (ks > 1 && ((long long)ks * n_pad > acc_rows || ks * SPLIT_MIN_STAGES > k_stages)) return NO_PARTS;
    return (unsigned long long)((tiles * ks + 255) / 256) * (unsigned)(stages + SPLIT_TILE_STAGES);
  });
}

// fp32 heads add three products per contraction (A B, A B_lo, A_lo B).  Where the parts of a launch leave room for it,
// each product is a part of its own, with its own slab, instead of three passes one after the other.
__host__ __device__ inline int split_products(int split_f32, int tiles, int ks, long long slab_rows, long long acc_rows) {
  return split_f32 && 3 * ks * tiles <= 256 && 3 * ks * slab_rows <= acc_rows ? 3 : 1;
}
__host__ __device__ inline int dh_products(int n_pad, int acc_rows, int tiles_n, int ks, int split_f32) {
  return split_products(split_f32, (n_pad / 256) * tiles_n, ks, n_pad, acc_rows);
}

// dW and dH run in tiles of 256 or of 320 (wide) output columns.  A wide tile takes 1.25 times as long, less WIDE_GAIN thousandths for the operand bytes
// that it saves, so it is chosen by the tiles that either needs, and by how these fill the rounds over 256 compute units.  A
// last round that is partly filled costs about the mean of its share and of a whole round: with the rest of the chip idle, what runs runs faster.
// Measured, launches in turn in one process, 256 / 320:
//   d = 5120 (20 / 16 tiles)   dH, 12000 rows, 3.67 / 2.94 rounds 7.72 / 6.99 ms, 16384 rows, 5 / 4 rounds 3.69 / 3.57;
//                              dW, 10 / 8 rounds of 128 vocab tiles 3.60 / 3.48 ms, 46.4 / 37.1 rounds, 11 stages 1323 / 1273 us
//   d = 4096 (16 / 13 tiles)   dH, 10000 rows, 2.5 / 2.03 rounds 5.82 / 6.51 ms (stays 256), 4100 rows, split 4.00 / 3.95;
//                              dW, 37.1 / 30.2 rounds, 16 stages 1308 / 1255 us, 65 stages, bf16 3.55 / 3.51 ms
//   d = 1920 (8 / 6 tiles)     20000 rows, dW 2.98 / 2.65 ms, dH 3.10 / 2.66
constexpr int WIDE_GAIN = 35;
// The 320 rows of a W^T or H^T of this leading dimension lie within the 32-bit range of one tile's loads (SlabLoader); what the calls accept is bounded by 256.
__host__ __device__ inline bool wide_fits(long long ld) { return (unsigned long long)ld * 2 * WIDE_ROWS < 1ull << 32; }
__host__ __device__ inline int store_tiles_n(int n, bool wide) { return wide ? (n + WIDE_ROWS - 1) / WIDE_ROWS : (n + BN - 1) / BN; }
__host__ __device__ inline long long launch_cost(int tiles, int stages, bool wide) {
  const long long rounds_x512 = ((long long)tiles + 255) / 256 * 256 + tiles;
  return rounds_x512 * (stages + SPLIT_TILE_STAGES) * (wide ? GW * (1000 - WIDE_GAIN) : GM * 1000);
}
__host__ __device__ inline bool wide_pays(int tiles_m, int n, Parts p256, Parts p320) {
  return launch_cost(tiles_m * p320.ks * store_tiles_n(n, true), p320.stages, true) < launch_cost(tiles_m * p256.ks * store_tiles_n(n, false), p256.stages, false);
}
// A dH of so few tiles that eight parts leave most compute units idle: as many parts as one round holds, up to DH_PARTS_MAX, or fewer where their
// slabs would cost more than they save (written, and read again by the scatter: DH_ROUND_SLABS stages per round full of them).
// Eight parts / more, dH launch and scatter together: 100 rows, d = 1024, V = 65536 (4 tiles, 48 parts) 164 / 60 us; 200 rows, d = 1024, V = 8000 (16 parts)
// 33.9 / 30.2; 100 rows, d = 4096, V = 32000 (13 tiles) 134 / 115; 200 rows, d = 5120, V = 151936 (16) 452 / 371; 300 x 2560 x 50000 179 / 142; fp32
// 512 rows, 64 x 1000 (8 / 12 slabs) 20.5 / 17.4, 1024 rows, 256 x 4000 50.7 / 36.0, 2000 rows, 512 x 10000 94 / 75.
// The most parts whose cost is below that of eight / those of least cost, whole calls: 100 rows, 1024 x 65536 188.5 / 185.1 us, normed 203.6 / 199.9;
// 215 of 12174 rows, 2752 x 13018, normed 265.8 / 252.6; 177 of 12352 rows, 2304 x 15669 173.4 / 167.7; 200 rows, 4096 x 151936 the same.
// The three products of an fp32 head one after the other cost a tile two more starts, DH_PRODUCTS_STAGES; side by side they leave room for fewer parts.
// Whole calls, side by side wherever they fit / in turn: 4178 of 6011 rows, 704 x 22504 (1 / 5 parts) 1645 / 1524 us; 5747 of 8279, 256 x 13783 (1 / 5) 992 / 918;
// 2638 rows, 128 x 27007 (3 / 11) 671 / 655; but 1126 rows, 256 x 17739 (8 / 24) 276 / 280, 2134 of 3091, 512 x 8761 (4 / 10) 372 / 378.  Over 300 such
// calls the choice costs 1.2 % at most where it is wrong.
constexpr int DH_MIN_STAGES = 4, DH_ROUND_SLABS = 16, DH_PRODUCTS_STAGES = 12;
__host__ __device__ inline Parts dh_parts(int n_pad, int acc_rows, int tiles_n, int k_stages) {
  const Parts few = dh_split(n_pad, acc_rows, tiles_n, k_stages);
  const long long tiles = (long long)(n_pad / 256) * tiles_n;
  auto fits = [&](int ks) { return tiles * ks <= 256 && (long long)ks * n_pad <= acc_rows && ks * DH_MIN_STAGES <= k_stages; };
  if (n_pad <= 0 || !fits(few.ks + 1)) return few;
  return least_parts<DH_PARTS_MAX>(k_stages, [&](int ks, int stages) -> unsigned long long {
    if (ks < few.ks || (ks > few.ks && !fits(ks))) return NO_PARTS;
    const int t = (int)tiles * ks;
    return (unsigned long long)((t + 255) / 256 * 256) * (unsigned)(stages + SPLIT_TILE_STAGES) + (unsigned)(t * DH_ROUND_SLABS);
  });
}
// The form of a dH contraction that may be split (the rows of a single token block): parts, products (slabs: ks products) and tiles.
struct DhForm { int ks, products; bool wide; };
__host__ __device__ inline DhForm dh_form(int n_pad, int acc_rows, int n, int k_stages, int split_f32, bool wide_ok) {
  const int tiles_n = store_tiles_n(n, false);
  const Parts p256 = dh_parts(n_pad, acc_rows, tiles_n, k_stages);
  if (split_f32) {        // the products side by side, where they and the parts fit one round and that is the shorter
    const Parts three = dh_parts(n_pad, acc_rows / 3, 3 * tiles_n, k_stages);
    const long long tiles = (long long)(n_pad / 256) * tiles_n;
    const long long beside = 256ll * (three.stages + SPLIT_TILE_STAGES) + 3 * tiles * three.ks * DH_ROUND_SLABS;
    const long long in_turn = (tiles * p256.ks + 255) / 256 * 256 * (3ll * p256.stages + SPLIT_TILE_STAGES + DH_PRODUCTS_STAGES) + tiles * p256.ks * DH_ROUND_SLABS;
    if (beside < in_turn && dh_products(n_pad, acc_rows, tiles_n, three.ks, split_f32) == 3) return DhForm{three.ks, 3, false};
  }
  if (split_f32 || !wide_ok) return DhForm{p256.ks, 1, false};
  const Parts p320 = dh_parts(n_pad, acc_rows, store_tiles_n(n, true), k_stages);
  const bool wide = wide_pays(n_pad / BM, n, p256, p320);
  return DhForm{wide ? p320.ks : p256.ks, 1, wide};
}

// Split-K factor of the dW contraction (over the stages of dw_stages) of a head so small that its tiles leave most
// compute units idle: parts of at least DW_MIN_STAGES stages, at most `cap` of them (what the slabs hold).
constexpr int DW_MIN_STAGES = 4, DW_SPLIT_MAX = 16;
// Stages of the dW contraction over `rows` active rows: it ends at the last stage that holds one, not at the padded count
// (rows beyond the active ones are zeros in both operands).  675 rows, 11 stages instead of 12: call 3103 -> 3001 us
// (d = 5120); 2869 rows, 45 instead of 48: 9241 -> 9160; 4100 rows, 65 instead of 68: 11 978 -> 11 893 (d = 4096).
__host__ __device__ inline int dw_stages(int rows) { return rows > 0 ? (rows + BK - 1) / BK : 0; }
__host__ __device__ inline int dw_split(int stages, int cap) { return imax(1, imin(stages / DW_MIN_STAGES, cap)); }

// ---- operand slabs in LDS ----------------------------------------------------------
// Row r (one of 256) holds its 64 k-values as eight 16-byte chunks; chunk c is stored at
// position c ^ ((r >> 1) & 7): a 16-lane group of an operand read (16 consecutive rows, same
// logical chunk) then touches 16 distinct bank groups (measured: zero bank conflicts).
// One wavefront load instruction fills 1024 contiguous LDS bytes (8 rows); lane l lands at row
// l/8, position l%8, so it fetches the logical chunk (l%8) ^ ((row>>1)&7) of that row.
// Loads beyond the buffer resource's size return 0, which pads ragged tiles.
// G: MFMA rows of a wavefront, i.e. the slab has 64 G rows.
static_assert(BM == BN, "one loader serves both operands");
template <int G>
struct SlabLoader {
  static constexpr int GROUPS = G;
  static constexpr uint32_t k_step = BK * 2;   // bytes from one stage to the next
  __device__ __forceinline__ bool on(int kt, int nk) const { return kt < nk; }
  const void* base;
  uint32_t bytes;
  uint32_t voff[G];

  // Buffer resource over the operand; with on == false its range is empty, so loads through it
  // fetch nothing and deliver zeros (used to switch the loads off beyond the last stage without
  // a branch in the schedule).
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(bool on) const {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, on ? bytes : 0u, 0x00020000);
  }

  // The resource covers only the (up to) 64 G rows of this tile, from byte k_byte0 of its first
  // row to the end of its last existing row, so operands of any number of rows can be addressed (a
  // resource's range and the lane offsets are 32-bit: 64 G rows lie below 4 GiB, see wide_fits) and rows beyond rows_total read as 0.
  __device__ __forceinline__ void init(const void* base_, int rows_total, int row0, int ld_elems, uint32_t k_byte0,
                                       int tid) {
    const int rows = min(max(rows_total - row0, 0), 64 * G);
    const uint64_t b = reinterpret_cast<uint64_t>(base_) + (uint64_t)row0 * (uint64_t)ld_elems * 2u + k_byte0;
    // the tile index is the same for the whole workgroup: keep the resource in scalar registers
    // (left to itself the compiler treats it as per-lane and loops over every load)
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    base = reinterpret_cast<const void*>(((uint64_t)hi << 32) | lo);
    bytes = __builtin_amdgcn_readfirstlane(rows > 0 ? (uint32_t)rows * (uint32_t)ld_elems * 2u - k_byte0 : 0u);
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const int row = (i * NW + wave) * 8 + (lane >> 3);
      const int chunk = (lane & 7) ^ ((row >> 1) & 7);
      voff[i] = (uint32_t)row * (uint32_t)ld_elems * 2u + (uint32_t)chunk * 16u;
    }
  }

  // global -> LDS, bypassing registers: chunk i (1 KiB = 8 rows) of this wavefront's share of one
  // operand slab.  `wave` must be wave-uniform (it addresses LDS through M0).
  __device__ __forceinline__ void issue1(__amdgpu_buffer_rsrc_t r, int i, uint32_t k_byte_off, char* slab,
                                         int wave) const {
    char* dst = slab + (i * NW + wave) * 1024;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)dst, 16, voff[i], k_byte_off, 0, 0);
  }
};
typedef SlabLoader<GM> TileLoader;

// An A operand whose k runs over the ROWS of its matrix (X[k][n], n contiguous): a slab is 64 rows x 64 G
// columns, 128 G bytes per row, and the fragments are read transposed (ds_read_b64_tr_b16: a 16-lane group reads 4 rows
// x 16 columns, lane i receives the 4 rows of column i).  The 32-byte column group p of row r is stored at position
// p ^ swizzle(r): the eight rows that a half-wavefront reads (four in a row, and the four that lie eight further) then lie in eight
// different groups of 8 banks.  Rows of 512 bytes all begin in the same bank, so that takes three bits; rows of 640 begin in either half of
// the banks in turn, which leaves two, and keeps the twenty column groups among themselves.
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
template <int G>
struct RowsLoader {
  static_assert(G == 4 || G == 5, "rows of 512 or 640 bytes");
  static constexpr int GROUPS = G, ROW_BYTES = 128 * G, ROW_CHUNKS = ROW_BYTES / 16;
  static __host__ __device__ inline int swizzle(int row) { return G == 4 ? (row & 3) | (((row >> 3) & 1) << 2) : ((row >> 1) & 1) | (((row >> 3) & 1) << 1); }
  const void* base;
  uint32_t bytes;
  uint32_t voff[G];
  uint32_t k_step;      // bytes from one stage to the next
  int rows;             // rows that exist
  // (a stage without a single row is switched off: its offset would lie beyond the resource's range)
  __device__ __forceinline__ bool on(int kt, int nk) const { return kt < nk && kt * BK < rows; }

  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(bool on) const {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, on ? bytes : 0u, 0x00020000);
  }
  // Where 16-byte chunk c of the slab in LDS (counted through its rows) comes from: row and byte in the row
  static __host__ __device__ inline void source(int c, int& row, int& byte) {
    row = c / ROW_CHUNKS;
    const int q = c - row * ROW_CHUNKS;
    byte = ((((q >> 1) ^ swizzle(row)) << 1) | (q & 1)) * 16;
  }
  // rows [k_row0, k_rows) of a matrix of row length ld, from column col0 on.  Rows at and beyond k_rows read as
  // zero; columns beyond the matrix read whatever follows in memory within it (they only reach output columns
  // that are not stored).  (k_rows - k_row0) ld 2 must stay below 4 GiB.
  __device__ __forceinline__ void init(const void* base_, int k_rows, int k_row0, int ld, int col0, int tid) {
    const uint64_t b = reinterpret_cast<uint64_t>(base_) + ((uint64_t)k_row0 * (uint64_t)ld + (uint64_t)col0) * 2u;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    base = reinterpret_cast<const void*>(((uint64_t)hi << 32) | lo);
    rows = __builtin_amdgcn_readfirstlane(max(k_rows - k_row0, 0));
    bytes = __builtin_amdgcn_readfirstlane(rows > 0 ? (uint32_t)rows * (uint32_t)ld * 2u - (uint32_t)col0 * 2u : 0u);
    k_step = (uint32_t)BK * (uint32_t)ld * 2u;
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int i = 0; i < G; ++i) {
      int row, byte;
      source((i * NW + wave) * 64 + lane, row, byte);
      voff[i] = (uint32_t)row * (uint32_t)ld * 2u + (uint32_t)byte;
    }
  }
  __device__ __forceinline__ void issue1(__amdgpu_buffer_rsrc_t r, int i, uint32_t k_byte_off, char* slab, int wave) const {
    char* dst = slab + (i * NW + wave) * 1024;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)dst, 16, voff[i], k_byte_off, 0, 0);
  }
};

// One transposed read.  (The pointer is a restrict parameter so that the read carries alias information of its own: without
// it the compiler waits for every outstanding global -> LDS load in front of it.  The schedule's barriers order the two.)
__device__ __forceinline__ bf16x4 ds_read_tr(lds_bf16x4* __restrict__ p) { return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(p); }

// Which 16 rows of the A slab MFMA tile i of wavefront row wm has: 64 in a row per wavefront, and the fifth tiles of the four behind them, so that what
// a wavefront stores begins on a 128-byte line (80 rows in a row per wavefront: an accumulating dW of d = 4096 took 6 % longer).
__host__ __device__ inline int mfma_rows(int wm, int i) { return i < GM ? wm * GM + i : WM * GM + wm; }

// Fragments of the A slab: MFMA tile i of this wavefront, k-half ks of the stage.
template <class Loader> struct FragA;
template <int G> struct FragA<SlabLoader<G>> {
  uint32_t off, off5, koff[2];
  __device__ __forceinline__ FragA(int lane, int wm) {
    off = (uint32_t)(mfma_rows(wm, 0) * 16 + (lane & 15)) * 128u;
    off5 = (uint32_t)(mfma_rows(wm, GM) * 16 + (lane & 15)) * 128u;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) koff[ks] = (uint32_t)(((ks * 4 + (lane >> 4)) ^ ((lane >> 1) & 7)) << 4);
  }
  __device__ __forceinline__ bf16x8 read(const char* st, int ks, int i) const {
    return *reinterpret_cast<const bf16x8*>(st + (i < GM ? off + i * (16 * 128) : off5) + koff[ks]);
  }
};
template <int G> struct FragA<RowsLoader<G>> {
  static constexpr int ROW_BYTES = RowsLoader<G>::ROW_BYTES;
  uint32_t off[G];
  __device__ __forceinline__ FragA(int lane, int wm) {
    const int row = (lane >> 4) * 8 + ((lane & 15) >> 2), s = RowsLoader<G>::swizzle(row);       // (the same four rows further)
#pragma unroll
    for (int i = 0; i < G; ++i) off[i] = (uint32_t)row * ROW_BYTES + (uint32_t)(mfma_rows(wm, i) ^ s) * 32u + (uint32_t)(lane & 3) * 8u;
  }
  __device__ __forceinline__ bf16x8 read(const char* st, int ks, int i) const {
    const char* p = st + off[i] + ks * (32 * ROW_BYTES);
    const bf16x4 lo = ds_read_tr((lds_bf16x4*)p), hi = ds_read_tr((lds_bf16x4*)(p + 4 * ROW_BYTES));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

// Where a main loop begins, in the 32-byte pieces that instructions are fetched in.  It decides how closely the workgroups of an XCD stay
// together in k, and with that how often their operands meet in its L2: forward-only, d = 5120, 16384 rows, 0, 4 or 8 bytes into a piece
// 17.65 ms and 96 GB fetched, 12 bytes 16.9 and 52, 16 to 28 16.8 and 48 (d = 4096, 14.4 / 13.65 / 13.55 ms; loss calls' forward 1 %).  dW, dH
// and the recompute: 0.3 to 1 % (dH of 2869 rows 2 %) longer at 0 and 4 than from 8 to 28.  (Left to itself the position changes with any
// line in front of it.)  PAD: four-byte steps from a piece's start, to which the compiler adds what it puts in front of the loop.
template <int PAD>
__device__ __forceinline__ void place_loop() { asm volatile(".p2align 5\n\t.rept %0\n\ts_nop 0\n\t.endr" ::"n"(PAD)); }

// The order of a stage's MFMAs: every one shares an operand with the one before it.  The matrix cores draw less where an operand stays, and the
// chip is power-limited: operands in registers (256 workgroups of 8 wavefronts, the engine's 4 x 8 tiles, random values), column by column
// from row 0 down 2088 TFLOP/s, mfma_snake 2135, mfma_pairs 2148, neither operand shared 2030.  In the contractions, against
// column by column: forward only 13.35 -> 13.22 ms (16384 rows, d = 4096) and 33.56 -> 33.26 ms (32768 rows, d = 5120) with the snake, which the pairs make
// longer (13.37 and 34.18: their LDS reads come in twos, and the workgroups of an XCD drift further apart); dW and dH of 12000 rows, d = 5120, together
// 26.04 -> 25.81 ms with the snake and 25.66 with the pairs.
// MFMA q (of G) of step s, NJ columns of G rows in each k-half.  Snake: column s, every second column from the last row up.
template <int NJ>
__device__ __forceinline__ void mfma_snake(int s, int q, const bf16x8 (&a)[2][GM], const bf16x8 (&bq)[4], f32x4 (&acc)[GM][GN]) {
  const int i = s % 2 ? GM - 1 - q : q, ks = s / NJ, j = s % NJ;
  acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][i], bq[s & 3], acc[i][j], 0, 0, 0);
}
// Pairs: steps 2p and 2p + 1 take the columns 2p and 2p + 1 together, row 0 in columns 0, 1, row 1 in columns 1, 0, and so on; every second pair from
// the last row up.
template <int NJ, int G>
__device__ __forceinline__ void mfma_pairs(int s, int q, const bf16x8 (&a)[2][G], const bf16x8 (&bq)[4], f32x4 (&acc)[G][GN]) {
  const int p = s / 2, z = (s % 2) * G + q, u = z / 2;         // pair of columns, place in it, place of the row in its order
  const int i = p % 2 ? G - 1 - u : u, h = (u + z) % 2;
  const int ks = s / NJ, j = (2 * p) % NJ + h;
  acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][i], bq[(2 * p + h) & 3], acc[i][j], 0, 0, 0);
}

// Accumulates C(64G x 256) += A(64G x K) B(256 x K)^T for this workgroup's tile, K = 64 nk, G = 4 or 5.
// acc[i][j] is the 16x16 MFMA tile at rows 16 mfma_rows(wm, i), cols wn*128+j*16 of the workgroup tile;
// within it, register r of lane l is row 4*(l>>4)+r, column l&15.
//
// Tiles of 320 rows: a tenth fewer operand bytes and an eighth fewer LDS reads per flop, which is what a power-limited contraction is made of.  This loop
// alone, 256 / 320 rows: d x tokens of 5120 x 16384 over 32768 1484 / 1550 TFLOP/s, V x tokens of 151936 x 8192 over 5120 1539 / 1593, d x V of
// 5120 x 151936 over 2816 1513 / 1542.  (More rows do not fit: two stages of LDS are 144 KiB here, and 160 of 256 registers accumulators.)
//
// A stage (64 of k) is 16 steps s = (ks, j) of G MFMAs.  Per wavefront and stage:
//   steps 0..1   second half of the B loads of stage kt+1 (the first half went out in the
//                previous tail), A fragments of the second k-half
//   step  G      barrier X: every A read of this stage is complete -> its A slab is free
//   then         A loads of stage kt+2 into that slab, one in each of G steps
//   step  13     barrier Y: every B read of this stage is complete and stage kt+1 has landed
//                (the wavefront leaves only its G newest loads, the A loads of kt+2, in flight)
//   steps 14,15  "tail": first half of the B loads of stage kt+2, first LDS reads of stage kt+1,
//                under the last 2 G MFMAs of stage kt
// On return every load has landed and every wavefront has passed a barrier, so the caller may
// reuse the LDS.  The barriers carry their own waits; the "memory" clobber keeps LDS accesses on
// their side of them.
template <class LoaderA>
__device__ __forceinline__ void mainloop(const LoaderA& LA, const TileLoader& LB, int nk, char* smem,
                                         f32x4 (&acc)[LoaderA::GROUPS][GN]) {
  constexpr int G = LoaderA::GROUPS;
  constexpr int A_BYTES = G * 64 * BK * 2, STAGE = A_BYTES + SLAB_BYTES;      // A slab, then B slab
  constexpr int NS = 2 * GN;          // steps per stage
  constexpr int TAIL = 2;             // steps behind barrier Y
  constexpr int XS = G;               // barrier X follows this step
  constexpr int BH = CHUNKS / 2;      // B loads per half
  static_assert(CHUNKS == 4 && BH <= XS && XS + G < NS - TAIL && G + 2 <= TAIL * G, "load schedule");
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int lrow = lane & 15;
  const int xr = (lane >> 1) & 7;
  const FragA<LoaderA> fa(lane, wm);
  const uint32_t b_off = (uint32_t)(wn * WCOLS + lrow) * 128u + A_BYTES;
  uint32_t koff[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) koff[ks] = (uint32_t)(((ks * 4 + (lane >> 4)) ^ xr) << 4);
  if (nk <= 0) return;

  bf16x8 a[2][G], bq[4];
  auto rdA = [&](const char* st, int ks, int i) -> bf16x8 { return fa.read(st, ks, i); };
  auto rdB = [&](const char* st, int s) -> bf16x8 {   // B fragment of step s
    return *reinterpret_cast<const bf16x8*>(st + b_off + (s % GN) * (16 * 128) + koff[s / GN]);
  };

  {  // prologue: stage 0 complete, A and the first half of B of stage 1
    const __amdgpu_buffer_rsrc_t ra = LA.rsrc(LA.on(0, nk)), rb = LB.rsrc(true);
#pragma unroll
    for (int i = 0; i < G; ++i) LA.issue1(ra, i, 0, smem, wave);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) LB.issue1(rb, i, 0, smem + A_BYTES, wave);
    const bool a1 = LA.on(1, nk);
    const __amdgpu_buffer_rsrc_t ra1 = LA.rsrc(a1), rb1 = LB.rsrc(nk > 1);
#pragma unroll
    for (int i = 0; i < G; ++i) LA.issue1(ra1, i, a1 ? LA.k_step : 0u, smem + STAGE, wave);
#pragma unroll
    for (int i = 0; i < BH; ++i) LB.issue1(rb1, i, BK * 2, smem + STAGE + A_BYTES, wave);
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(G + BH) : "memory");   // all but the G + BH newest
  bq[0] = rdB(smem, 0);
#pragma unroll
  for (int i = 0; i < G; ++i) a[0][i] = rdA(smem, 0, i);
  bq[1] = rdB(smem, 1);

  place_loop<3>();
  for (int kt = 0; kt < nk; ++kt) {
    char* cur = smem + (kt & 1) * STAGE;
    char* nxt = smem + ((kt + 1) & 1) * STAGE;
    const uint32_t kb1 = (uint32_t)(kt + 1) * (BK * 2), kb2 = (uint32_t)(kt + 2) * (BK * 2);
    const bool a2 = LA.on(kt + 2, nk);
    const uint32_t ka2 = a2 ? (uint32_t)(kt + 2) * LA.k_step : 0u;
    const __amdgpu_buffer_rsrc_t rb1 = LB.rsrc(kt + 1 < nk);
    const __amdgpu_buffer_rsrc_t ra2 = LA.rsrc(a2), rb2 = LB.rsrc(kt + 2 < nk);
#pragma unroll
    for (int s = 0; s < NS - TAIL; ++s) {
      if (s % 2 == 0) { bq[(s + 2) & 3] = rdB(cur, s + 2); bq[(s + 3) & 3] = rdB(cur, s + 3); }
      if (s < G) a[1][s] = rdA(cur, 1, s);
      if (s < BH) LB.issue1(rb1, BH + s, kb1, nxt + A_BYTES, wave);
      if (s > XS && s <= XS + G) LA.issue1(ra2, s - XS - 1, ka2, cur, wave);
#pragma unroll
      for (int q = 0; q < G; ++q) mfma_pairs<GN>(s, q, a, bq, acc);
      // barrier X: all LDS reads but those of an even step XS, two B fragments, are complete
      if (s == XS) asm volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" ::"n"(XS % 2 ? 0 : 2) : "memory");
      __builtin_amdgcn_sched_barrier(0);   // keep this read/load/MFMA interleave as written
    }
    // barrier Y
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(G) : "memory");
#pragma unroll
    for (int m = 0; m < TAIL * G; ++m) {
      if (m < 2) bq[m] = rdB(nxt, m);
      else if (m < 2 + G) a[0][m - 2] = rdA(nxt, 0, m - 2);
      if (m % G == 0) LB.issue1(rb2, m / G, kb2, cur + A_BYTES, wave);
      mfma_pairs<GN>(NS - TAIL + m / G, m % G, a, bq, acc);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- the same main loop as a stream of tiles (persistent workgroups) -------------------------------
// A persistent workgroup walks a sequence of tiles that share the operands' leading dimensions
// and the contraction length.  The per-lane offsets are then the same for every tile (OperandLanes);
// what changes from tile to tile is the wave-uniform base address and byte range (TileSrc).  The
// stage schedule above keeps two stages of loads in flight, and across a tile boundary those are
// simply the first two stages of the next tile: the load stream never drains, the next tile's
// stage 0 has landed and most of its stage 1 is in flight when the current tile's last MFMA
// retires, and the epilogue runs with those loads in flight.  The epilogue must therefore not touch
// the two stage buffers (the first 2 x STAGE_BYTES of the dynamic LDS).
struct OperandLanes {
  uint32_t voff[CHUNKS];
  __device__ __forceinline__ void init(int ld_elems, int tid) {
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int row = (i * NW + wave) * 8 + (lane >> 3);
      const int chunk = (lane & 7) ^ ((row >> 1) & 7);
      voff[i] = (uint32_t)row * (uint32_t)ld_elems * 2u + (uint32_t)chunk * 16u;
    }
  }
};

struct TileSrc {
  uint32_t lo, hi, bytes;       // wave-uniform (scalar registers)
  // rows [row0, row0 + 256) of an operand with rows_total rows of ld_elems elements, from byte
  // k_byte0 of each row on; rows beyond rows_total read as zero; bytes = 0 switches the loads off
  __device__ __forceinline__ void set(const void* base_, int rows_total, int row0, int ld_elems, uint32_t k_byte0) {
    const int rows = min(max(rows_total - row0, 0), BM);
    const uint64_t b = reinterpret_cast<uint64_t>(base_) + (uint64_t)row0 * (uint64_t)ld_elems * 2u + k_byte0;
    lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    bytes = __builtin_amdgcn_readfirstlane(rows > 0 ? (uint32_t)rows * (uint32_t)ld_elems * 2u - k_byte0 : 0u);
  }
  __device__ __forceinline__ void off() { lo = 0; hi = 0; bytes = 0; }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc() const {
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uint64_t)hi << 32) | lo), 0, bytes, 0x00020000);
  }
};

__device__ __forceinline__ void issue_lds(__amdgpu_buffer_rsrc_t r, const OperandLanes& L, int i, uint32_t k_byte_off,
                                          char* slab, int wave) {
  char* dst = slab + (i * NW + wave) * 1024;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)dst, 16, L.voff[i], k_byte_off, 0, 0);
}

// Buffer resource and k byte offset of stage g (counted from this tile's stage 0) of the stream:
// stages 0 .. nk-1 belong to this tile, nk and nk+1 to the next one (nk >= 2).  All of it is
// wave-uniform and stays in scalar registers; the sources are passed as plain values for that.
__device__ __forceinline__ void pick_stage(const TileSrc cur, const TileSrc nxt, int g, int nk,
                                           __amdgpu_buffer_rsrc_t& r, uint32_t& kb) {
  const bool ahead = g >= nk;
  kb = (uint32_t)(ahead ? g - nk : g) * (BK * 2);
  TileSrc t;
  t.lo = __builtin_amdgcn_readfirstlane(ahead ? +nxt.lo : +cur.lo);
  t.hi = __builtin_amdgcn_readfirstlane(ahead ? +nxt.hi : +cur.hi);
  t.bytes = __builtin_amdgcn_readfirstlane(ahead ? +nxt.bytes : +cur.bytes);
  r = t.rsrc();
}

// The last token tile of the forward may hold few rows.  A tile of `cols` live columns runs NJ = 8, 6 or 4 of the 8 MFMA columns
// of every wavefront.  A stage of NJ = 4 is as long as its loads, so nothing shorter; and where a vocab tile has more than two
// token tiles, one that ends early starts the next before the others are there and their W no longer meets in the L2
// (d = 4096, V = 151936, 677 rows: 3.7 GB read instead of 1.8), so NJ = 6 loses what it saves.  Forward-only call, whole
// tiles against this: 128 rows 295 -> 267 us, 192 331 -> 291, 384 473 -> 454, 448 487 -> 484, 640 681 -> 675, 2176 2002 -> 1967; NJ = 6
// at 704 rows 743 -> 755, at 1216 1208 -> 1233.  (The dH contraction and the recompute of the logits gained nothing: +-0.3 %.)
// Where a vocab tile's token tiles are handed out before the next one (no logits kept), the early start costs more the more of them share W
// in the last panel (of SB_N), and the longer the contraction: from five on at K >= 3072 the tile stays whole (short_tile_pays), unless the launch is so
// short that what does not fill its last round counts for more.  Forward-only,
// last tile short / whole: d = 5120, V = 473637, 1150 rows 4480 / 4260 us, 1664 rows 6244 / 5926; V = 151936, 1400 rows 1693 / 1633, 3968 rows 4388 / 4252;
// d = 3072, 1400 rows 1025 / 1005, 1150 rows 854 / 854; but d = 2560, 1150 rows 711 / 721; four tiles, 800 rows, d = 4096 869 / 873, d = 5120 1093 /
// 1099; one, 2176 rows 1967 / 2002, 2458 / 2498; short contractions d = 2048, V = 100000, 1150 rows 387 / 388, 1400 rows 458 / 464;
// fewer than eight rounds of tiles, d = 5120, 1578 rows, V = 28498, 3.06 rounds 392 / 414, d = 4096, 1144 rows, 4.1 rounds 409 / 424, 1664 rows, 4.3 and 6.4 rounds 425 /
// 431 and 625 / 626; but 10.7 rounds 1028 / 1006, d = 5120, 1400 rows, 7.3 and 9.2 rounds 887 / 879 and 1101 / 1093.
__host__ __device__ inline int fwd_nj(int cols, int tiles_t) { return cols > (tiles_t > 2 ? 128 : 192) ? 8 : cols > 128 ? 6 : 4; }
__host__ __device__ inline bool short_tile_pays(int tiles_t, int K, int tiles, int grid) { return K < 3072 || (tiles_t - 1) % SB_N < 4 || tiles / 8 < grid; }

// The two wavefronts of a row take the 16-column groups of the tile in turn, so that the first NJ MFMA columns of both are its
// first 32 NJ columns:
__device__ __forceinline__ int stream_col(int j, int wn, int lane) { return j * (16 * WN) + wn * 16 + (lane & 15); }

// The schedule: NJ = 6 leaves out four of the 16 steps; NJ = 4 has half of them, reads two A fragments per step, passes X after
// step 2 and issues the A loads in steps 3..5.  The loads are those of a whole tile (columns beyond the operand read as zero).
template <int NJ>
struct Steps {
  static constexpr int NS = 2 * NJ;          // steps per stage
  static constexpr int TAIL = 2;             // steps behind barrier Y
  static constexpr int A_READS = NJ == 4 ? 2 : 1;      // A fragments of the second k-half read per step
  static constexpr int XS = NJ == 4 ? 2 : 4; // barrier X follows this step
  static constexpr int BH = CHUNKS / 2;      // B loads per half
  // A loads [first, last) of step s
  static constexpr int a_first(int s) { return s <= XS ? 0 : NJ == 4 ? (s == XS + 1 ? 0 : s - XS) : s - XS - 1; }
  static constexpr int a_last(int s) { return s <= XS ? 0 : NJ == 4 ? s - XS + 1 : s - XS; }
  static_assert(NJ == 4 || NJ == 6 || NJ == 8, "steps in multiples of four: B fragments rotate through four registers");
  static_assert(CHUNKS == 4 && GM == 4 && BH <= XS && a_last(NS - TAIL - 1) >= CHUNKS && GM / A_READS <= XS && GM / A_READS <= NJ, "schedule");
};

// One tile of the stream: acc += A(256 x K) B(256 x K)^T with K = 64 nk, for the first 32 NJ columns.
//   A0, B0    operand sources of this tile; A1, B1 of the next one (bytes = 0 where the stream
//             ends).  A tile of a single stage (nk = 1) cannot run ahead by two stages: the caller
//             then passes switched-off next sources, cold = true for every tile, and waits for
//             vmcnt(0) and a barrier before the next call.
//   cold      the stream starts here: nothing of this tile is in flight yet
//   par0      stage buffer (0 / 1) that holds, or will hold, this tile's stage 0; the next tile's is
//             (par0 + nk) & 1
// On return the first two stages of the next tile are in the stage buffers or on their way (this
// wavefront's newest CHUNKS + BH loads may still be in flight) and nobody reads the buffers until the
// next call's opening barrier.
template <int NJ>
__device__ __forceinline__ void mainloop_stream(const OperandLanes& VA, const OperandLanes& VB, const TileSrc A0,
                                                const TileSrc B0, const TileSrc A1, const TileSrc B1, int nk,
                                                bool cold, int par0, char* smem,
                                                f32x4 (&acc)[GM][GN]) {
  typedef Steps<NJ> St;
  constexpr int NS = St::NS, TAIL = St::TAIL, XS = St::XS, BH = St::BH;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int lrow = lane & 15;
  const int xr = (lane >> 1) & 7;
  const uint32_t a_off = (uint32_t)(wm * WROWS + lrow) * 128u;
  const uint32_t b_off = (uint32_t)(wn * 16 + lrow) * 128u + SLAB_BYTES;
  uint32_t koff[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) koff[ks] = (uint32_t)(((ks * 4 + (lane >> 4)) ^ xr) << 4);

  bf16x8 a[2][GM], bq[4];
  auto rdA = [&](const char* st, int ks, int i) -> bf16x8 {
    return *reinterpret_cast<const bf16x8*>(st + a_off + i * (16 * 128) + koff[ks]);
  };
  auto rdB = [&](const char* st, int s) -> bf16x8 {
    return *reinterpret_cast<const bf16x8*>(st + b_off + (s % NJ) * (32 * 128) + koff[s / NJ]);
  };

  if (cold) {   // stage 0 complete, A and the first half of B of stage 1
    char* s0 = smem + par0 * STAGE_BYTES;
    char* s1 = smem + (par0 ^ 1) * STAGE_BYTES;
    __amdgpu_buffer_rsrc_t ra, rb;
    uint32_t kb;
    pick_stage(A0, A1, 0, nk, ra, kb);
    pick_stage(B0, B1, 0, nk, rb, kb);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) issue_lds(ra, VA, i, 0, s0, wave);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) issue_lds(rb, VB, i, 0, s0 + SLAB_BYTES, wave);
    pick_stage(A0, A1, 1, nk, ra, kb);
    pick_stage(B0, B1, 1, nk, rb, kb);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) issue_lds(ra, VA, i, kb, s1, wave);
#pragma unroll
    for (int i = 0; i < BH; ++i) issue_lds(rb, VB, i, kb, s1 + SLAB_BYTES, wave);
  }
  // stage 0 has landed: all but this wavefront's CHUNKS + BH newest loads are complete
  asm volatile("s_waitcnt vmcnt(6)\n\ts_barrier" ::: "memory");
  {
    const char* s0 = smem + par0 * STAGE_BYTES;
    bq[0] = rdB(s0, 0);
#pragma unroll
    for (int i = 0; i < GM; ++i) a[0][i] = rdA(s0, 0, i);
    bq[1] = rdB(s0, 1);
  }

  place_loop<0>();      // (16 or 20 bytes into a piece)
  for (int kt = 0; kt < nk; ++kt) {
    char* cur = smem + ((par0 + kt) & 1) * STAGE_BYTES;
    char* nxt = smem + ((par0 + kt + 1) & 1) * STAGE_BYTES;
    __amdgpu_buffer_rsrc_t rb1, ra2, rb2;
    uint32_t kb1, kb2, kb2b;
    pick_stage(B0, B1, kt + 1, nk, rb1, kb1);
    pick_stage(A0, A1, kt + 2, nk, ra2, kb2);
    pick_stage(B0, B1, kt + 2, nk, rb2, kb2b);
#pragma unroll
    for (int s = 0; s < NS - TAIL; ++s) {
      bq[(s + 2) & 3] = rdB(cur, s + 2);
#pragma unroll
      for (int q = s * St::A_READS; q < (s + 1) * St::A_READS && q < GM; ++q) a[1][q] = rdA(cur, 1, q);
      if (s < BH) issue_lds(rb1, VB, BH + s, kb1, nxt + SLAB_BYTES, wave);
#pragma unroll
      for (int q = St::a_first(s); q < St::a_last(s) && q < CHUNKS; ++q) issue_lds(ra2, VA, q, kb2, cur, wave);
#pragma unroll
      for (int q = 0; q < 4; ++q) mfma_snake<NJ>(s, q, a, bq, acc);
      if (s == XS) asm volatile("s_waitcnt lgkmcnt(1)\n\ts_barrier" ::: "memory");   // barrier X
      __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");          // barrier Y
#pragma unroll
    for (int m = 0; m < TAIL * GM; ++m) {
      if (m == 0) bq[0] = rdB(nxt, 0);
      else if (m <= GM) a[0][m - 1] = rdA(nxt, 0, m - 1);
      else if (m == GM + 1) bq[1] = rdB(nxt, 1);
      if (m % GM == 0) issue_lds(rb2, VB, m / GM, kb2b, cur + SLAB_BYTES, wave);
      mfma_snake<NJ>(NS - TAIL + m / GM, m % GM, a, bq, acc);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}
__device__ __forceinline__ void mainloop_stream(const OperandLanes& VA, const OperandLanes& VB, const TileSrc A0, const TileSrc B0,
                                                const TileSrc A1, const TileSrc B1, int nk, bool cold, int par0, int nj, char* smem,
                                                f32x4 (&acc)[GM][GN]) {
  if (nj == 8) mainloop_stream<8>(VA, VB, A0, B0, A1, B1, nk, cold, par0, smem, acc);
  else if (nj == 6) mainloop_stream<6>(VA, VB, A0, B0, A1, B1, nk, cold, par0, smem, acc);
  else mainloop_stream<4>(VA, VB, A0, B0, A1, B1, nk, cold, par0, smem, acc);
}

// ---- tile queue of the persistent kernels ----------------------------------------------------------
// The eight XCDs of the chip run at different clocks under load (each has its own frequency
// control: 1.58 to 1.80 GHz were measured side by side in one launch), so an equal share of the
// tiles per XCD (which is what the hardware dispatcher hands out: workgroup b runs on XCD b mod 8)
// makes a launch as slow as its slowest XCD.  The MFMA kernels are therefore persistent (one
// workgroup per compute unit) and take their tiles from a queue: XCD y owns the tiles that the
// XCD-aware order (map_tile / map_tile_interleaved) gives to the workgroups b = 8 i + y,
// i = 0 .. n_y - 1; its workgroups take them in that order with one atomic increment of cnt[y], and
// once its share is used up they take tiles from the XCD that has most left.  Which workgroup
// computes a tile does not change the tile's result, so results stay bitwise repeatable.
// The first entries of every share are dealt by workgroup index (entry), without the counter: a workgroup starts on its first
// loads at once, and where that is all there is, no counter is touched (fp32 head of 64 x 1000, 1024 rows: call 85.0 -> 81.8
// us; d = 4096, 677 rows forward only: 704 -> 697).
// With few more tiles than workgroups, as few workgroups as that takes get two and the others none: one for everybody first is the same
// two rounds with all of the chip's power and bandwidth spent in the first.  Forward only, one for everybody / two for few: d = 4096,
// 24 rows, 257 tiles 185 / 150 us; 1024 rows, 284 tiles 171 / 148; 1280 rows, 360 tiles 168 / 159, 400 tiles 168 / 168, 450 tiles 180 / 182; 192
// rows, 380 tiles 189 / 184; d = 2048, 256 rows, 360 tiles 121 / 112, 400 tiles 127 / 123, 430 tiles 127 / 127, 490 tiles 144 / 145.
// (The caller says where it may, few: see lmhead_fwd_body.)
// cnt[0..7] must be zero at launch.
struct TileQueue {
  unsigned* cnt;
  int total;          // tiles of the launch
  int interleaved;    // 0: map_tile order, 1: map_tile_interleaved order
  int home;           // XCD this workgroup runs on
  int stride = 0;     // workgroup b is dealt the entries (b >> 3) + k stride of XCD b & 7 for k < rounds, if (b >> 3) < stride,
  int dealt = 0;      // which are the first rounds * stride of every share

  // rounds: how many entries a workgroup is dealt at most
  __host__ __device__ inline void deal(int grid, int rounds, bool few) {      // (the grid is a multiple of 8)
    stride = grid >> 3;
    if (few && rounds == 2 && total <= grid + grid * 9 / 16) stride = imin(stride, (total + 15) / 16);
    dealt = rounds * stride;
  }
  __device__ __forceinline__ void init(unsigned* cnt_, int total_, int interleaved_, int rounds, bool few = false) {
    cnt = cnt_; total = total_; interleaved = interleaved_;
    deal((int)gridDim.x, rounds, few);
    unsigned x;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
    home = (int)(x & 7u);
  }
  // n_y: how many workgroup indices b = 8 i + y map to a tile
  __host__ __device__ inline int share(int y) const {
    if (!interleaved) {
      const int per = (total + 7) / 8;
      return imin(imax(total - y * per, 0), per);
    }
    const int full = (total / 256) * 256, rem = total - full, per = (rem + 7) / 8;
    return full / 8 + imin(imax(rem - y * per, 0), per);
  }
  // the workgroup index that map_tile / map_tile_interleaved would have seen for entry i of XCD y
  static __host__ __device__ inline int encode(int y, int i) { return (i << 3) | y; }

  // The entry that a workgroup is dealt in a round, encoded, or -1 where there is none for it.
  __host__ __device__ inline int entry(int block, int round) const {
    const int y = block & 7, i = (block >> 3) + round * stride;
    return (block >> 3) < stride && i < share(y) ? encode(y, i) : -1;
  }

  // Issues the claim on the home share; the ticket is resolved later, so that the atomic's latency
  // hides behind whatever runs in between.  (atomicInc with the largest bound is an add of one; unlike
  // atomicAdd the compiler does not turn it into a wave-wide reduction that needs the result at once.)
  __device__ __forceinline__ unsigned ticket() const { return atomicInc(cnt + home, 0xffffffffu); }

  // What ticket tk of XCD y's counter stands for, encoded, or -1 beyond its share: tickets count from behind the dealt entries.
  __host__ __device__ inline int claimed(int y, unsigned tk) const {
    const int i = (int)(tk < 0x40000000u ? tk : 0x40000000u) + dealt;
    return i < share(y) ? encode(y, i) : -1;
  }
  // Workgroup index (see encode) of the claimed tile, or -1 when no tile is left anywhere.  Every failed
  // attempt means one more XCD's share is used up, so the loop ends after at most nine rounds.
  // drawn(y): tickets drawn from counter y so far; draw(y): the next one.
  // steal = false confines every XCD to its own share (used by the measurement tool only).
  template <class Drawn, class Draw>
  __host__ __device__ inline int resolve(unsigned tk, bool steal, Drawn&& drawn, Draw&& draw) const {
    const int own = claimed(home, tk);
    if (own >= 0 || !steal) return own;
    for (int attempt = 0; attempt < 9; ++attempt) {
      int best = -1, best_left = 0;
      for (int y = 0; y < 8; ++y) {
        const unsigned c = drawn(y);
        const int left = share(y) - dealt - (int)(c < 0x40000000u ? c : 0x40000000u);
        if (left > best_left) { best_left = left; best = y; }
      }
      if (best < 0) return -1;
      const int b = claimed(best, draw(best));
      if (b >= 0) return b;
    }
    return -1;
  }
  __device__ __forceinline__ int resolve(unsigned tk, bool steal = true) const {
    return resolve(
        tk, steal, [&](int y) { return __hip_atomic_load(cnt + y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
        [&](int y) { return atomicInc(cnt + y, 0xffffffffu); });
  }
};

// ---- workgroups of an XCD in step ------------------------------------------------------------------
// The 32 workgroups of an XCD work on tiles that share operands, and what one has fetched is in the 4 MiB L2 for the others only while they are within some
// ten stages of each other.  Nothing holds them there: over the hundreds of rounds of a long forward they drift apart, some XCDs by a few
// stages, some by most of a tile (starts of one round in one launch: within 0.3 us on two XCDs, spread over 80 us of 118 on four).  So every 256 stages or so
// a workgroup counts itself in on its XCD's counter when its main loop ends, and behind the statistics thread 0 looks whether all have, which by
// then costs nothing if they are together.  It waits for the others at most POLLS looks (some 50 us, once: a workgroup whose wait runs out, or that has no next tile,
// counts for good and looks no more; workgroups that have no compute unit, because another stream holds it, cost no more than that).  A matter of speed only.
// Forward only, without / with: d = 5120, 131072 rows 136.6 / 133.8, 141.0 / 138.6 and, on a card whose XCDs drift less, 136.1 / 135.6 ms, 32768 rows 33.4 / 33.2 and 33.8 / 33.3; d = 4096, 16384 rows 13.33 / 13.30 and
// 13.43 / 13.35 ms (35 / 30 GB fetched, 30 being what 32 tiles at a time must).  At 131072 rows every tile instead of every fourth 134.4, every sixteenth 134.0; at
// d = 1024, 20000 rows every fourth of 16 stages 1649 / 1667 us.  Launches of fewer than ROUNDS rounds do not drift that far (39 rounds: 3751 / 3756 us), and a
// forward that parks its logits, whose look would wait for the stores, gains nothing: 12000 rows 13.43 / 13.55 ms, 16384 17.66 / 17.59.
struct InStep {
  static constexpr int STAGES = 256, POLLS = 48, ROUNDS = 64;
  static constexpr unsigned FOR_GOOD = 1u << 24;      // more than a launch can count
  unsigned* cnt;        // of this XCD
  unsigned peers, want;
  int period, left;     // tiles from one look to the next, until the next
  bool on;
  __device__ __forceinline__ void init(unsigned* counters, int home, int grid, int nk, bool on_) {
    cnt = counters + home; peers = (unsigned)grid >> 3; want = 0u; on = on_;
    period = left = 4;
    if (on) period = left = imax(4, STAGES / nk);      // (the other launches are spared the division: 128 tiles of d = 128 13.9 -> 13.7 us)
  }
  // thread 0 only, both: when a tile's main loop has ended, and before the next tile
  __device__ __forceinline__ void count(bool more) {
    if (!on) return;
    if (!more) atomicAdd(cnt, FOR_GOOD);
    else if (--left == 0) { atomicAdd(cnt, 1u); want += peers; }
  }
  __device__ __forceinline__ void wait() {
    if (!on || left > 0) return;
    left = period;
    for (int poll = 0; poll < POLLS; ++poll) {
      if (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= want) return;
      __builtin_amdgcn_s_sleep(8);
    }
    on = false;
    atomicAdd(cnt, FOR_GOOD);
  }
};

// Thread 0 claims, everybody learns the claim through one LDS word.  `slot` must lie outside whatever the
// kernel's epilogue uses; the call contains a workgroup barrier (LDS only: vector memory operations
// in flight are not waited for).
__device__ __forceinline__ int queue_broadcast(volatile int* slot, int value_of_thread0) {
  if (threadIdx.x == 0) *slot = value_of_thread0;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  const int v = __builtin_amdgcn_readfirstlane(*slot);
  return v;
}

// Row (m) index inside a 16x16 MFMA tile of accumulator register r for this lane;
// the column (n) is lane & 15.
__device__ __forceinline__ int acc_row(int r, int lane) { return ((lane >> 4) << 2) + r; }

template <int G>
__device__ __forceinline__ void zero_acc(f32x4 (&acc)[G][GN]) {
#pragma unroll
  for (int i = 0; i < G; ++i)
#pragma unroll
    for (int j = 0; j < GN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
}

}  // namespace pg
