// Argument blocks and launchers of the device kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pg {

struct Ctl;

// Tile-queue counters in the workspace: one set of 8 (one per XCD) for every persistent launch of a
// call (the forward, then recompute / dW / dH / remainder recompute of every vocab chunk), all cleared
// by the pre-pass.
constexpr int QUEUE_SET_WORDS = 8;
inline int queue_sets(int nchunks) { return 1 + 4 * nchunks; }     // per token block

// Scratch leading dimensions (multiples of 64 elements = 128 bytes) are made an odd number of
// 128-byte lines, so that the rows of a tile spread over the memory channels instead of
// landing on a few of them (power-of-two strides measured 3 % slower).
__host__ __device__ inline long long pad_ld(long long n) { return ((n / 64) % 2 == 0) ? n + 64 : n; }

// Few active rows (most samples rejected: known only on the device).  The chunk scratch is sized for
// t_cap rows; when the rows that are really active are so few that dS of the WHOLE vocabulary fits it, the
// first chunk's launches cover the whole vocabulary (the same buffers, laid out as [n_pad, ld_s_all] and
// [V_pad, pad_ld(n_pad)]) and the later chunks' launches return at once: dS, dW, and dH up to DIRECT_MAX_ROWS rows,
// where it reads W as it lies or the caller's W^T (the workspace's W^T is one chunk's: beyond, dH keeps its chunks and
// reads its columns of the wide dS).  Fewer launch tails, one pass over the dH accumulator, longer parts for its split: 3000
// rows of a d = 4096 head planned in three chunks, dW 2536 -> 2420 us, dH 2356 -> 2203 us.
// Every kernel takes the decision from the same device-side values.
struct Rechunk {
  int enabled;          // the backward was planned in more than one vocab chunk
  int chunk;            // this launch's chunk
  int tiles_v_all;      // 256-row vocab tiles of the whole head
  int ld_s_all;         // pad_ld(256 tiles_v_all)
  long long cap_s;      // elements of the dS scratch
  long long cap_t;      // elements of the dS^T scratch
  int V;                // vocab rows of the head
  int dw_whole;         // dW may run whole (it is not split into slabs)
  int dh_whole;         // dH may run whole up to DIRECT_MAX_ROWS rows
};
__device__ inline bool rechunk_all(const Rechunk& r, int n_pad, int& ld_t_all) {
  ld_t_all = (int)pad_ld(n_pad);
  return r.enabled && n_pad > 0 && (long long)n_pad * r.ld_s_all <= r.cap_s &&
         (long long)r.tiles_v_all * 256 * ld_t_all <= r.cap_t;
}

// Logits kept for the backward.  The dS of the backward needs the logits a second time, after the rows'
// logsumexp is known.  Recomputing them is a fourth contraction as long as the other three; keeping the
// fp32 accumulators of a 256 x 256 tile costs 256 KiB of HBM written once and read once.  The workspace holds
// a bounded number of such tiles (cap): the forward parks the tiles of the first kept_vocab_tiles() vocab
// tiles (all live token tiles each), as they lie in the registers, and the backward finishes those from
// memory (dlogits_kept_kernel) and recomputes only the rest.  The kept accumulators are the very values a
// recompute gives, so dS does not depend on how many are kept.
struct Kept {
  float* tiles;         // [cap][KEPT_TILE_FLOATS], null: nothing is kept
  int cap;
};
constexpr int KEPT_TILE_FLOATS = 256 * 256;
__host__ __device__ inline int kept_vocab_tiles(const Kept& k, int tiles_v, int live_tiles_t) {
  if (!k.tiles || live_tiles_t <= 0) return 0;
  const int n = k.cap / live_tiles_t;
  return n < tiles_v ? n : tiles_v;
}

// The dH contraction runs over the vocabulary, i.e. over the rows of W as the caller holds it.  With W^T it reads
// 8 consecutive k per lane; without, its fragments are read from LDS transposed (RowsLoader in gemm_core.h), which
// makes the contraction 3..5 % slower but saves writing and reading W^T, a cost that does not depend on the rows.
// Measured, dH and transposition per call: V = 151936, d = 5120, 768 rows 615 + 574 us against 694 us; d = 4096,
// 4100 rows 3585 + 457 us against 3752 us; d = 5120, 32768 rows 37.3 + 0.48 ms against 38.1 ms.  Around the line the
// two are equal for the call: W as it lies takes 0.997 of its time at 8448 to 10752 rows and 0.999 at 12032 (d = 4096), 0.997
// at 8448, 1.000 at 10752 and 1.004 at 12032 (d = 5120), 1.002, 1.004 and 1.004 at V = 18992.  The active rows are known only on the device: where they may lie on either side, both forms are launched
// and one returns at once (ctl != null).
constexpr int DIRECT_MAX_ROWS = 8192;
struct DirectRule {
  const Ctl* ctl;
};
__device__ inline bool dh_runs_whole(const Rechunk& r, int n_pad) {
  int ld_t_all;
  return r.dh_whole && n_pad <= DIRECT_MAX_ROWS && rechunk_all(r, n_pad, ld_t_all);
}

// Token blocks.  Where the kept logits of all rows do not fit their share of the workspace, but those of a good
// number of rows over the whole vocabulary do, the rows are worked off in blocks of at most cap_t token tiles: forward,
// row epilogue, dS, dW (added to the block before) and dH of a block, then the next one, so that nothing is ever
// recomputed.  The active rows are known only on the device: the host launches as many blocks as its rows may need
// and the launches of a block without any return at once.  cap_t is the largest number of tiles that fits and whose
// dH launch (cap_t ceil(d / 256) tiles over 256 compute units) does not reach into another round, so that cutting the
// rows adds few half-empty rounds: dealt evenly, 133 tiles at d = 2048 took 2 x 3 rounds instead of 5, and the call
// 41.6 ms against 41.0 ms in one block.  At d = 5120, V = 151936, 32768 rows, two blocks of 64 tiles took the call from
// 128.1 to 116.0 ms: the recompute of half of the logits (16 ms) went, the second pass over dW cost 0.4 ms.
struct TokenBlocks {
  int cap_t;            // token tiles per block at most; 0: one block holds every row
  int b;                // this launch's block
};
// Where keeping pays, by the contraction length K that a recompute would repeat (once more for the remainders of an fp32
// head): K = 512 1990 us kept against 1811 us recomputed, 768 2440 / 2390, 1024 2866 / 2990, 2048 4620 / 5370 (4000 rows,
// V = 103936); and always where no workgroup has more than one tile to recompute, which is a latency: recomputed against kept,
// 3 tiles K = 64 71 / 74 us, 256 88 / 88, 1024 115 / 101, fp32 d = 64 102 / 85; 256 tiles K = 64 110 / 120, 512 164 / 166, 1024
// 207 / 200, fp32 d = 64 174 / 181 (not worth a rule of its own: the heads that are trained have K of 1024 and more).  Token blocks pass over
// dW and W once more per block: 33912 rows, K = 1024 27.3 ms in blocks against 24.9 ms in one, 1536 31.3 / 33.1,
// 3072 55.8 / 58.5.  And the dH contraction of a block runs over the whole vocabulary however few tiles the block has
// (the rows that remain in the last block above all), so a full block has to fill the chip well, two rounds at least.
// In blocks against in one, one tile more than whole blocks and every row active:
//   one round:  K = 1536, V = 512000  37.8 / 23.0 and 63.7 / 45.3 ms;  V = 256000  28.6 / 22.5 and 50.2 / 45.7;
//               V = 151936  31.6 / 29.1 and 58.9 / 61.8;  K = 5120, V = 512000  55.4 / 42.9 and 94.8 / 82.0
//   two rounds: K = 1536, V = 100000  21.3 / 20.1 and 43.1 / 45.2;  K = 2048, V = 151936  30.0 / 28.7 and 69.5 / 77.4;
//               K = 8192, V = 512000  96.6 / 83.3 and 303 / 353
constexpr int KEEP_MIN_K = 1024, KEEP_ANY_TILES = 256;
constexpr int BLOCK_MIN_K = 1536;
constexpr int BLOCK_MIN_ROUNDS = 2;     // rounds of a block's dH launch
constexpr int BLOCK_MIN_TILES = 16;     // smaller blocks would make the passes over dW and W dearer than a recompute
// Token tiles [t0, t0 + nt) of block k.b when `live` tiles are live.
__host__ __device__ inline void token_block(const TokenBlocks& k, int live, int& t0, int& nt) {
  if (k.cap_t <= 0) { t0 = 0; nt = k.b == 0 ? live : 0; return; }
  t0 = k.b * k.cap_t < live ? k.b * k.cap_t : live;
  nt = live - t0 < k.cap_t ? live - t0 : k.cap_t;
}

// ---- MFMA kernels ---------------------------------------------------------------------
struct FwdArgs {
  const void* W;        // [V, ldw] bf16
  const void* Hc;       // [t_cap, ldh] bf16, compacted rows, zero padded
  int w_rows, h_rows;   // rows that exist in W / Hc (loads beyond them give 0)
  int ldw, ldh;         // elements
  int K;                // contraction length (multiple of 64)
  int V;
  int tiles_v, tiles_t; // tile counts (tiles_t from t_cap; tiles beyond n_pad exit)
  int t_cap;
  float scale;          // log2(e) / tau
  const int* yc;        // [t_cap] compacted token ids (-1 on padding)
  float* zy;            // [t_cap] scaled logit of the sampled token
  float* part_m;        // [tiles_v, t_cap] each
  float* part_s;
  float* part_u;
  Kept kept;
  TokenBlocks blk;
  Ctl* ctl;             // (its step counters)
  unsigned* queue;      // [8] tile counters of this launch's queue, zero at launch
};

struct DlogitsArgs {
  const void* W;
  const void* Hc;
  int w_rows, h_rows;   // rows that exist in W / Hc (loads beyond them give 0)
  int ldw, ldh;
  int K;
  int V;
  int v0;               // first vocab row of this chunk
  int ld_s;             // leading dimension of dS   (>= chunk capacity)
  int ld_t;             // leading dimension of dS^T (>= t_cap)
  int tiles_v, tiles_t; // tiles of this chunk
  int t_cap;
  float scale;
  const int* yc;
  const float* lse2;    // [t_cap] log2-domain logsumexp
  const float* coefc;   // [t_cap] coef / tau (0 on padding)
  __bf16* dS;           // [t_cap, ld_s]
  __bf16* dST;          // [vc, ld_t]
  __bf16* dS_lo;        // fp32 heads: the bf16 remainders dS - bf16(dS), same two layouts; else null
  __bf16* dST_lo;
  const Ctl* ctl;
  unsigned* queue;      // [8] tile counters of this launch's queue, zero at launch
  unsigned* queue_lo;   // [8] the same for the launch that stores the remainders
  Rechunk rc;
  Kept kept;            // as the forward had it
  TokenBlocks blk;      // dS and dS^T hold this block's rows only
  int tiles_v_all;      // 256-row vocab tiles of the whole head
};

struct StoreArgs {
  const void* A;        // [M, lda] bf16
  const void* B;        // [N, ldb] bf16
  const void* A_lo;     // fp32 heads: bf16 remainders of A and B (same shapes; A_lo with A's leading dimension,
  const void* B_lo;     // B_lo with ldb_lo); the contraction then adds A B_lo and A_lo B to A B.  Both null otherwise.
  int ldb_lo;
  DirectRule rule;      // ctl != null: the launch whose form (b_k_rows) the rule does not choose returns at once
  int b_k_rows;         // B and B_lo are [K, ldb] instead (k runs over their rows): b_rows rows of k exist
  int a_rows, b_rows;   // rows that exist in A / B (loads beyond them give 0)
  int lda, ldb;
  int M, N, K;
  int tiles_m, tiles_n; // in tiles of 256 x 256 (StoreShape has those of the launch)
  void* C;              // [M, ldc] fp32 or bf16
  int ldc;
  int accumulate;
  int out_bf16;
  int k_from_ctl;       // contraction length = active tokens, up to whole stages (dw_stages)
  int m_from_ctl;       // row extent = active tokens: rows of C from there on, up to the padded count, are left as they are
  TokenBlocks blk;      // of the token extent
  int split_k;          // with m_from_ctl: cut K into the parts that Ctl names (DhForm), part p writes rows p n_pad + m
  int acc_rows;         // rows of C
  int wide_ok;          // tiles of 320 n can address their operand (wide_fits); of a dH see DhRule
  int dw_cap;           // > 0, with k_from_ctl: cut K into dw_split(K stages, dw_cap) parts (times three products for fp32
                        // heads); part p writes rows p slab_rows + m of `slabs`, fp32 scratch that dw_fold adds up.
                        // A single part is written to C like an unsplit one (19 of 2698 rows, d = 2304, V = 2322, bf16:
                        // through a slab and the fold 5.9 us more)
  int slab_rows;
  float* slabs;
  const Ctl* ctl;
  unsigned* queue;      // [8] tile counters of this launch's queue, zero at launch
  Rechunk rc;           // see there; rc_role 0: not a chunked launch, 1: dW of a chunk, 2: dH of a chunk
  int rc_role;
  int v0;               // first vocab row of the chunk: its rows of the whole-vocabulary dS^T, its columns of dS
};

hipError_t init_gemm_kernels();
void launch_lmhead_fwd(const FwdArgs& a, hipStream_t s);
void launch_lmhead_dlogits(const DlogitsArgs& a, hipStream_t s);
void launch_gemm_store(const StoreArgs& a, hipStream_t s);

// dW (+)= the slabs of a split dW contraction, in order
struct DwFoldArgs {
  const float* slabs;   // [parts][slab_rows, d]
  void* dW;             // [rows, d] of this chunk, fp32 or bf16
  long long n;          // rows d, a multiple of 4
  long long slab;       // elements from one slab to the next
  int dw_cap, products; // see StoreArgs
  int accumulate, out_bf16;
  const Ctl* ctl;
};
void launch_dw_fold(const DwFoldArgs& a, hipStream_t s);

// ---- row / vector kernels ----------------------------------------------------------------
struct TrlooArgs {
  const float* rewards;
  const uint8_t* valid;
  int P, K, Tmax;
  float gamma;
  double* returns_out;
  double* adv_out;
  int* group_n_out;
  int group_mean;      // 0: leave-one-out baseline (Eq. 5), 1: group-mean baseline (Eq. 3)
};
void launch_trloo(const TrlooArgs& a, hipStream_t s);

struct PrepArgs {
  // inputs
  const uint8_t* mask;       // [T] loss / row mask (nullable = all ones)
  const int* cu;             // [S+1] (nullable: no segments, every row its own weight 1)
  int S;
  const double* adv;
  const int* seg_sample;
  const uint8_t* sample_keep; // indexed like adv (nullable = keep all): 0 drops the segment
  int n_samples;             // entries of adv / sample_keep (0 = unknown: indices are not range-checked)
  const float* old_logp;
  const float* rollout_logp;
  int T, t_cap;
  int mismatch_mode;
  float geo_lo, geo_hi, veto_ratio, trunc_c, norm_override;
  // workspace
  uint8_t* flag;             // [T]
  float* c_tok;              // [T]
  float* a_tok;              // [T]
  int* rows;                 // [t_cap]
  int* pos;                  // [T]
  float* zy;                 // [t_cap]
  unsigned long long* counters; // [8]
  unsigned* queue;           // [queue_words] tile-queue counters of the persistent kernels, cleared here
  int queue_words;
  Ctl* ctl;
  // per-row outputs to clear
  float* out0; float* out1; float* out2;
  // every row active and nothing gathered: the token ids (null: left to the gather), see GatherArgs
  const int* y;
  int* yc;
  int y_offset, V;
  // fp32 heads: W and its split operand (w_elems = 0: none)
  const float* W;
  __bf16* Wc;            // [V, 3d] bf16 = [hi | lo | hi]
  size_t w_elems;
  int d;
};
void launch_prepass(const PrepArgs& a, hipStream_t s);

struct GatherArgs {
  const void* H;        // [T, d] bf16 or fp32
  const int* y;
  int d, t_cap;
  int is_f32;
  const int* rows;
  __bf16* Hc;           // [t_cap, ldh]   bf16: ldh = d;  fp32: ldh = 3d = [hi | hi | lo]
  __bf16* HcT;          // [d, ld_t] (nullable): transpose of the bf16 operand / of the hi parts
  __bf16* HcT_lo;       // [d, ld_t] (nullable, fp32 only): transpose of the lo parts
  int ld_t;             // leading dimension of HcT and HcT_lo
  int* yc;              // y - y_offset where that lies in [0, V), else -1
  int y_offset, V;      // first vocab row and number of vocab rows of the weight operand
  const Ctl* ctl;
};
void launch_gather(const GatherArgs& a, hipStream_t s);
// HcT[j, i] = Hc[i, j] over d columns of row stride ldh, for the live rows
void launch_transpose_hc(const __bf16* Hc, int ldh, __bf16* HcT, const GatherArgs& g, hipStream_t s);

// What the form of the dH launches (dh_form) goes by, beside the active rows.
struct DhRule {
  int n;                // columns of dH; 0: the call has none
  int acc_rows;         // rows of the accumulator
  int stages;           // of the first chunk's contraction
  int split_f32, wide_ok;
  Rechunk rc;
};

struct CombineArgs {
  int tiles_v, t_cap;
  const float* part_m; const float* part_s; const float* part_u;
  const float* zy;
  const int* rows;
  float* lse2;
  float* logp_out; float* ent_out; float* lse_out;      // original-row indexed, nullable
  // loss epilogue: 0 none, 1 clipped surrogate, 2 cross-entropy (l = -logp, dl/dlogp = -1)
  int with_loss;
  const float* old_logp;     // original-row indexed, nullable
  const float* c_tok; const float* a_tok;
  float eps_lo, eps_hi, inv_tau;
  float* coefc;              // [t_cap]
  float* lossterm;           // [t_cap]
  unsigned long long* counters;
  // vocab-sharded head: partials_out != null writes the merged state of the row as
  // (m, s, u, z_y) in natural-log units at [row][4] and stops; partials_in != null takes the
  // row's state from there (the state merged over all shards) instead of from part_*.
  float* partials_out;
  const float* partials_in;
  TokenBlocks blk;
  DhRule dh;                 // the first block's combine settles the form of the dH launches
  Ctl* ctl;
};
void launch_combine(const CombineArgs& a, hipStream_t s);

struct FinishArgs {
  const float* lossterm;
  const unsigned long long* counters;
  float* loss_out;
  long long* counters_out;
  const Ctl* ctl;
};

// W[v0 .. v0+cols) x d  ->  WT [d, ldt] bf16 (zeros for v >= V)
void launch_transpose_w(const void* W, int is_f32, int64_t V, int d, int ldw, int v0, int cols, int ldt, __bf16* WT,
                        const DirectRule& rule, hipStream_t s);

struct ScatterArgs {
  const float* acc;     // [t_cap, d]
  const int* pos;       // [T]
  void* dH;             // [T, d]
  int T, d;
  int out_f32;
  const Ctl* ctl;       // n_pad, and the slabs of the accumulator (dh_slabs)
};
// (the loss and the counters, and the fold of a dW split over one vocab chunk, come from the same launch; fold.n = 0: none)
void launch_scatter_dh(const ScatterArgs& a, const FinishArgs& fin, const DwFoldArgs& fold, hipStream_t s);

// RMS normalisation fused around the head (h = x rstd gamma in front of it, its backward behind dH):
// the forward is applied while the active rows are compacted, the backward while dH is scattered.
struct NormFuse {
  const void* X;        // [T, d] bf16 or fp32: the rows in front of the normalisation
  const void* gamma;    // [d] same dtype
  float eps;
  float* rstd_c;        // [t_cap] workspace: 1 / rms of every compacted row
  float* partial;       // [NORM_STRIPS, d] workspace: dgamma partial sums
  float* dgamma;        // [d] output
};
// Hc[i, :] = normalised row rows[i] of X (zeros on padding), yc[i] as launch_gather; then Hc -> HcT.
void launch_norm_gather(const GatherArgs& g, const NormFuse& n, hipStream_t s);
// dX[t, :] = RMSNorm backward of the accumulated dH row of t (zeros for rows that are not active); dgamma.
void launch_scatter_dx_norm(const ScatterArgs& a, const NormFuse& n, const FinishArgs& fin, const DwFoldArgs& fold, hipStream_t s);

// out[t] = merge(a[t], b[t]) of two per-row softmax states (m, s, u, z_y), [T][4] each.
void launch_merge_partials(const float* a, const float* b, float* out, long long T, hipStream_t s);
// logsumexp = m + ln s, log-prob = z_y - logsumexp, entropy = ln s - u / s per row; 0 on empty rows.
void launch_finish_partials(const float* parts, long long T, float* logp, float* ent, float* lse, hipStream_t s);

// ---- stages around the path -------------------------------------------------------------
struct RewardArgs {
  const uint8_t* correct;
  const float* t_reference; const float* t_kernel;
  const float* t_generated; const float* t_total;   // both nullable
  long long n;
  float cap;
  float* rewards_out;
  float* pr_out;                                    // nullable
};
void launch_turn_reward(const RewardArgs& a, hipStream_t s);

struct PrsArgs {
  const float* pr;
  const uint8_t* valid;     // nullable
  long long n;
  float tau, s;
  int hard;
  unsigned long long seed;
  uint8_t* keep_out;
  float* p_out;             // nullable
};
void launch_prs_retain(const PrsArgs& a, hipStream_t s);

constexpr int MON_BLOCKS = 1024;     // partial sums per reduced quantity
struct MonitorArgs {
  const float* logp_train; const float* logp_rollout; const float* entropy;
  const uint8_t* mask;
  long long T;
  const void* dH; int dH_f32; long long dH_elems;
  const void* dW; int dW_f32; long long dW_elems;
  double* partial;          // [6][MON_BLOCKS]
  double* out;              // [8]
};
void launch_monitors(const MonitorArgs& a, hipStream_t s);

constexpr int NORM_STRIPS = 1024;    // row strips of the RMSNorm backward (one workgroup and one dgamma partial each)
constexpr int NORM_MAX_D = 8192;     // both kernels keep a row in registers (backward: 4 x 8 columns per thread of 256)
struct NormArgs {
  const void* X;        // [T, d] bf16 or fp32
  const void* gamma;    // [d]    same dtype
  long long T;
  int d;                // multiple of 8
  float eps;
  int is_f32;
  // forward
  void* H;              // [T, d] same dtype
  float* rstd_out;      // [T], nullable
  // backward
  const void* dH;       // [T, d] same dtype
  void* dX;             // [T, d] same dtype
  float* partial;       // [NORM_STRIPS, d]
  float* dgamma;        // [d]
  int strips;           // partials in use
};
void launch_rmsnorm_fwd(const NormArgs& a, hipStream_t s);
void launch_rmsnorm_bwd(const NormArgs& a, hipStream_t s);

void launch_fill_f32(float* p, size_t n, float v, hipStream_t s);
void launch_fill_zero_bytes(void* p, size_t nbytes, hipStream_t s);   // nbytes multiple of 4

}  // namespace pg
