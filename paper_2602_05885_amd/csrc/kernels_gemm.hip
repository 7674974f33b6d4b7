// The MFMA kernels of the policy-gradient head (see gemm_core.h for the tile engine), and the kernel that forms dS
// from kept logits.
//
// Accumulator layout they all rely on: acc[i][j][r] of lane l is
//   engine row     wm*64  + i*16 + 4*(l>>4) + r      (i < 4, r < 4; the fifth of a wide tile of the store kernel, i = 4: 256 + wm*16 + 4*(l>>4) + r)
//   engine column  wn*128 + j*16 + (l & 15)          (j < 8; in the forward j*32 + wn*16 + (l & 15))
// so one lane holds 16 rows (20 wide) of each of its 8 columns, and the four 16-lane groups of a
// wavefront hold the other 48 (60) rows of the same columns.  The two logits kernels put the
// vocabulary on the rows (a token's statistics then reduce inside a lane first); the store
// kernel puts the output's contiguous dimension there (4 consecutive elements per lane).
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "kernels.h"
#include "gemm_core.h"

namespace pg {

extern __shared__ __attribute__((aligned(16))) char g_smem[];

// Softmax partial state in the log2 domain: t = z * log2(e) / tau,
// m = max t, s = sum 2^(t-m), u = sum 2^(t-m) (t-m).
__device__ __forceinline__ void merge_state(float& m, float& s, float& u, float m2, float s2, float u2) {
  const float mm = fmaxf(m, m2);
  const float a1 = __builtin_amdgcn_exp2f(m - mm), a2 = __builtin_amdgcn_exp2f(m2 - mm);
  u = a1 * (u + (m - mm) * s) + a2 * (u2 + (m2 - mm) * s2);
  s = a1 * s + a2 * s2;
  m = mm;
}

// Two registers after an exchange of lanes.  swap_halves: a = {first half of a, first half of b}, b = {second half of a, second
// half of b}.  swap_rows: a = rows {a0, b0, a2, b2}, b = rows {a1, b1, a3, b3} of 16 lanes.
struct Two { float a, b; };
__device__ __forceinline__ Two swap_halves(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  const unsigned x = r[0], y = r[1];      // (a bit cast of the vector's element itself would take element 0)
  return {__builtin_bit_cast(float, x), __builtin_bit_cast(float, y)};
}
__device__ __forceinline__ Two swap_rows(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  const unsigned x = r[0], y = r[1];      // (a bit cast of the vector's element itself would take element 0)
  return {__builtin_bit_cast(float, x), __builtin_bit_cast(float, y)};
}
// Finite stand-in for -inf (keeps 0 * (t - m) finite).  A power of two, so that its product
// with the logit scale is exact and "t - max" of an all-masked column is exactly zero.
constexpr float NEG_BIG = -0x1p100f;

// ------------------------------------------------------------------------------------
// Forward: a tile is 256 vocab rows x 256 compacted tokens.  What leaves the kernel is one (m, s, u) triple
// per token and vocab tile, plus the scaled logit of the sampled token, and for the loss calls the
// accumulators of the tiles that are kept for the backward (Kept in kernels.h).
// Persistent: one workgroup per compute unit takes tiles from the XCD-aware queue (gemm_core.h)
// until none is left.  The operand loads of the next tile run ahead through the tile boundary
// (mainloop_stream), so the statistics epilogue of a tile executes while the first two stages of
// the next one arrive, and a tile costs no launch, no cold prologue and no drain.  A workgroup
// always knows its next tile (the loads need it) and has the claim for the one after that in
// flight.  LDS: the two stage buffers, then the cross-wavefront merge array, the sampled-token ids
// of the tile (double-buffered; loaded one tile ahead so that the epilogue waits on no global load)
// and the words that hand the claimed tiles to all wavefronts.
// ------------------------------------------------------------------------------------
constexpr int FWD_RED_OFF = 2 * STAGE_BYTES;                 // [m, s, u][WM][256 tokens] floats
constexpr int FWD_STASH_OFF = FWD_RED_OFF + WM * 256 * 3 * 4; // [2][256] ints
constexpr int FWD_CLAIM_OFF = FWD_STASH_OFF + 2 * 256 * 4;    // [4] ints
constexpr int FWD_LDS_BYTES = FWD_CLAIM_OFF + 16;

// Where a kept tile holds 16-column group c of 64-row group wm, in units of f32x4: GM accumulators of 64 lanes.
__device__ __forceinline__ int kept_column(int wm, int c) { return (wm * (BN / 16) + c) * (GM * 64); }

// PROBE = true (the stand-alone measurement tool only) records wall-clock and shader-clock stamps of
// tiles PROBE_FIRST .. PROBE_FIRST + PROBE_TILES - 1 of every workgroup in tl[wg][tile][4] (main loop
// start, main loop end, epilogue end, shader clock at the epilogue's end) and lets the tool switch the
// stealing between XCDs off; the library instantiates PROBE = false, which compiles to none of it.
constexpr int PROBE_FIRST = 150, PROBE_TILES = 16;

template <bool PROBE>
__device__ __forceinline__ void lmhead_fwd_body(FwdArgs a, bool steal, unsigned long long* tl) {
  const Ctl ctl = *a.ctl;
  int t0, nt;
  token_block(a.blk, ctl.n_pad / BN, t0, nt);
  const int tiles_t = min(a.tiles_t, nt);                      // live token tiles: known only on the device
  if (tiles_t <= 0) return;
  const int live_rows = ctl.n_active - t0 * BN;                // of this block and those behind it
  a.Hc = static_cast<const char*>(a.Hc) + (size_t)t0 * BN * a.ldh * 2; a.h_rows = min(a.h_rows - t0 * BN, live_rows);
  a.yc += t0 * BN; a.zy += t0 * BN;
  a.part_m += t0 * BN; a.part_s += t0 * BN; a.part_u += t0 * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  TileQueue Q;
  const bool two = a.tiles_v * tiles_t > (int)gridDim.x;      // (of at most one tile per workgroup there is no second)
  // Two tiles for few workgroups (TileQueue): not where logits are parked, K is long and the last token tile is a short one: a launch of
  // which a part costs less than half is over sooner where no workgroup has two whole tiles.  One for everybody / two for few, d = 4096,
  // 544 rows, 285 tiles 141 / 158 us, 375 tiles 173 / 179, d = 5120 179 / 196 and 213 / 223, 288 rows, 398 tiles 225 / 236; but d = 2048, 288 rows, 316
  // tiles 90 / 77, 1312 rows, 318 tiles 97 / 91, and all token tiles whole, d = 4096, 1024 rows, 260 tiles 174 / 165, d = 5120, 256 rows, 316 tiles 268 / 247.
  const bool few = a.kept.tiles == nullptr || a.K < 3072 || fwd_nj(live_rows - (tiles_t - 1) * BN, tiles_t) == GN;
  Q.init(a.queue, a.tiles_v * tiles_t, 0, two ? 2 : 1, few);
  const int kept_v = kept_vocab_tiles(a.kept, a.tiles_v, tiles_t);
  // Tile order: all token tiles of a vocab tile in a row, unless tiles are parked.  Forward-only calls, vocabulary fastest
  // against tokens fastest: d = 4096, 768 rows 722 -> 706 us, 4100 rows 3725 -> 3705, 16384 rows 13.95 -> 13.65 ms; d = 5120, 131072
  // rows 142.4 -> 138.7 ms (W is read from HBM once per panel of eight token tiles, and meets in the L2 more often).  The
  // forward of a loss call that keeps its logits is the other way round: d = 5120, 12000 rows 13.73 against 14.09 ms, d = 4096, 2869
  // rows 2.71 against 2.75 (every tile ends in 256 KiB of stores, which drives the tiles further apart in time).
  const bool tokens_first = a.kept.tiles == nullptr;
  const bool whole = tokens_first && !short_tile_pays(tiles_t, a.K, a.tiles_v * tiles_t, (int)gridDim.x);
  float* red = reinterpret_cast<float*>(g_smem + FWD_RED_OFF);
  int* stash = reinterpret_cast<int*>(g_smem + FWD_STASH_OFF);
  volatile int* claim = reinterpret_cast<volatile int*>(g_smem + FWD_CLAIM_OFF);

  // the first two tiles
  const bool all_dealt = Q.total <= 2 * (int)gridDim.x;
  int b_cur = Q.entry(blockIdx.x, 0), b_nxt = two ? Q.entry(blockIdx.x, 1) : -1;
  if (!all_dealt && (b_cur < 0 || b_nxt < 0)) {      // (an XCD with a short share: others may have more)
    if (tid == 0) {
      claim[0] = b_cur < 0 ? Q.resolve(Q.ticket(), steal) : b_cur;
      claim[1] = Q.resolve(Q.ticket(), steal);
    }
    __syncthreads();
    b_cur = __builtin_amdgcn_readfirstlane(claim[0]); b_nxt = __builtin_amdgcn_readfirstlane(claim[1]);
  }
  InStep in_step;
  in_step.init(a.ctl->step, Q.home, (int)gridDim.x, a.K / BK, a.kept.tiles == nullptr && Q.total >= InStep::ROUNDS * (int)gridDim.x);
  if (b_cur < 0) {
    if (tid == 0) in_step.count(false);
    return;
  }
  int tm, tn, tm1 = 0, tn1 = 0;
  map_tile(b_cur, a.tiles_v, tiles_t, tm, tn, tokens_first);
  bool more = b_nxt >= 0;
  if (more) map_tile(b_nxt, a.tiles_v, tiles_t, tm1, tn1, tokens_first);
  OperandLanes VA, VB;
  VA.init(a.ldw, tid);
  VB.init(a.ldh, tid);
  const bool ahead = a.K / BK >= 2;        // single-stage tiles cannot run two stages ahead
  TileSrc A0, B0, A1, B1;
  A0.set(a.W, a.w_rows, tm * BM, a.ldw, 0u);
  B0.set(a.Hc, a.h_rows, tn * BN, a.ldh, 0u);
  A1.set(a.W, (more && ahead) ? a.w_rows : 0, tm1 * BM, a.ldw, 0u);
  B1.set(a.Hc, (more && ahead) ? a.h_rows : 0, tn1 * BN, a.ldh, 0u);
  const int nk = a.K / BK;
  if (tid < BN) stash[tid] = a.yc[tn * BN + tid];     // visible to everybody behind the main loop's barriers
  int par = 0;

  for (int n = 0;; ++n) {
    const int* ys = stash + (n & 1) * BN;
    f32x4 acc[GM][GN];
    zero_acc(acc);
    const bool probe = PROBE && tl && tid == 0 && n >= PROBE_FIRST && n < PROBE_FIRST + PROBE_TILES;
    unsigned long long* stamp = probe ? tl + ((size_t)blockIdx.x * PROBE_TILES + (n - PROBE_FIRST)) * 4 : nullptr;
    if (probe) stamp[0] = wall_clock64();
    const int nj = whole ? GN : fwd_nj(live_rows - tn * BN, tiles_t);
    mainloop_stream(VA, VB, A0, B0, A1, B1, nk, n == 0 || !ahead, par, nj, g_smem, acc);
    par = (par + nk) & 1;
    if (probe) stamp[1] = wall_clock64();
    if (!ahead) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    // claim the tile after the next one: issued here, behind the main loop's last loads (memory
    // operations return in order, an atomic in front of them would hold up their completion), and
    // picked up at the end of the epilogue.  (Left uninitialised on the other threads on purpose: a
    // merged value would make the compiler wait for the atomic right here.)
    unsigned ticket;
    if (tid == 0) {
      if (more) ticket = Q.ticket();
      in_step.count(more);
    }
    // the next tile's token ids: fetched now, parked in LDS before this tile's stores are issued, so
    // that neither this epilogue nor the next one waits on memory
    int y_next = 0;
    if (more && tid < BN) y_next = a.yc[tn1 * BN + tid];

    const int v_base = tm * BM + wm * WROWS;            // first vocab row of this wavefront's block
    const bool ragged = (tm * BM + BM > a.V);
    // park the accumulators for the backward, 1 KiB per instruction, before the statistics, so that the stores drain
    // under them (d = 5120, V = 151936, all tiles kept: 609 -> 640 us at 768 rows; at 32768 rows in two token blocks
    // 36.4 -> 36.5 ms)
    if (tm < kept_v) {
      f32x4* kp = reinterpret_cast<f32x4*>(a.kept.tiles + ((size_t)tm * tiles_t + tn) * KEPT_TILE_FLOATS) + kept_column(wm, wn) + lane;
#pragma unroll
      for (int j = 0; j < GN; ++j) {
        if (j >= nj) continue;
#pragma unroll
        for (int i = 0; i < GM; ++i) __builtin_nontemporal_store(acc[i][j], kp + (kept_column(0, j * WN) + i * 64));
      }
    }
    // Statistics of this wavefront's 64 vocab rows, per token: their maximum first, known to all four lanes of a token, so that
    // the sums over the lanes are plain additions.  Cross-lane steps are half-wavefront and row swaps (no LDS latency); a swap
    // of two different values reduces both at once.  Against merging lane-local states through the LDS unit, main loops at the same
    // place (place_loop): forward only, d = 5120, 32768 rows 34.5 -> 34.1 ms, d = 4096, 16384 rows 13.93 -> 13.68, 4100 rows 3758 -> 3706 us.  (Without any
    // statistics 33.3, 13.23 and 3563.)
    float mx[GN];
#pragma unroll
    for (int j = 0; j < GN; ++j) {
      float mr = NEG_BIG;
#pragma unroll
      for (int i = 0; i < GM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (ragged && (v_base + i * 16 + acc_row(r, lane) >= a.V)) acc[i][j][r] = NEG_BIG;
          mr = fmaxf(mr, acc[i][j][r]);
        }
      const Two h = swap_halves(mr, mr);
      mr = fmaxf(h.a, h.b);
      const Two q = swap_rows(mr, mr);
      mx[j] = fmaxf(q.a, q.b) * a.scale;
    }
#pragma unroll
    for (int j0 = 0; j0 < GN; j0 += 2) {
      float su[2];          // lanes 0..31 s, lanes 32..63 u of token column j0 + h
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int j = j0 + h;
        const float nmx = -mx[j];
        float s = 0.f, u = 0.f;
#pragma unroll
        for (int i = 0; i < GM; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float dlt = fmaf(acc[i][j][r], a.scale, nmx);
            const float e = __builtin_amdgcn_exp2f(dlt);
            s += e;
            u = fmaf(e, dlt, u);
          }
        const Two x = swap_halves(s, u);
        su[h] = x.a + x.b;
        const int tok_l = stream_col(j, wn, lane);
        const int ytok = ys[tok_l];
        const int yrel = ytok - v_base;
        const bool mine = (yrel >= 0) && (yrel < WROWS) && (ytok < a.V) && (((yrel >> 2) & 3) == (lane >> 4));
        if (__any(mine)) {
          float zy = 0.f;
#pragma unroll
          for (int i = 0; i < GM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (yrel == i * 16 + acc_row(r, lane)) zy = acc[i][j][r] * a.scale;
          if (mine) a.zy[tn * BN + tok_l] = zy;
        }
      }
      // rows of 16 lanes: s of j0, s of j0 + 1, u of j0, u of j0 + 1
      const Two y = swap_rows(su[0], su[1]);
      const int tok_l = stream_col(j0 + ((lane >> 4) & 1), wn, lane);
      red[(1 + (lane >> 5)) * (WM * BN) + wm * BN + tok_l] = y.a + y.b;
      if (lane < 32) red[wm * BN + tok_l] = lane < 16 ? mx[j0] : mx[j0 + 1];
    }
    if (tid == 0) {
      claim[2] = more ? Q.resolve(ticket, steal) : -1;
      in_step.wait();
    }
    // LDS-only synchronisation: a full __syncthreads() would also wait for the next tile's loads
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int b_nn = __builtin_amdgcn_readfirstlane(claim[2]);
    if (tid < BN) {
      stash[((n + 1) & 1) * BN + tid] = y_next;
      const float* p = red + tid;
      float m = p[0], s = p[WM * BN], u = p[2 * WM * BN];
#pragma unroll
      for (int w = 1; w < WM; ++w) merge_state(m, s, u, p[w * BN], p[(WM + w) * BN], p[(2 * WM + w) * BN]);
      const size_t o = (size_t)tm * a.t_cap + (size_t)tn * BN + tid;
      a.part_m[o] = m; a.part_s[o] = s; a.part_u[o] = u;
    }
    if (probe) { stamp[2] = wall_clock64(); stamp[3] = clock64(); }
    if (!more) break;
    tm = tm1; tn = tn1;
    A0.set(a.W, a.w_rows, tm * BM, a.ldw, 0u);
    B0.set(a.Hc, a.h_rows, tn * BN, a.ldh, 0u);
    more = b_nn >= 0;
    if (more) map_tile(b_nn, a.tiles_v, tiles_t, tm1, tn1, tokens_first);
    A1.set(a.W, (more && ahead) ? a.w_rows : 0, tm1 * BM, a.ldw, 0u);
    B1.set(a.Hc, (more && ahead) ? a.h_rows : 0, tn1 * BN, a.ldh, 0u);
  }
}

__global__ __launch_bounds__(NTHREADS) void lmhead_fwd_kernel(FwdArgs a) { lmhead_fwd_body<false>(a, true, nullptr); }

// ------------------------------------------------------------------------------------
// Backward recompute (of logits that were not kept): the same contraction, finished with
//   dS[t,v] = c_t * (onehot(y_t)[v] - 2^(t2 - lse2_t)),  c_t = coef_t / tau,
// rounded to bf16 and written for one vocab chunk in both orientations
// (dS [t_cap, ld_s] for dH, dS^T [vc, ld_t] for dW).  Both go through an LDS transposition
// stage so that global stores are 16 B per lane and 512 B per row.
// ------------------------------------------------------------------------------------
// Where the persistent kernels keep the word that hands a claimed tile to all wavefronts: behind the
// recompute epilogue's staging area (the largest LDS user).
constexpr int CLAIM_OFF = GEMM_LDS_BYTES;
constexpr int PERSISTENT_LDS_BYTES = CLAIM_OFF + 16;
constexpr int STORE_CLAIM_OFF = WIDE_LDS_BYTES, STORE_LDS_BYTES = STORE_CLAIM_OFF + 16;

// Takes tiles from the queue until it has none for this workgroup: with steal = false the XCD's own
// share only, with steal = true the own share first and then whatever is left on other XCDs.
// tile(b, after_loop, before_stores) computes the tile with workgroup index b (TileQueue::encode) and
// calls the two hooks once each, on every thread: after_loop behind its main loop's last load (the
// claim for the next tile is issued there: memory operations return in order, an atomic in front of
// the loads would hold up their completion), before_stores at a point that at least one workgroup
// barrier separates from the end of the tile and that lies before the tile's own global stores
// (the claim is picked up there; later it would wait for those stores to complete).
template <class TileFn>
__device__ __forceinline__ void drain_queue(const TileQueue& Q, bool steal, volatile int* claim, TileFn&& tile) {
  const int tid = threadIdx.x;
  const bool all_dealt = Q.total <= (int)gridDim.x;
  int b = Q.entry(blockIdx.x, 0);
  if (b < 0 && !all_dealt) b = queue_broadcast(claim, tid == 0 ? Q.resolve(Q.ticket(), steal) : 0);
  while (b >= 0) {
    // (ticket is left uninitialised on the other threads on purpose: a merged value would make the
    // compiler wait for the atomic where it is issued)
    unsigned ticket;
    tile(b, [&]() { if (tid == 0 && !all_dealt) ticket = Q.ticket(); }, [&]() { if (tid == 0 && !all_dealt) claim[0] = Q.resolve(ticket, steal); });
    if (all_dealt) return;
    b = __builtin_amdgcn_readfirstlane(claim[0]);
    // every wavefront is done with the tile's LDS before the next tile's loads land in it
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
}

// Workgroup barrier that orders LDS accesses only: vector memory operations in flight are not waited for.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// What dS needs of one token column.
struct DsColumn {
  float c, k2;
  uint32_t sgn;
  int y;
  __device__ __forceinline__ DsColumn(const DlogitsArgs& a, int tok) {
    c = a.coefc[tok];
    k2 = __builtin_amdgcn_logf(fabsf(c)) - a.lse2[tok];
    sgn = c > 0.f ? 0x80008000u : 0u;
    y = a.yc[tok];
  }
};

// dS of one MFMA tile column (GM tiles of 4 rows per lane) from its logits.
// dS = c (onehot - p) is formed as  -sign(c) 2^(t2 - lse2 + log2|c|)  for every element (one fma
// and one exp2 each; c = 0 gives 2^-inf = 0), the one-hot term c is added to the single element
// that holds the sampled token (rare, wave-uniform branch), and the sign goes on with the bf16
// packing.  Fp32 heads also take the remainders dS - bf16(dS).
enum DsPart { DS_VALUE, DS_REST, DS_EITHER };       // DS_EITHER: `rest` says which at run time
template <DsPart PART>
__device__ __forceinline__ void ds_pack(const DlogitsArgs& a, const DsColumn& col, int v_base, const f32x4 (&z)[GM],
                                        uint32_t (&pk)[GM][2], bool rest = false) {
  const int lane = threadIdx.x & 63;
  const bool ragged = v_base + WROWS > a.V;
  const int yrel = col.y - v_base;
  const bool mine = (yrel >= 0) && (yrel < WROWS) && (((yrel >> 2) & 3) == (lane >> 4));
  const bool any_mine = __any(mine);
#pragma unroll
  for (int i = 0; i < GM; ++i) {
    float g[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) g[r] = __builtin_amdgcn_exp2f(fmaf(z[i][r], a.scale, col.k2));
    if (any_mine) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (yrel == i * 16 + acc_row(r, lane)) g[r] -= fabsf(col.c);     // sign is applied below
    }
    if (ragged) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (v_base + i * 16 + acc_row(r, lane) >= a.V) g[r] = 0.f;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
      bf16x2 two;
      two[0] = (__bf16)g[2 * h];
      two[1] = (__bf16)g[2 * h + 1];
      if constexpr (PART == DS_REST) {
        two[0] = (__bf16)(g[2 * h] - (float)two[0]);
        two[1] = (__bf16)(g[2 * h + 1] - (float)two[1]);
      }
      if constexpr (PART == DS_EITHER) {
        two[0] = (__bf16)(g[2 * h] - (rest ? (float)two[0] : 0.f));
        two[1] = (__bf16)(g[2 * h + 1] - (rest ? (float)two[1] : 0.f));
      }
      pk[i][h] = __builtin_bit_cast(uint32_t, two) ^ col.sgn;
    }
  }
}

// ---- orientation 1: dS[tok][v], staged as rows of 256 v (wn: 128-token half of the staging area) ----
template <int HALVES, int C>
__device__ __forceinline__ void ds_stage_rows(const uint32_t (&pk)[GM][C][2], char* st, int wm, int wn, int lane) {
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int tok_l = (HALVES > 1 ? wn * WCOLS : 0) + j * 16 + (lane & 15);
#pragma unroll
    for (int i = 0; i < GM; ++i) {
      const int v_l = wm * WROWS + i * 16 + ((lane >> 4) << 2);
      *reinterpret_cast<uint2*>(st + tok_l * EPI_STRIDE + v_l * 2) = make_uint2(pk[i][j][0], pk[i][j][1]);
    }
  }
}

// ---- orientation 2: dS^T[v][tok], staged as rows of tokens ----
// A quad of lanes holds a 4 (vocab rows) x 4 (tokens) block, one token per lane.  Two
// butterfly exchanges inside the quad turn it so that lane q holds row q of all four tokens,
// which then goes to LDS as one 8-byte store (instead of sixteen 2-byte ones per block).
template <int C>
__device__ __forceinline__ void ds_stage_cols(const uint32_t (&pk)[GM][C][2], char* st, int stride, int wm, int wn, int lane) {
  const int q = lane & 3;
  const uint32_t sel = (q & 1) ? 0x03020706u : 0x05040100u;   // v_perm byte selectors, see below
  const bool upper = q >= 2;
  const int row_l = wm * WROWS + ((lane >> 4) << 2) + q;
  const int tok0_l = wn * WCOLS + (((lane & 15) >> 2) << 2);
#pragma unroll
  for (int j = 0; j < C; ++j) {
#pragma unroll
    for (int i = 0; i < GM; ++i) {
      const uint32_t w0 = pk[i][j][0], w1 = pk[i][j][1];        // rows (0,1), (2,3) of my token
      // neighbour in the lane pair: even lanes keep the even row of both tokens, odd lanes the odd row
      const uint32_t p0 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w0, 0xB1, 0xf, 0xf, false);
      const uint32_t p1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w1, 0xB1, 0xf, 0xf, false);
      const uint32_t x0 = __builtin_amdgcn_perm(p0, w0, sel);   // row (q&1),   tokens of my pair
      const uint32_t x1 = __builtin_amdgcn_perm(p1, w1, sel);   // row 2+(q&1), tokens of my pair
      // other pair of the quad: lanes 0,1 collect rows 0,1 and lanes 2,3 rows 2,3 of all four tokens
      const uint32_t send = upper ? x0 : x1;
      const uint32_t recv = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0x4E, 0xf, 0xf, false);
      const uint2 two = upper ? make_uint2(recv, x1) : make_uint2(x0, recv);
      *reinterpret_cast<uint2*>(st + (row_l + i * 16) * stride + (tok0_l + j * 16) * 2) = two;
    }
  }
}

// ROWS staged rows of ROW_BYTES (LDS pitch STRIDE) -> dst (row pitch ld elements), 16 bytes per lane.
template <int ROWS, int ROW_BYTES, int STRIDE, int THREADS>
__device__ __forceinline__ void ds_store(const char* st, __bf16* dst, int ld, int tid) {
  constexpr int LANES = ROW_BYTES / 16, STEP = THREADS / LANES;
  const int chunk = tid % LANES, r0 = tid / LANES;
#pragma unroll 4
  for (int ps = 0; ps < ROWS / STEP; ++ps) {
    const int row = r0 + ps * STEP;
    const i32x4 v = *reinterpret_cast<const i32x4*>(st + row * STRIDE + chunk * 16);
    __builtin_nontemporal_store(v, reinterpret_cast<i32x4*>(dst + (size_t)row * ld + chunk * 8));
  }
}

template <bool LO, class AfterLoop, class BeforeStores>
__device__ __forceinline__ void dlogits_tile(const DlogitsArgs& a, int tm, int tn, AfterLoop&& after_loop,
                                             BeforeStores&& before_stores) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;

  TileLoader LA, LB;
  LA.init(a.W, a.w_rows, a.v0 + tm * BM, a.ldw, 0u, tid);
  LB.init(a.Hc, a.h_rows, tn * BN, a.ldh, 0u, tid);
  f32x4 acc[GM][GN];
  zero_acc(acc);
  mainloop(LA, LB, a.K / BK, g_smem, acc);
  after_loop();

  // pk[i][j][h] holds rows 2h, 2h+1 of this lane's 4-row group as a bf16 pair.
  uint32_t pk[GM][GN][2];
#pragma unroll
  for (int j = 0; j < GN; ++j) {
    f32x4 z[GM];
#pragma unroll
    for (int i = 0; i < GM; ++i) z[i] = acc[i][j];
    const DsColumn col(a, tn * BN + wn * WCOLS + j * 16 + (lane & 15));
    uint32_t p[GM][2];
    ds_pack<LO ? DS_REST : DS_VALUE>(a, col, a.v0 + tm * BM + wm * WROWS, z, p);
#pragma unroll
    for (int i = 0; i < GM; ++i) { pk[i][j][0] = p[i][0]; pk[i][j][1] = p[i][1]; }
  }

  __bf16* const dS = (LO ? a.dS_lo : a.dS) + ((size_t)tn * BN) * a.ld_s + (size_t)tm * BM;
  __bf16* const dST = (LO ? a.dST_lo : a.dST) + ((size_t)tm * BM) * a.ld_t + (size_t)tn * BN;
  ds_stage_rows<WN>(pk, g_smem, wm, wn, lane);
  before_stores();
  lds_barrier();
  ds_store<256, 512, EPI_STRIDE, NTHREADS>(g_smem, dS, a.ld_s, tid);
  lds_barrier();
  ds_stage_cols(pk, g_smem, EPI_STRIDE_T, wm, wn, lane);
  lds_barrier();
  ds_store<256, 512, EPI_STRIDE_T, NTHREADS>(g_smem, dST, a.ld_t, tid);
}

// Leading vocab tiles of this chunk whose logits the forward kept.
__device__ __forceinline__ int kept_in_chunk(const DlogitsArgs& a, int tiles_t) {
  return imin(imax(kept_vocab_tiles(a.kept, a.tiles_v_all, tiles_t) - a.v0 / BM, 0), a.tiles_v);
}

template <bool LO>
__global__ __launch_bounds__(NTHREADS) void lmhead_dlogits_kernel(DlogitsArgs a) {
  const Ctl ctl = *a.ctl;
  int ld_t_all;
  if (rechunk_all(a.rc, ctl.n_pad, ld_t_all)) {         // few active rows: the first chunk's launch covers the vocabulary
    if (a.rc.chunk > 0) return;
    a.v0 = 0; a.tiles_v = a.rc.tiles_v_all; a.ld_s = a.rc.ld_s_all; a.ld_t = ld_t_all;
  }
  const int tiles_t = min(a.tiles_t, ctl.n_pad / BN);   // live token tiles: known only on the device
  a.h_rows = min(a.h_rows, ctl.n_active);
  const int skip = kept_in_chunk(a, tiles_t);           // these are finished by dlogits_kept_kernel
  a.v0 += skip * BM; a.tiles_v -= skip;
  a.dS += skip * BM; a.dST += (size_t)skip * BM * a.ld_t;
  if (LO) { a.dS_lo += skip * BM; a.dST_lo += (size_t)skip * BM * a.ld_t; }
  if (a.tiles_v == 0 || tiles_t == 0) return;
  TileQueue Q;
  Q.init(a.queue, a.tiles_v * tiles_t, 0, 1);
  volatile int* claim = reinterpret_cast<volatile int*>(g_smem + CLAIM_OFF);
  // persistent: one workgroup per compute unit takes tiles from the XCD-aware queue until none is left
  drain_queue(Q, true, claim, [&](int b, auto&& after_loop, auto&& before_stores) {
    int tm, tn;
    map_tile(b, a.tiles_v, tiles_t, tm, tn);
    dlogits_tile<LO>(a, tm, tn, after_loop, before_stores);
  });
}

// dS of the vocab tiles whose logits the forward kept: the epilogue of the recompute with the accumulators
// read back instead of computed.  Bound by HBM (256 KiB read and 256 KiB written per 256 x 256 tile); a
// workgroup takes 256 vocab rows x 128 tokens, i.e. half of a kept tile, so that two fit a
// compute unit (72 KiB of LDS each) and one's loads run under the other's stores.  Measured at d = 5120,
// V = 151936: 768 rows 119 us (recompute 639 us; 7.8 TB/s, part of the kept tiles still sits in the
// memory-side cache), 32768 rows in two token blocks 7.7 ms, 5.2 TB/s, above the rate of a plain copy (recompute
// 36 ms).  Requesting a quarter or half of the next half tile before the stores: 126 us at 768 rows.
constexpr int KEPT_THREADS = 256;
// C: 16-column groups of an item.  Rows of dS^T in LDS: 16 C tokens and a pad (72 dwords for 128 tokens, see EPI_STRIDE_T).
constexpr int kept_stride_t(int C) { return C * 32 + (C == GN ? 32 : 16); }
constexpr int kept_lds_bytes(int C) { return 256 * kept_stride_t(C) > C * 16 * EPI_STRIDE ? 256 * kept_stride_t(C) : C * 16 * EPI_STRIDE; }
static_assert(2 * kept_lds_bytes(GN) <= 160 * 1024, "LDS budget");

// FEW: of at most two token tiles or two rounds of workgroups (or an fp32 head), where a group that was not parked is not loaded.  Elsewhere
// another one's is, as the branch holds the other loads up: d = 5120, 12000 rows 2.80 -> 2.71 ms, 768 rows 187 -> 179 us, 1536 rows, 942 tiles 103.6 -> 99.5;
// but 24 rows of d = 4096 50 -> 53 us, 1536 rows, 348 tiles 38.6 -> 40.0, 1312 rows, 318 tiles 36.0 -> 37.6, fp32 64 x 1000, 1024 rows 15.3 -> 16.5 us.
// Items of 32 tokens (C = KEPT_SMALL) where items of 128 leave most compute units idle: an item is a chain of latencies (loads, LDS, stores of one
// compute unit), whose length goes with its tokens.  128 / 32 tokens: fp32 64 x 1000, 512 rows (32 half tiles) 15.5 / 9.3 us, 1024 rows (64) 15.5 / 8.6..11.3;
// 200 rows, d = 1024, V = 8000 (64) 13.3 / 9.7; 700 x 512 x 3000 (72) 14.1 / 12.2; beyond, 32 tokens' stores lose (64-byte pieces of dS^T): 600 x 1024 x 12000
// (282) 17.6 / 23.9, 1024 x 256 x 4000 fp32 (256) 16.1 / 20.3.  Items of 64 tokens lie between the two on either side (13.0 at 64, 14.9 at 256).
constexpr int KEPT_SMALL = 2, KEPT_SMALL_HALVES = 96;
template <bool SPLIT, bool FEW, int C>
__global__ __launch_bounds__(KEPT_THREADS, 2) void dlogits_kept_kernel(DlogitsArgs a) {
  const Ctl ctl = *a.ctl;
  int ld_t_all;
  if (rechunk_all(a.rc, ctl.n_pad, ld_t_all)) {
    if (a.rc.chunk > 0) return;
    a.v0 = 0; a.tiles_v = a.rc.tiles_v_all; a.ld_s = a.rc.ld_s_all; a.ld_t = ld_t_all;
  }
  int t0, nt;
  token_block(a.blk, ctl.n_pad / BN, t0, nt);
  const int tiles_t = min(a.tiles_t, nt);
  if (tiles_t <= 0) return;
  a.yc += t0 * BN; a.lse2 += t0 * BN; a.coefc += t0 * BN;
  constexpr int PER_TILE = BN / 16 / C;             // items of a kept tile
  const int items = PER_TILE * kept_in_chunk(a, tiles_t) * tiles_t, total = SPLIT ? 2 * items : items;
  const int tid = threadIdx.x, lane = tid & 63, wm = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tm0 = a.v0 / BM;
  f32x4 acc[GM][C];
  // 16-column groups [C part, C part + C) of a kept tile; those beyond the live ones were not parked and count as zero
  auto fetch = [&](int tile, int part, int groups) {
    const f32x4* kp = reinterpret_cast<const f32x4*>(a.kept.tiles + ((size_t)tm0 * tiles_t + tile) * KEPT_TILE_FLOATS) + kept_column(wm, part * C) + lane;
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int i = 0; i < GM; ++i) {
        if (FEW) {
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (j < groups) acc[i][j] = __builtin_nontemporal_load(kp + (kept_column(0, j) + i * 64));
        } else {
          const f32x4 v = __builtin_nontemporal_load(kp + (kept_column(0, j < groups ? j : 0) + i * 64));
          acc[i][j] = j < groups ? v : f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
  };
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const bool rest = SPLIT && item >= items;         // fp32 heads: the remainders as items of their own
    const int h = rest ? item - items : item;
    const int tile = h / PER_TILE, part = h % PER_TILE, tm = tile / tiles_t, tn = tile - tm * tiles_t;
    const int groups = WN * fwd_nj(ctl.n_active - (t0 + tn) * BN, tiles_t) - part * C;
    if (groups <= 0) continue;                        // columns without a row: nobody reads their dS
    fetch(tile, part, groups);
    const int col0 = tn * BN + part * (16 * C);
    const size_t o_s = (size_t)col0 * a.ld_s + (size_t)tm * BM, o_t = ((size_t)tm * BM) * a.ld_t + col0;
    uint32_t pk[GM][C][2];
#pragma unroll
    for (int j = 0; j < C; ++j) {
      f32x4 z[GM];
#pragma unroll
      for (int i = 0; i < GM; ++i) z[i] = acc[i][j];
      const DsColumn col(a, col0 + j * 16 + (lane & 15));
      uint32_t p[GM][2];
      ds_pack<SPLIT ? DS_EITHER : DS_VALUE>(a, col, a.v0 + tm * BM + wm * WROWS, z, p, rest);
#pragma unroll
      for (int i = 0; i < GM; ++i) { pk[i][j][0] = p[i][0]; pk[i][j][1] = p[i][1]; }
    }
    ds_stage_rows<1>(pk, g_smem, wm, 0, lane);
    lds_barrier();
    ds_store<C * 16, 512, EPI_STRIDE, KEPT_THREADS>(g_smem, (rest ? a.dS_lo : a.dS) + o_s, a.ld_s, tid);
    lds_barrier();
    ds_stage_cols(pk, g_smem, kept_stride_t(C), wm, 0, lane);
    lds_barrier();
    ds_store<256, C * 32, kept_stride_t(C), KEPT_THREADS>(g_smem, (rest ? a.dST_lo : a.dST) + o_t, a.ld_t, tid);
    lds_barrier();
  }
}

// ------------------------------------------------------------------------------------
// Plain contraction with a store epilogue: C[m,n] (+)= sum_k A[m,k] B[n,k].
// Used for dW (A = dS^T chunk, B = H^T, k = compacted tokens) and for dH
// (A = dS chunk, B = W^T chunk, k = vocab chunk).  The extent marked by k_from_ctl /
// m_from_ctl follows from the active-token count, which only the device knows (StoreShape).
// ------------------------------------------------------------------------------------
// The engine's row side (4 consecutive rows per lane and MFMA tile) is given the B matrix, so that a
// lane owns 4 consecutive n of one m and C[m, n..n+3] leaves as one 16-byte (fp32) or 8-byte (bf16)
// access; N is a multiple of 4.  (Accumulating with fp32 adds performed at the L2 instead of the
// read-modify-write below was measured 6 % slower on the dH contraction.)
// A lane pair (columns 2q, 2q + 1) swaps half of two MFMA tiles first, so that an instruction writes 128 bytes of each of 8
// rows: pieces of 64 bytes go through a compute unit at half the rate (256 KiB of stores alone, with 8 or 128 compute units active:
// 16 rows x 64 B 7.6 us, whole rows 3.7 us; with all 256 either takes 12 us, the HBM's rate).
// dW of 675 rows, d = 5120: 1258 -> 1158 us.  The old values of an accumulated output are requested one column ahead of the
// stores (2869 rows, d = 4096, accumulating: call 9160 -> 9025 us; without, no gain).  (The lane masks of the row conditions
// and the two widths spill 130 scalar registers, the form that reads W as it lies 16 vector registers too, 68 bytes a lane; none of that lies in a main loop.)
__device__ __forceinline__ float of_lane_pair(float x) {      // x of lane ^ 1
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, true));
}
// G: MFMA tiles of the wavefront along n (mfma_rows).  N is a multiple of 64: either all of the first four lie within it or none.  The fifth has no
// neighbour to be swapped with and leaves in pieces of 64 bytes.
template <typename OutT, bool ACCUMULATE, int G>
__device__ __forceinline__ void store_tile(const StoreArgs& a, int tm, int tn, int m_lim, f32x4 (&acc)[G][GN]) {
  typedef __attribute__((ext_vector_type(4))) OutT out4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const bool odd = lane & 1;
  const int n_w = tn * (64 * G) + wm * WROWS, n_5 = tn * (64 * G) + mfma_rows(wm, GM) * 16;
  if (n_w >= a.N) return;                              // (the fifth lies beyond it then too)
  const bool fifth = G > GM && n_5 < a.N;
  const int m_w = tm * BM + wn * WCOLS, m0 = m_w + (lane & 14), m1 = m_w + (lane & 15);
  OutT* const C = reinterpret_cast<OutT*>(a.C) + (size_t)m0 * a.ldc + n_w + (odd ? 16 : 0) + ((lane >> 4) << 2);
  OutT* const C5 = reinterpret_cast<OutT*>(a.C) + (size_t)m1 * a.ldc + n_5 + ((lane >> 4) << 2);
  out4 old[2][G];
  auto fetch = [&](int j) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (m0 + j * 16 + h < m_lim)
#pragma unroll
        for (int i = 0; i < GM; i += 2) old[j & 1][i + h] = *reinterpret_cast<const out4*>(C + (size_t)(j * 16 + h) * a.ldc + i * 16);
    if (fifth && m1 + j * 16 < m_lim) old[j & 1][G - 1] = *reinterpret_cast<const out4*>(C5 + (size_t)(j * 16) * a.ldc);
  };
  auto put = [&](OutT* p, const f32x4& v, const out4& was) {
    out4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = (OutT)(ACCUMULATE ? v[r] + (float)was[r] : v[r]);
    *reinterpret_cast<out4*>(p) = o;
  };
  if (ACCUMULATE) fetch(0);
#pragma unroll
  for (int j = 0; j < GN; ++j) {
    if (ACCUMULATE && j + 1 < GN) fetch(j + 1);
#pragma unroll
    for (int i = 0; i < GM; i += 2) {
      f32x4 v[2];                                      // columns 2q and 2q + 1; even lanes MFMA tile i of both, odd lanes i + 1
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float lo = acc[i][j][r], hi = acc[i + 1][j][r];
        const float lo_x = of_lane_pair(lo), hi_x = of_lane_pair(hi);
        v[0][r] = odd ? hi_x : lo;
        v[1][r] = odd ? hi : lo_x;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (m0 + j * 16 + h < m_lim) put(C + (size_t)(j * 16 + h) * a.ldc + i * 16, v[h], old[j & 1][i + h]);
    }
    if (fifth && m1 + j * 16 < m_lim) put(C5 + (size_t)(j * 16) * a.ldc, acc[G - 1][j], old[j & 1][G - 1]);
  }
}

// The run-time extents of a store contraction (the active-token count is known only on the device).
struct StoreShape {
  int m_lim, tiles_m, tiles_n, K, ks, products, slab_rows, total;
  bool wide;              // tiles of 320 n
  int t0, nt;             // token tiles of this launch's block
  uint32_t b_off;         // dW: byte offset of the block's first column in a row of H^T
  __device__ __forceinline__ void init(const StoreArgs& a, const Ctl& ctl) {
    token_block(a.blk, ctl.n_pad / BM, t0, nt);
    m_lim = a.m_from_ctl ? min(a.M, max(0, min(nt * BM, ctl.n_active - t0 * BM))) : a.M;      // (rows beyond the active ones are not written, and must not be read)
    tiles_m = min(a.tiles_m, (m_lim + BM - 1) / BM);
    K = a.k_from_ctl ? min(nt * BM, dw_stages(ctl.n_active - t0 * BM) * BK) : a.K;
    b_off = a.k_from_ctl ? (uint32_t)t0 * BM * 2u : 0u;
    ks = 1; products = 1; slab_rows = ctl.n_pad;
    wide = false;
    if (a.split_k && a.m_from_ctl && nt * BM == ctl.n_pad) {
      ks = ctl.dh_ks; products = ctl.dh_products; wide = ctl.dh_wide;
    } else if (a.dw_cap > 0) {
      ks = dw_split(K / BK, a.dw_cap);
      products = a.A_lo ? 3 : 1;
      slab_rows = a.slab_rows;
    } else if (!a.A_lo && a.wide_ok) {
      wide = wide_pays(tiles_m, a.N, Parts{1, K / BK}, Parts{1, K / BK});
    }
    tiles_n = store_tiles_n(a.N, wide);
    total = tiles_m * ks * products * tiles_n;
  }
};

template <bool DIRECT, int G, class AfterLoop, class BeforeStores>
__device__ __forceinline__ void gemm_store_tile(StoreArgs a, const StoreShape& sh, int b, AfterLoop&& after_loop,
                                                BeforeStores&& before_stores) {
  const int tid = threadIdx.x;
  int tm, tn, slab;
  map_tile_interleaved(b, sh.tiles_m, sh.tiles_n, sh.ks * sh.products, slab, tm, tn);
  // (divisions only where the contraction is split, and in 32 bits: they run in front of every tile's first load)
  int part = 0, s0 = 0, s1 = sh.K / BK;
  if (sh.ks * sh.products > 1) {
    part = sh.products == 3 ? slab / 3 : slab;
    const int product = slab - part * sh.products;
    if (product == 1) { a.B = a.B_lo; a.ldb = a.ldb_lo; }
    if (product == 2) a.A = a.A_lo;
    static_assert((long long)imax(DH_PARTS_MAX, DW_SPLIT_MAX) * ((1 << 30) / BK) < 1ll << 32, "V and T are at most 2^30");
    const unsigned stages = (unsigned)s1;
    s0 = (int)((unsigned)part * stages / (unsigned)sh.ks);
    s1 = (int)((unsigned)(part + 1) * stages / (unsigned)sh.ks);
  }
  const uint32_t kb = (uint32_t)s0 * BK * 2u;          // byte offset of this part's first k

  // (a tile here is hundreds of stages long: the claim for the next one simply travels under the main loop)
  after_loop();
  typename std::conditional<DIRECT, RowsLoader<G>, SlabLoader<G>>::type LA;      // engine rows <- n
  TileLoader LB;
  auto init_n = [&](const void* B, int ldb) {
    if constexpr (DIRECT) LA.init(B, a.b_rows, s0 * BK, ldb, tn * (64 * G), tid);
    else LA.init(B, a.b_rows, tn * (64 * G), ldb, kb + sh.b_off, tid);
  };
  init_n(a.B, a.ldb);
  LB.init(a.A, a.a_rows, tm * BM, a.lda, kb, tid);     // engine columns <- m
  f32x4 acc[G][GN];
  zero_acc(acc);
  mainloop(LA, LB, s1 - s0, g_smem, acc);
  if (G == GM && a.A_lo && sh.products == 1) {   // split fp32 operands: add the two cross terms (the product of the remainders is dropped)
    __syncthreads();
    init_n(a.B_lo, a.ldb_lo);
    mainloop(LA, LB, s1 - s0, g_smem, acc);
    __syncthreads();
    init_n(a.B, a.ldb);
    LB.init(a.A_lo, a.a_rows, tm * BM, a.lda, kb, tid);
    mainloop(LA, LB, s1 - s0, g_smem, acc);
  }
  before_stores();
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the claim is visible behind this barrier
  a.C = static_cast<char*>(a.C) + (size_t)slab * sh.slab_rows * a.ldc * (a.out_bf16 ? 2 : 4);
  if (a.out_bf16) {
    if (a.accumulate) store_tile<__bf16, true, G>(a, tm, tn, sh.m_lim, acc);
    else store_tile<__bf16, false, G>(a, tm, tn, sh.m_lim, acc);
  } else {
    if (a.accumulate) store_tile<float, true, G>(a, tm, tn, sh.m_lim, acc);
    else store_tile<float, false, G>(a, tm, tn, sh.m_lim, acc);
  }
}

template <bool DIRECT>
__global__ __launch_bounds__(NTHREADS) void gemm_store_kernel(StoreArgs a) {
  const Ctl ctl = *a.ctl;
  if (a.rule.ctl && (ctl.n_pad <= DIRECT_MAX_ROWS) != DIRECT) return;
  int ld_t_all;
  if (a.rc_role && rechunk_all(a.rc, ctl.n_pad, ld_t_all)) {   // few active rows, see Rechunk
    if (a.rc_role == 1 && a.rc.dw_whole) {                     // dW: the first chunk's launch does it all
      if (a.rc.chunk > 0) return;
      a.M = a.rc.V; a.tiles_m = a.rc.tiles_v_all; a.a_rows = a.rc.tiles_v_all * BM;
      a.lda = ld_t_all;
    } else if (a.rc_role == 2 && dh_runs_whole(a.rc, ctl.n_pad)) {      // dH: likewise
      if (a.rc.chunk > 0) return;
      a.K = a.rc.tiles_v_all * BM;
      if (DIRECT) a.b_rows = a.rc.V;
      a.lda = a.rc.ld_s_all;
    } else if (a.rc_role == 1) {   // dW: this chunk's rows of the dS^T that spans the whole vocabulary
      a.A = static_cast<const char*>(a.A) + (size_t)a.v0 * ld_t_all * 2;
      if (a.A_lo) a.A_lo = static_cast<const char*>(a.A_lo) + (size_t)a.v0 * ld_t_all * 2;
      a.lda = ld_t_all;
    } else {                       // dH: this chunk's columns of the dS rows that span the whole vocabulary
      a.A = static_cast<const char*>(a.A) + (size_t)a.v0 * 2;
      if (a.A_lo) a.A_lo = static_cast<const char*>(a.A_lo) + (size_t)a.v0 * 2;
      a.lda = a.rc.ld_s_all;
    }
  }
  StoreShape sh;
  sh.init(a, ctl);
  // The grid has room for the largest split.  Workgroups beyond one per tile leave before they crowd the queue (2161 rows of
  // d = 832, 21 of them active: dW 26.3 -> 23.6 us, dH 23.7 -> 21.7).
  if ((int)blockIdx.x >= grid_for_tiles(sh.total, 1)) return;
  if (a.blk.b > 0) {
    if (sh.nt <= 0) return;
    if (a.k_from_ctl) a.accumulate = 1;                              // dW: on top of the blocks before
  }
  if (a.dw_cap > 0 && sh.ks * sh.products > 1) { a.C = a.slabs; a.accumulate = 0; a.out_bf16 = 0; }
  if (a.m_from_ctl) a.C = static_cast<float*>(a.C) + (size_t)sh.t0 * BM * a.ldc;      // dH: this block's rows of the accumulator
  TileQueue Q;
  Q.init(a.queue, sh.total, 1, 1);
  volatile int* claim = reinterpret_cast<volatile int*>(g_smem + STORE_CLAIM_OFF);
  // persistent: one workgroup per compute unit takes tiles from the XCD-aware queue until none is left
  if (sh.wide) drain_queue(Q, true, claim, [&](int b, auto&& after_loop, auto&& before_stores) { gemm_store_tile<DIRECT, GW>(a, sh, b, after_loop, before_stores); });
  else drain_queue(Q, true, claim, [&](int b, auto&& after_loop, auto&& before_stores) { gemm_store_tile<DIRECT, GM>(a, sh, b, after_loop, before_stores); });
}

// ---- host-side launchers -------------------------------------------------------------
// Workgroups of a persistent launch: one per compute unit, a multiple of the 8 XCDs.
static int g_persistent_grid = 256;

hipError_t init_gemm_kernels() {
  hipError_t e;
  if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(lmhead_fwd_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               FWD_LDS_BYTES)) != hipSuccess) return e;
  if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(lmhead_dlogits_kernel<false>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, PERSISTENT_LDS_BYTES)) != hipSuccess) return e;
  if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(lmhead_dlogits_kernel<true>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, PERSISTENT_LDS_BYTES)) != hipSuccess) return e;
  for (const void* k : {reinterpret_cast<const void*>(gemm_store_kernel<false>), reinterpret_cast<const void*>(gemm_store_kernel<true>)})
    if ((e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, STORE_LDS_BYTES)) != hipSuccess) return e;
  for (const void* k : {reinterpret_cast<const void*>(dlogits_kept_kernel<false, false, GN>), reinterpret_cast<const void*>(dlogits_kept_kernel<false, true, GN>),
                        reinterpret_cast<const void*>(dlogits_kept_kernel<true, true, GN>)})
    if ((e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kept_lds_bytes(GN))) != hipSuccess) return e;
  int dev = 0, cus = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  g_persistent_grid = cus >= 8 ? (cus / 8) * 8 : 8;
  return hipSuccess;
}

// The grid covers the host-side maximum of tiles (the live extent is known only on the device) but
// never more than one workgroup per compute unit.
static int persistent_grid(int tiles_m, int tiles_n) { return min(grid_for_tiles(tiles_m, tiles_n), g_persistent_grid); }

void launch_lmhead_fwd(const FwdArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(lmhead_fwd_kernel, dim3(persistent_grid(a.tiles_v, a.tiles_t)), dim3(NTHREADS), FWD_LDS_BYTES, s, a);
}
void launch_lmhead_dlogits(const DlogitsArgs& a, hipStream_t s) {
  if (a.kept.cap > 0) {    // at most: every half tile of the launch's widest form
    const long long halves = (a.dS_lo ? 4ll : 2ll) * (a.rc.enabled ? a.rc.tiles_v_all : a.tiles_v) * a.tiles_t;
    const bool few = a.tiles_t <= 2 || halves <= 4 * g_persistent_grid, small = halves <= KEPT_SMALL_HALVES;
    const int items = (int)std::min<long long>(small ? halves * (GN / KEPT_SMALL) : halves, 2 * g_persistent_grid);
    auto kernel = small ? (a.dS_lo ? dlogits_kept_kernel<true, true, KEPT_SMALL> : dlogits_kept_kernel<false, true, KEPT_SMALL>)
                        : a.dS_lo ? dlogits_kept_kernel<true, true, GN> : few ? dlogits_kept_kernel<false, true, GN> : dlogits_kept_kernel<false, false, GN>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)items), dim3(KEPT_THREADS), small ? kept_lds_bytes(KEPT_SMALL) : kept_lds_bytes(GN), s, a);
    if ((long long)a.kept.cap >= (long long)a.tiles_v_all * a.tiles_t) return;      // whatever is live, all of it is kept
  }
  hipLaunchKernelGGL(lmhead_dlogits_kernel<false>, dim3(persistent_grid(a.tiles_v, a.tiles_t)), dim3(NTHREADS), PERSISTENT_LDS_BYTES, s, a);
  if (a.dS_lo) {   // fp32 head: the remainders, from a second pass over the same tiles with a queue of its own
    DlogitsArgs lo = a;
    lo.queue = a.queue_lo;
    hipLaunchKernelGGL(lmhead_dlogits_kernel<true>, dim3(persistent_grid(a.tiles_v, a.tiles_t)), dim3(NTHREADS), PERSISTENT_LDS_BYTES, s, lo);
  }
}
void launch_gemm_store(const StoreArgs& a, hipStream_t s) {
  // (a split dH has at most acc_rows / 256 row tiles over all parts, a split dW dw_cap parts of every product)
  const int tiles_m = a.rc_role == 1 && a.rc.enabled && a.rc.dw_whole ? a.rc.tiles_v_all : a.tiles_m;
  const dim3 grid(persistent_grid(a.split_k ? max(a.tiles_m, a.acc_rows / BM) : tiles_m * max(1, a.dw_cap) * (a.dw_cap && a.A_lo ? 3 : 1), a.tiles_n));
  if (a.b_k_rows) hipLaunchKernelGGL(gemm_store_kernel<true>, grid, dim3(NTHREADS), STORE_LDS_BYTES, s, a);
  else hipLaunchKernelGGL(gemm_store_kernel<false>, grid, dim3(NTHREADS), STORE_LDS_BYTES, s, a);
}

}  // namespace pg
