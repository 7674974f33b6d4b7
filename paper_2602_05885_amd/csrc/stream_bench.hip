// Stand-alone measurement of the forward contraction (logits tiles -> online softmax statistics) at the
// 14B head shape in three forms, side by side on the same operands:
//   tile    one workgroup per 256 x 256 tile, dispatched by the hardware (the library's earlier form)
//   stream  the library's persistent kernel: one workgroup per compute unit, tiles from the XCD-aware
//           queue of gemm_core.h, operand loads running ahead across tile boundaries so that the
//           epilogue of a tile overlaps the arrival of the next - once with every XCD confined to an
//           equal share of the tiles, once with stealing between XCDs (what the library runs)
// and a timeline of the persistent form (100 MHz wall clock and shader clock, per workgroup and tile):
// main-loop time, epilogue time, gap between tiles, and per XCD the sustained shader clock and the
// progress after TL_FIRST tiles.  Both forms must produce identical partial sums (checked).
// Usage: stream_bench [tokens [iters]]      (defaults: 32768 tokens, 3 timed launches per form)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "kernels_gemm.hip"
using namespace pg;

#define CK(x)                                                                 \
  do {                                                                        \
    hipError_t e_ = (x);                                                      \
    if (e_ != hipSuccess) {                                                   \
      printf("HIP error %s at line %d\n", hipGetErrorString(e_), __LINE__);   \
      exit(1);                                                                \
    }                                                                         \
  } while (0)

constexpr int TL_FIRST = PROBE_FIRST, TL_TILES = PROBE_TILES;   // tiles of every workgroup the timeline records

namespace pg {

// The forward as one workgroup per tile, placed by the hardware dispatcher (workgroup b on XCD b mod 8): the same statistics and
// the same tile order as the persistent form, cold prologue and drain for every tile.
__global__ __launch_bounds__(NTHREADS) void fwd_one_tile_kernel(FwdArgs a) {
  const Ctl ctl = *a.ctl;
  int tm, tn;
  // the live token tiles are known only on the device; the grid covers the host-side maximum
  if (!map_tile(blockIdx.x, a.tiles_v, min(a.tiles_t, ctl.n_pad / BN), tm, tn, true)) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;

  TileLoader LA, LB;
  LA.init(a.W, a.w_rows, tm * BM, a.ldw, 0u, tid);
  LB.init(a.Hc, a.h_rows, tn * BN, a.ldh, 0u, tid);
  f32x4 acc[GM][GN];
  zero_acc(acc);
  mainloop(LA, LB, a.K / BK, g_smem, acc);

  const int v_base = tm * BM + wm * WROWS;            // first vocab row of this wavefront's block
  const bool ragged = (tm * BM + BM > a.V);
  float* red = reinterpret_cast<float*>(g_smem);      // [m, s, u][WM][256 tokens]

  // the library's statistics (lmhead_fwd_body): maxima first, then plain sums, two token columns at a time
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
    float su[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = j0 + h, tok = tn * BN + wn * WCOLS + j * 16 + (lane & 15);
      float s = 0.f, u = 0.f;
#pragma unroll
      for (int i = 0; i < GM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float dlt = fmaf(acc[i][j][r], a.scale, -mx[j]);
          const float e = __builtin_amdgcn_exp2f(dlt);
          s += e;
          u = fmaf(e, dlt, u);
        }
      const Two x = swap_halves(s, u);
      su[h] = x.a + x.b;
      // sampled token's logit: at most one lane of the whole grid owns (tok, y[tok])
      const int ytok = a.yc[tok];
      const int yrel = ytok - v_base;
      const bool mine = (yrel >= 0) && (yrel < WROWS) && (ytok < a.V) && (((yrel >> 2) & 3) == (lane >> 4));
      if (__any(mine)) {
        float zy = 0.f;
#pragma unroll
        for (int i = 0; i < GM; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (yrel == i * 16 + acc_row(r, lane)) zy = acc[i][j][r] * a.scale;
        if (mine) a.zy[tok] = zy;
      }
    }
    const Two y = swap_rows(su[0], su[1]);
    const int tok_l = wn * WCOLS + (j0 + ((lane >> 4) & 1)) * 16 + (lane & 15);
    red[(1 + (lane >> 5)) * (WM * BN) + wm * BN + tok_l] = y.a + y.b;
    if (lane < 32) red[wm * BN + tok_l] = lane < 16 ? mx[j0] : mx[j0 + 1];
  }
  __syncthreads();
  if (tid < BN) {
    const float* p = red + tid;
    float m = p[0], s = p[WM * BN], u = p[2 * WM * BN];
#pragma unroll
    for (int w = 1; w < WM; ++w) merge_state(m, s, u, p[w * BN], p[(WM + w) * BN], p[(2 * WM + w) * BN]);
    const size_t o = (size_t)tm * a.t_cap + (size_t)tn * BN + tid;
    a.part_m[o] = m; a.part_s[o] = s; a.part_u[o] = u;
  }
}

// The library's persistent forward with the probe compiled in.
__global__ __launch_bounds__(NTHREADS) void fwd_persistent_probe_kernel(FwdArgs a, int steal, unsigned long long* tl) {
  lmhead_fwd_body<true>(a, steal != 0, tl);
}

}  // namespace pg

__global__ void fill_kernel(__bf16* p, size_t n, unsigned seed, float scale) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    unsigned x = (unsigned)(i * 2654435761u) ^ seed;
    x ^= x >> 16; x *= 0x85ebca6bu; x ^= x >> 13; x *= 0xc2b2ae35u; x ^= x >> 16;
    p[i] = (__bf16)(((float)(x & 0xffff) / 65536.f - 0.5f) * scale);
  }
}

int main(int argc, char** argv) {
  const int T = argc > 1 ? atoi(argv[1]) : 32768;
  const int iters = argc > 2 ? atoi(argv[2]) : 3;
  const int d = 5120, V = 151936;
  if (T < 256 || T % 256) { printf("tokens must be a positive multiple of 256\n"); return 1; }
  CK(init_gemm_kernels());
  CK(hipFuncSetAttribute(reinterpret_cast<const void*>(fwd_persistent_probe_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                         FWD_LDS_BYTES));
  CK(hipFuncSetAttribute(reinterpret_cast<const void*>(fwd_one_tile_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                         GEMM_LDS_BYTES));
  int cus = 0;
  CK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, 0));
  const int pgrid = std::max(8, cus / 8 * 8);
  __bf16 *W, *H;
  int* yc;
  float *zy, *pm, *ps, *pu;
  Ctl* ctl;
  unsigned* queue;
  unsigned long long* tl;
  const int tiles_v = (V + 255) / 256, tiles_t = T / 256;
  CK(hipMalloc(&W, (size_t)V * d * 2)); CK(hipMalloc(&H, (size_t)T * d * 2));
  CK(hipMalloc(&yc, T * 4)); CK(hipMalloc(&zy, T * 4));
  CK(hipMalloc(&pm, (size_t)tiles_v * T * 4)); CK(hipMalloc(&ps, (size_t)tiles_v * T * 4)); CK(hipMalloc(&pu, (size_t)tiles_v * T * 4));
  CK(hipMalloc(&ctl, sizeof(Ctl))); CK(hipMalloc(&queue, 64));
  CK(hipMalloc(&tl, (size_t)pgrid * TL_TILES * 4 * 8));
  Ctl h{T, T, 1.f, {}, 1};
  CK(hipMemcpy(ctl, &h, sizeof h, hipMemcpyHostToDevice));
  CK(hipMemset(yc, 0, T * 4));
  fill_kernel<<<1024, 256>>>(W, (size_t)V * d, 1u, 0.07f);      // W ~ U(-0.035, 0.035): standard deviation 0.02
  fill_kernel<<<1024, 256>>>(H, (size_t)T * d, 2u, 3.4f);       // H ~ U(-1.7, 1.7): unit RMS
  FwdArgs a{};
  a.W = W; a.Hc = H; a.w_rows = V; a.h_rows = T; a.ldw = d; a.ldh = d; a.K = d; a.V = V;
  a.tiles_v = tiles_v; a.tiles_t = tiles_t; a.t_cap = T; a.scale = 1.4427f; a.yc = yc; a.zy = zy;
  a.part_m = pm; a.part_s = ps; a.part_u = pu; a.ctl = ctl; a.queue = queue;
  const int grid = grid_for_tiles(tiles_v, tiles_t);
  const char* names[3] = {"tile                    ", "stream, equal XCD shares", "stream, stealing        "};
  std::vector<float> ref(4096), got(4096);
  auto run = [&](int form, unsigned long long* timeline) {
    if (form == 0) {
      hipLaunchKernelGGL(fwd_one_tile_kernel, dim3(grid), dim3(NTHREADS), GEMM_LDS_BYTES, 0, a);
    } else {
      CK(hipMemsetAsync(queue, 0, 64, 0)); CK(hipMemsetAsync(ctl->step, 0, sizeof ctl->step, 0));
      hipLaunchKernelGGL(fwd_persistent_probe_kernel, dim3(std::min(grid, pgrid)), dim3(NTHREADS), FWD_LDS_BYTES, 0, a,
                         form == 2 ? 1 : 0, timeline);
    }
  };
  for (int round = 0; round < 2; ++round)
    for (int form = 0; form < 3; ++form) {
      CK(hipMemset(ps, 0, (size_t)tiles_v * T * 4));
      run(form, nullptr); run(form, nullptr);
      CK(hipDeviceSynchronize());
      hipEvent_t e0, e1;
      CK(hipEventCreate(&e0)); CK(hipEventCreate(&e1));
      CK(hipEventRecord(e0));
      for (int i = 0; i < iters; ++i) run(form, nullptr);
      CK(hipEventRecord(e1)); CK(hipEventSynchronize(e1));
      float ms;
      CK(hipEventElapsedTime(&ms, e0, e1));
      ms /= iters;
      CK(hipMemcpy((form ? got : ref).data(), ps + (size_t)(tiles_v - 1) * T + T - 4096, 4096 * 4, hipMemcpyDeviceToHost));
      size_t bad = 0;
      if (form) for (size_t i = 0; i < got.size(); ++i) if (got[i] != ref[i]) ++bad;
      printf("[%s] tokens=%d  %.3f ms per launch  %.1f TFLOP/s (%.1f%% of 2500)  differences from the tile kernel: %zu\n",
             names[form], T, ms, 2.0 * V * (double)T * d / ms / 1e9, 2.0 * V * (double)T * d / ms / 1e9 / 25.0, bad);
      fflush(stdout);
      if (bad) return 1;
    }
  if ((long long)tiles_v * tiles_t / pgrid < TL_FIRST + TL_TILES) return 0;   // too few tiles per workgroup for the timeline
  for (int form = 1; form < 3; ++form) {
    CK(hipMemset(tl, 0, (size_t)pgrid * TL_TILES * 4 * 8));
    run(form, tl);
    CK(hipDeviceSynchronize());
    std::vector<unsigned long long> t((size_t)pgrid * TL_TILES * 4);
    CK(hipMemcpy(t.data(), tl, t.size() * 8, hipMemcpyDeviceToHost));
    unsigned long long t0 = ~0ull;
    for (int wg = 0; wg < pgrid; ++wg) t0 = std::min(t0, t[(size_t)wg * TL_TILES * 4]);
    double ml = 0, ep = 0, gap = 0;
    for (int wg = 0; wg < pgrid; ++wg)
      for (int k = 0; k < TL_TILES; ++k) {
        const unsigned long long* p = &t[((size_t)wg * TL_TILES + k) * 4];
        ml += p[1] - p[0]; ep += p[2] - p[1];
        if (k) gap += p[0] - p[-2];
      }
    printf("[%s] tiles %d..%d of every workgroup: main loop %.2f us, epilogue %.2f us, gap to the next tile %.2f us\n",
           names[form], TL_FIRST, TL_FIRST + TL_TILES - 1, ml / (pgrid * TL_TILES) * 0.01, ep / (pgrid * TL_TILES) * 0.01,
           gap / (pgrid * (TL_TILES - 1)) * 0.01);
    for (int x = 0; x < 8; ++x) {       // workgroup b runs on XCD b % 8
      double mlx = 0, ghz = 0, lag = 0;
      int n = 0;
      for (int wg = x; wg < pgrid; wg += 8, ++n) {
        const unsigned long long* p0 = &t[((size_t)wg * TL_TILES + 0) * 4];
        const unsigned long long* pl = &t[((size_t)wg * TL_TILES + TL_TILES - 1) * 4];
        ghz += (double)(pl[3] - p0[3]) / (double)(pl[2] - p0[2]) * 0.1;
        lag += (p0[0] - t0) * 0.01;
        for (int k = 0; k < TL_TILES; ++k) mlx += t[((size_t)wg * TL_TILES + k) * 4 + 1] - t[((size_t)wg * TL_TILES + k) * 4];
      }
      printf("    XCD %d: shader clock %.3f GHz, main loop %.2f us per tile, starts its tile %d %.0f us after the first workgroup\n",
             x, ghz / n, mlx / (n * TL_TILES) * 0.01, TL_FIRST, lag / n);
    }
    fflush(stdout);
  }
  return 0;
}
