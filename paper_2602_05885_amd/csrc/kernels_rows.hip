// Vector / row kernels around the MFMA kernels: TRLOO advantages, mismatch pre-pass, row
// compaction, operand staging, the per-row softmax combine with the surrogate epilogue,
// and the final scatter of dH.  None of them is bandwidth- or flop-significant next to the
// contractions; they are written for determinism (fixed reduction orders, integer atomics
// only) and to keep the host out of the loop (no synchronisation, counts stay on device).
#include "kernels.h"
#include "gemm_core.h"

namespace pg {

// ------------------------------------------------------------------ fills
__global__ void fill_f32_kernel(float* p, size_t n, float v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}
void launch_fill_f32(float* p, size_t n, float v, hipStream_t s) {
  if (!p || n == 0) return;
  const int grid = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  hipLaunchKernelGGL(fill_f32_kernel, dim3(grid), dim3(256), 0, s, p, n, v);
}
void launch_fill_zero_bytes(void* p, size_t nbytes, hipStream_t s) {
  launch_fill_f32(reinterpret_cast<float*>(p), nbytes / 4, 0.f, s);
}

// ------------------------------------------------------------------ TRLOO (Sec. 4.2, Eq. 2, 3 and 5)
// A segmented group reduction: one wavefront per (prompt, turn) group, its 64 lanes striding over the
// K rollouts (the group's members lie Tmax elements apart in the [P, K, Tmax] tensors).  Every lane
// evaluates the returns of its rollouts once, by Horner's rule from the last turn backwards, and keeps
// them in registers (up to TRLOO_HELD per lane, i.e. K <= 64 TRLOO_HELD; beyond that they are evaluated
// again in the second sweep); the group's sum and count are then reduced across the wavefront by a
// butterfly of shuffles, whose order is fixed, so results repeat bit for bit.  fp64 throughout.  The
// leave-one-out mean is (sum - own) / (N - 1), the group mean of the comparison baseline sum / N.
constexpr int TRLOO_HELD = 4;

__device__ __forceinline__ double turn_return(const float* r, int t, int Tmax, double gamma) {
  double g = 0.0;
  for (int tp = Tmax - 1; tp >= t; --tp) g = (double)r[tp] + gamma * g;
  return g;
}

__global__ __launch_bounds__(256) void trloo_kernel(TrlooArgs a) {
  const int lane = threadIdx.x & 63;
  const int g = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);      // wavefront-uniform
  if (g >= a.P * a.Tmax) return;
  const int p = g / a.Tmax, t = g % a.Tmax;
  const double gamma = (double)a.gamma;
  double held[TRLOO_HELD];
  double sum = 0.0;
  int n = 0;
  for (int k = lane, i = 0; k < a.K; k += 64, ++i) {
    const size_t base = ((size_t)p * a.K + k) * a.Tmax;
    const double G = turn_return(a.rewards + base, t, a.Tmax, gamma);
    if (i < TRLOO_HELD) held[i] = G;
    if (a.returns_out) a.returns_out[base + t] = G;
    if (a.valid[base + t]) { sum += G; ++n; }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sum += __shfl_xor(sum, off);
    n += __shfl_xor(n, off);
  }
  if (lane == 0 && a.group_n_out) a.group_n_out[g] = n;
  for (int k = lane, i = 0; k < a.K; k += 64, ++i) {
    const size_t base = ((size_t)p * a.K + k) * a.Tmax;
    double A = 0.0;
    if (a.valid[base + t]) {
      const double G = i < TRLOO_HELD ? held[i] : turn_return(a.rewards + base, t, a.Tmax, gamma);
      if (a.group_mean) A = G - sum / (double)n;                    // Eq. (3); n >= 1 here
      else if (n >= 2) A = G - (sum - G) / (double)(n - 1);         // Eq. (5)
    }
    a.adv_out[base + t] = A;
  }
}
void launch_trloo(const TrlooArgs& a, hipStream_t s) {
  const int n = a.P * a.Tmax;                                       // groups, 4 per workgroup
  hipLaunchKernelGGL(trloo_kernel, dim3((n + 3) / 4), dim3(256), 0, s, a);
}

// ------------------------------------------------------------------ pre-pass
__device__ __forceinline__ void split_bf16(float x, __bf16& hi, __bf16& lo) {
  hi = (__bf16)x;
  lo = (__bf16)(x - (float)hi);
}
// fp32 head weight -> [V, 3d] bf16 = [hi | lo | hi]: the workgroups behind the first `blocks` of the pre-pass's first launch (it
// depends on nothing; as a launch of its own, 64 x 1000 head, 1024 rows, 81.8 instead of 80.5 us a call).
__device__ __forceinline__ void split_w(const PrepArgs& a, int blocks) {
  const size_t stride = (size_t)(gridDim.x - blocks) * blockDim.x;
  for (size_t i = (size_t)(blockIdx.x - blocks) * blockDim.x + threadIdx.x; i < a.w_elems; i += stride) {
    const size_t v = i / a.d, k = i % a.d;
    __bf16 hi, lo;
    split_bf16(a.W[i], hi, lo);
    __bf16* o = a.Wc + v * 3 * (size_t)a.d + k;
    o[0] = hi; o[a.d] = lo; o[2 * (size_t)a.d] = hi;
  }
}

__device__ __forceinline__ void prep_init(const PrepArgs& a, int block, int blocks) {
  const int i = block * blockDim.x + threadIdx.x;
  for (int w = i; w < a.queue_words; w += blocks * blockDim.x) a.queue[w] = 0u;
  if (i < a.t_cap) a.zy[i] = 0.f;
  if (i < a.T) {
    if (a.out0) a.out0[i] = 0.f;
    if (a.out1) a.out1[i] = 0.f;
    if (a.out2) a.out2[i] = 0.f;
    if (!a.cu) {
      a.flag[i] = a.mask ? (a.mask[i] != 0) : 1;
      a.c_tok[i] = 1.f;
      a.a_tok[i] = 0.f;
    }
  }
  if (!a.cu) return;
  // Rows of no segment.  The offsets lead from the first to the last, so every row between these two is in one; of the others, none is unless
  // some offset goes back, which the wavefront looks for first.
  const bool outside = i < a.T && (a.S <= 0 || i < a.cu[0] || i >= a.cu[a.S]);
  if (!__any(outside)) return;
  bool back = false;
#pragma unroll 4
  for (int s = threadIdx.x & 63; s < a.S; s += 64) back |= a.cu[s + 1] < a.cu[s];
  bool in = false;
  if (__any(back) && outside)
    for (int s = 0; s < a.S; ++s) in |= i >= a.cu[s] && i < a.cu[s + 1];
  if (outside && !in) a.flag[i] = 0;
}

// One workgroup per segment (= one training sample): Sec. 5.1's geometric-mean ratio and
// token veto over the sample's loss tokens, decided in fp64, then per-row weights.  A sample
// whose keep flag is 0 (Sec. 5.2's rejection sampling), or whose index lies outside the
// advantage table, is skipped before any of that.  What there is to count goes into the rows' flags, from which the compaction sums
// it, so that nothing has to be cleared first and the segments are workgroups of the first launch.
constexpr unsigned FLAG_ACTIVE = 1, FLAG_PASSED = 2, FLAG_TRUNCATED = 4;               // of the row (passed: carries loss, but its segment is out)
constexpr unsigned FLAG_VETO = 8, FLAG_OUTSIDE = 16, FLAG_DROPPED = 32;                // of its segment, on the first row
__device__ __forceinline__ void prep_segment(const PrepArgs& a, int s) {
  __shared__ double sh_sum[256];
  __shared__ double sh_min[256];
  __shared__ int sh_n[256];
  __shared__ unsigned sh_seg;
  const int tid = threadIdx.x;
  int lo = a.cu[s], hi = a.cu[s + 1];
  lo = max(lo, 0);
  hi = min(hi, a.T);
  const bool mm = a.mismatch_mode != 0;
  // table entry of this segment; an index outside the tables drops the segment and reads nothing
  const int idx = a.seg_sample ? a.seg_sample[s] : s;
  const bool in_table = a.n_samples <= 0 || (idx >= 0 && idx < a.n_samples);
  double sum = 0.0, mn = 1.0e300;
  int n = 0;
  for (int t = lo + tid; t < hi; t += 256) {
    if (a.mask[t]) {
      ++n;
      if (mm) {
        const double dl = (double)a.old_logp[t] - (double)a.rollout_logp[t];
        sum += dl;
        mn = fmin(mn, dl);
      }
    }
  }
  sh_sum[tid] = sum; sh_min[tid] = mn; sh_n[tid] = n;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) {
      sh_sum[tid] += sh_sum[tid + w];
      sh_min[tid] = fmin(sh_min[tid], sh_min[tid + w]);
      sh_n[tid] += sh_n[tid + w];
    }
    __syncthreads();
  }
  if (tid == 0) {
    unsigned seg = 0;
    const int nn = sh_n[0];
    const bool dropped = !in_table || (a.sample_keep && !a.sample_keep[idx]);
    if (dropped) {            // filtered out before training (PRS): as if the sample had no loss rows
      if (nn > 0) seg = FLAG_DROPPED;
    } else if (nn > 0) {
      if (mm) {
        const bool vetoed = (a.veto_ratio > 0.f) && (exp(sh_min[0]) < (double)a.veto_ratio);
        if (vetoed) seg |= FLAG_VETO;
        if (a.mismatch_mode == 1) {
          const double w = exp(sh_sum[0] / (double)nn);
          const bool inside = ((double)a.geo_lo <= w) && (w <= (double)a.geo_hi);
          if (!inside) seg |= FLAG_OUTSIDE;
        }
      }
    }
    sh_seg = seg;
  }
  __syncthreads();
  const unsigned seg = sh_seg;           // (a segment without a loss row has none of these, and no row to keep)
  const float A = in_table ? (float)a.adv[idx] : 0.f;
  for (int t = lo + tid; t < hi; t += 256) {
    const bool on = a.mask[t] != 0;
    unsigned flag = (t == lo ? seg : 0u) | (on ? !seg ? FLAG_ACTIVE : seg & FLAG_DROPPED ? 0u : FLAG_PASSED : 0u);
    float c = 0.f;
    if (on && !seg) {
      c = 1.f;
      if (a.mismatch_mode == 2) {
        const double ratio = exp((double)a.old_logp[t] - (double)a.rollout_logp[t]);
        if (ratio > (double)a.trunc_c) { flag |= FLAG_TRUNCATED; c = a.trunc_c; } else { c = (float)ratio; }
      }
    }
    a.flag[t] = (uint8_t)flag;
    a.c_tok[t] = c;
    a.a_tok[t] = A;
  }
}

// The segments, what has to be cleared, and an fp32 head's split of W, in one launch.  Clearing, segments and compaction as three launches / two:
// 512 rows, 64 x 1000 fp32 head 10.7 / 8.1 us, 16 082 rows 23.1 / 19.5, 43 697 rows 39.7 / 37.0.
__global__ __launch_bounds__(256) void prep_first_kernel(PrepArgs a, int segments, int blocks) {
  if ((int)blockIdx.x < segments) return prep_segment(a, (int)blockIdx.x);
  if ((int)blockIdx.x < segments + blocks) return prep_init(a, (int)blockIdx.x - segments, blocks);
  split_w(a, segments + blocks);
}

// Single workgroup: exclusive scan of the active flags -> compacted row list, inverse map, counts and the loss
// normaliser.  A wavefront takes a contiguous run of rows, 256 at a time (four flags per lane in one load), counts
// them, and after the wavefronts' totals are known ranks them with a lane prefix.  Latency is all there is: one row at a time per
// thread, as it was, took 64 us at 43697 rows and 19 us at 16082; so 24 and 9 us.
// SEGMENTS: the other kinds of flags are counted too (calls without segments have none: 18 000 of 20 000 rows 11.3 -> 10.6 us, 11 rows 2.96 -> 2.56).
template <bool SEGMENTS>
__global__ __launch_bounds__(1024) void prep_compact_kernel(PrepArgs a) {
  constexpr int KINDS = SEGMENTS ? 6 : 1;                       // of flags, see FLAG_ACTIVE
  __shared__ int total_of[KINDS][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int run = (a.T + 16 * 256 - 1) / (16 * 256) * 256;      // rows per wavefront (wave 15's may reach beyond T)
  const int lo = wave * run, hi = lo < a.T ? (a.T - lo < run ? a.T : lo + run) : lo;
  // four flags from row t on (the flag array is padded to whole groups; rows beyond T count as inactive)
  auto flags = [&](int t) -> unsigned {
    unsigned f = 0;
    if (t < hi) f = *reinterpret_cast<const unsigned*>(a.flag + t);
    if (t + 4 > hi && t < hi) f &= (1u << ((hi - t) * 8)) - 1u;
    return f;
  };
  int cnt[KINDS] = {};
#pragma unroll 4
  for (int t = lo + lane * 4; t < hi; t += 256) {
    const unsigned f = flags(t);
#pragma unroll
    for (int q = 0; q < KINDS; ++q) cnt[q] += __popc(f & (0x01010101u << q));
  }
#pragma unroll
  for (int q = 0; q < KINDS; ++q) {
    if (q == 0 || __any(cnt[q])) {                     // (all but the first are rare: all six reduced, 4.9 us at 512 rows, so 3.7)
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) cnt[q] += __shfl_xor(cnt[q], off);
    }
    if (lane == 0) total_of[q][wave] = cnt[q];
  }
  __syncthreads();
  int base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int c = total_of[0][w];
    if (w < wave) base += c;
    total += c;
  }
  unsigned ahead = flags(lo + lane * 4);
  for (int t0 = lo; t0 < hi; t0 += 256) {
    const int t = t0 + lane * 4;
    const unsigned f = ahead & 0x01010101u;
    ahead = flags(t + 256);
    const int c = __popc(f);
    int incl = c;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(incl, off);
      if (lane >= off) incl += v;
    }
    int idx = base + incl - c;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (t + e < hi) {
        const bool on = (f >> (8 * e)) & 1u;
        a.pos[t + e] = on ? idx : -1;
        if (on) a.rows[idx++] = t + e;
      }
    base += __shfl(incl, 63);
  }
  if (tid < 8) a.ctl->step[tid] = 0u;
  if (tid == 0) {
    a.ctl->n_active = total;
    a.ctl->n_pad = (total + 255) / 256 * 256;
    a.ctl->norm = a.norm_override > 0.f ? a.norm_override : (float)max(total, 1);
    a.ctl->dh_slabs = a.ctl->dh_ks = a.ctl->dh_products = 1;        // (what a call without rows is left with)
    a.ctl->dh_wide = 0;
  }
  if (tid < 8) {      // counter: the flags that it counts (1 and 2 are the combine's; 6: active rows and those passed over)
    const int kind = tid == 3 ? 4 : tid == 4 ? 3 : tid == 5 ? 2 : tid == 6 ? 1 : tid == 7 ? 5 : -1;
    unsigned long long sum = tid == 0 || tid == 6 ? (unsigned long long)total : 0ull;
    if (SEGMENTS && kind >= 0)
#pragma unroll
      for (int w = 0; w < 16; ++w) sum += (unsigned long long)total_of[kind][w];
    a.counters[tid] = sum;
  }
}

// A token id counted from the first vocab row of W, -1 where W does not hold it.
__device__ __forceinline__ int local_id(int y, int y_offset, int V) {
  const int l = y - y_offset;
  return l < 0 || l >= V ? -1 : l;
}

// Every row active (no mask, no segments): the compaction is the identity, and the whole pre-pass one launch.
// (yc: the token ids as the gather would leave them, for a call that reads H where it lies and gathers nothing: d = 2880, 134 rows
// forward only 158.3 -> 156.8 us.)
__global__ void prep_all_rows_kernel(PrepArgs a, int blocks) {
  if ((int)blockIdx.x >= blocks) return split_w(a, blocks);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 8) a.counters[i] = i == 0 || i == 6 ? (unsigned long long)a.T : 0ull;      // active = loss rows = T
  for (int w = i; w < a.queue_words; w += blocks * blockDim.x) a.queue[w] = 0u;
  if (i < a.t_cap) {
    a.zy[i] = 0.f;
    if (a.yc) a.yc[i] = i < a.T ? local_id(a.y[i], a.y_offset, a.V) : -1;
  }
  if (i < a.T) { a.rows[i] = i; a.pos[i] = i; }
  if (i < 8) a.ctl->step[i] = 0u;
  if (i == 0) {
    a.ctl->n_active = a.T;
    a.ctl->n_pad = a.t_cap;
    a.ctl->norm = a.norm_override > 0.f ? a.norm_override : (float)a.T;
    a.ctl->dh_slabs = a.ctl->dh_ks = a.ctl->dh_products = 1;        // (what a call without rows is left with)
    a.ctl->dh_wide = 0;
  }
}

void launch_prepass(const PrepArgs& a, hipStream_t s) {
  const int n = a.t_cap > 8 ? a.t_cap : 8, blocks = (n + 255) / 256;
  const size_t split = (a.w_elems + 255) / 256;
  const unsigned split_blocks = (unsigned)(split < 65536 ? split : 65536);
  if (!a.cu && !a.mask) {
    hipLaunchKernelGGL(prep_all_rows_kernel, dim3(blocks + split_blocks), dim3(256), 0, s, a, blocks);
    return;
  }
  const int segments = a.cu && a.S > 0 ? a.S : 0;
  hipLaunchKernelGGL(prep_first_kernel, dim3((unsigned)segments + blocks + split_blocks), dim3(256), 0, s, a, segments, blocks);
  if (a.cu) hipLaunchKernelGGL(prep_compact_kernel<true>, dim3(1), dim3(1024), 0, s, a);
  else hipLaunchKernelGGL(prep_compact_kernel<false>, dim3(1), dim3(1024), 0, s, a);
}

// ------------------------------------------------------------------ operand staging
// ---- 64 x 64 bf16 tile transposition through LDS with 16-byte global accesses ----
// Rows are staged with a stride of 68 elements (34 words): 8-byte aligned for the row writes and
// odd enough in words that the column reads of the transposed phase spread over the banks.
constexpr int TT_LD = 68;

// thread t: 16-byte chunk t&7 of rows (t>>3) and (t>>3)+32
__device__ __forceinline__ void tt_put(uint16_t* tile, int row, int chunk, const i32x4& v) {
  uint2* p = reinterpret_cast<uint2*>(tile + row * TT_LD + chunk * 8);
  p[0] = make_uint2((uint32_t)v[0], (uint32_t)v[1]);
  p[1] = make_uint2((uint32_t)v[2], (uint32_t)v[3]);
}
// column `col`, rows chunk*8 .. chunk*8+7, packed as one 16-byte row piece of the transpose
__device__ __forceinline__ i32x4 tt_get(const uint16_t* tile, int col, int chunk) {
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t lo = tile[(chunk * 8 + 2 * e) * TT_LD + col];
    const uint32_t hi = tile[(chunk * 8 + 2 * e + 1) * TT_LD + col];
    w[e] = lo | (hi << 16);
  }
  i32x4 v;
  v[0] = (int)w[0]; v[1] = (int)w[1]; v[2] = (int)w[2]; v[3] = (int)w[3];
  return v;
}

// 64 compacted rows x 64 columns per workgroup: copies (or splits) H rows into the compacted,
// zero-padded operand and writes its transpose for the dW contraction.
__global__ __launch_bounds__(256) void gather_kernel(GatherArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[64 * TT_LD];
  const Ctl ctl = *a.ctl;
  const int i0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
  if (i0 >= ctl.n_pad) return;
  const int tid = threadIdx.x;
  if (blockIdx.y == 0 && tid < 64) {
    const int i = i0 + tid;
    a.yc[i] = i < ctl.n_active ? local_id(a.y[a.rows[i]], a.y_offset, a.V) : -1;
  }
  if (!a.is_f32) {
    const int chunk = tid & 7;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int r = (tid >> 3) + 32 * p;
      const int i = i0 + r;
      i32x4 v = {0, 0, 0, 0};
      if (i < ctl.n_active)
        v = *reinterpret_cast<const i32x4*>(reinterpret_cast<const __bf16*>(a.H) + (size_t)a.rows[i] * a.d + j0 + chunk * 8);
      *reinterpret_cast<i32x4*>(a.Hc + (size_t)i * a.d + j0 + chunk * 8) = v;
      tt_put(tile, r, chunk, v);
    }
    if (!a.HcT) return;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int jj = (tid >> 3) + 32 * p;
      *reinterpret_cast<i32x4*>(a.HcT + (size_t)(j0 + jj) * a.ld_t + i0 + chunk * 8) = tt_get(tile, jj, chunk);
    }
    return;
  }
  // fp32 inputs: split into bf16 hi + lo parts, [hi | hi | lo] along k, and the transposes of both (16-byte accesses
  // throughout; element by element, and the remainders' transpose as a launch of its own, it took 9 + 2.5 us at 1024 x 64, so 4.4 us)
  __shared__ __attribute__((aligned(16))) uint16_t tile_lo[64 * TT_LD];
  const int ldh = 3 * a.d, chunk = tid & 7;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int r = (tid >> 3) + 32 * p, i = i0 + r;
    bf16x8 hi, lo;
    if (i < ctl.n_active) {
      const float4* src = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(a.H) + (size_t)a.rows[i] * a.d + j0 + chunk * 8);
      const float4 x = src[0], y = src[1];
      const float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) { __bf16 h, l; split_bf16(v[e], h, l); hi[e] = h; lo[e] = l; }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) { hi[e] = (__bf16)0.f; lo[e] = (__bf16)0.f; }
    }
    __bf16* o = a.Hc + (size_t)i * ldh + j0 + chunk * 8;
    *reinterpret_cast<bf16x8*>(o) = hi;
    *reinterpret_cast<bf16x8*>(o + a.d) = hi;
    *reinterpret_cast<bf16x8*>(o + 2 * a.d) = lo;
    tt_put(tile, r, chunk, __builtin_bit_cast(i32x4, hi));
    tt_put(tile_lo, r, chunk, __builtin_bit_cast(i32x4, lo));
  }
  if (!a.HcT) return;
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int jj = (tid >> 3) + 32 * p;
    const size_t o = (size_t)(j0 + jj) * a.ld_t + i0 + chunk * 8;
    *reinterpret_cast<i32x4*>(a.HcT + o) = tt_get(tile, jj, chunk);
    *reinterpret_cast<i32x4*>(a.HcT_lo + o) = tt_get(tile_lo, jj, chunk);
  }
}
void launch_gather(const GatherArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(gather_kernel, dim3(a.t_cap / 64, a.d / 64), dim3(256), 0, s, a);
}

// W rows [v0, v0+cols) (row stride ldw elements) -> WT[j][v - v0] (bf16; fp32 weights are rounded), zeros for v >= V.
__global__ __launch_bounds__(256) void transpose_w_kernel(const void* W, int is_f32, long long V, int ldw, int v0,
                                                          int ldt, __bf16* WT, DirectRule rule) {
  if (rule.ctl && rule.ctl->n_pad <= DIRECT_MAX_ROWS) return;
  __shared__ __attribute__((aligned(16))) uint16_t tile[64 * TT_LD];
  const int vt = blockIdx.x * 64, j0 = blockIdx.y * 64;
  const int tid = threadIdx.x;
  const int chunk = tid & 7;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int r = (tid >> 3) + 32 * p;
    const long long v = (long long)v0 + vt + r;
    i32x4 x = {0, 0, 0, 0};
    if (v < V) {
      const size_t o = (size_t)v * ldw + j0 + chunk * 8;
      if (is_f32) {
        const float* src = reinterpret_cast<const float*>(W) + o;
        bf16x8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = (__bf16)src[e];
        x = __builtin_bit_cast(i32x4, h);
      } else {
        x = *reinterpret_cast<const i32x4*>(reinterpret_cast<const __bf16*>(W) + o);
      }
    }
    tt_put(tile, r, chunk, x);
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int jj = (tid >> 3) + 32 * p;
    *reinterpret_cast<i32x4*>(WT + (size_t)(j0 + jj) * ldt + vt + chunk * 8) = tt_get(tile, jj, chunk);
  }
}
void launch_transpose_w(const void* W, int is_f32, int64_t V, int d, int ldw, int v0, int cols, int ldt, __bf16* WT,
                        const DirectRule& rule, hipStream_t s) {
  hipLaunchKernelGGL(transpose_w_kernel, dim3(cols / 64, d / 64), dim3(256), 0, s, W, is_f32, (long long)V, ldw, v0,
                     ldt, WT, rule);
}

// ------------------------------------------------------------------ combine + surrogate
// Merges the per-vocab-tile softmax partials of every compacted row with the online merge rule
// (m, s, u) + (m2, s2, u2), emits log-prob / entropy / logsumexp, and for the loss call evaluates
// the clipped surrogate and the coefficient that scales (onehot - softmax) in the backward.
// A workgroup of COMBINE_WAVES wavefronts takes R rows and deals their vocab tiles to its 1024 / R parts, each of which merges every 1024 / R-th tile's state
// (online, fixed order) with the loads of four tiles in flight; the parts' results are then merged in a fixed order, and R lanes finish
// the rows.  With few rows the serial chain of loads and merges is all there is, with many it is HBM-bound, and rows of 64 bytes cost more than they save.
// 594 tiles, R = 64 (the 16 results one after the other) / 16 (by exchange): 200 rows 14.0 / 9.0 us, 677 14.3 / 10.0, 3000 14.1 / 11.0, 6000 16.4 / 19.5,
// 24 000 36 / 58; up to 79 tiles 4.0..4.7 either way.  (Five tiles at once in one merge: no faster.)
constexpr int COMBINE_WAVES = 16;
constexpr int COMBINE_FEW_ROWS = 3072;

__device__ __forceinline__ void combine_merge(float& M, float& s, float& u, float m2, float s2, float u2) {
  const float mm = fmaxf(M, m2);
  const float a1 = __builtin_amdgcn_exp2f(M - mm), a2 = __builtin_amdgcn_exp2f(m2 - mm);
  u = a1 * (u + (M - mm) * s) + a2 * (u2 + (m2 - mm) * s2);
  s = a1 * s + a2 * s2;
  M = mm;
}

// The form of the call's dH launches, by one wavefront.  In front of every tile's first load, in each workgroup of a dH launch, the search took 1 to 3 us; here it
// runs beside the rows' epilogue and costs nothing.
__device__ __forceinline__ void settle_dh_form(const CombineArgs& a, int n_pad) {
  DhForm f{1, 1, false};
  if (a.blk.cap_t <= 0 || n_pad / BN <= a.blk.cap_t)       // (several token blocks are never split)
    f = dh_form(n_pad, a.dh.acc_rows, a.dh.n, dh_runs_whole(a.dh.rc, n_pad) ? a.dh.rc.tiles_v_all * (BM / BK) : a.dh.stages, a.dh.split_f32, a.dh.wide_ok);
  if ((threadIdx.x & 63) == 0) {
    a.ctl->dh_slabs = f.ks * f.products;
    a.ctl->dh_ks = f.ks; a.ctl->dh_products = f.products; a.ctl->dh_wide = f.wide;
  }
}

// SETTLES: the call has dH launches.
template <int R, bool SETTLES>
__global__ __launch_bounds__(64 * COMBINE_WAVES) void combine_kernel(CombineArgs a) {
  constexpr int PARTS = 64 * COMBINE_WAVES / R;
  __shared__ float sh[PARTS - 1][3][R];
  const Ctl ctl = *a.ctl;
  const int lane = threadIdx.x % R, part = threadIdx.x / R;
  int t0, nt;
  token_block(a.blk, ctl.n_pad / BN, t0, nt);
  if ((int)blockIdx.x * R >= nt * BN) return;   // whole workgroup beyond the padded rows
  const int i = t0 * BN + blockIdx.x * R + lane;
  float M = -1.0e30f, s = 0.f, u = 0.f;
  int k = part;
  for (; k + 3 * PARTS < a.tiles_v; k += 4 * PARTS) {
    float m2[4], s2[4], u2[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const size_t o = (size_t)(k + q * PARTS) * a.t_cap + i;
      m2[q] = a.part_m[o]; s2[q] = a.part_s[o]; u2[q] = a.part_u[o];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) combine_merge(M, s, u, m2[q], s2[q], u2[q]);
  }
  for (; k < a.tiles_v; k += PARTS) {
    const size_t o = (size_t)k * a.t_cap + i;
    combine_merge(M, s, u, a.part_m[o], a.part_s[o], a.part_u[o]);
  }
  if (R == 64) {
    if (part > 0) { sh[part - 1][0][lane] = M; sh[part - 1][1][lane] = s; sh[part - 1][2][lane] = u; }
    __syncthreads();
    if (part > 0) {
      if (SETTLES && blockIdx.x == 0 && part == COMBINE_WAVES - 1) settle_dh_form(a, ctl.n_pad);
      return;
    }
    for (int w = 0; w < PARTS - 1; ++w) combine_merge(M, s, u, sh[w][0][lane], sh[w][1][lane], sh[w][2][lane]);
  } else {                   // the parts of a wavefront by exchange, then those of the 16 wavefronts
#pragma unroll
    for (int w = R; w < 64; w *= 2) {
      const float m2 = __shfl_xor(M, w), s2 = __shfl_xor(s, w), u2 = __shfl_xor(u, w);
      combine_merge(M, s, u, m2, s2, u2);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) < R) { sh[wave][0][lane] = M; sh[wave][1][lane] = s; sh[wave][2][lane] = u; }
    __syncthreads();
    if (wave > 0) {
      if (SETTLES && blockIdx.x == 0 && wave == COMBINE_WAVES - 1) settle_dh_form(a, ctl.n_pad);
      return;
    }
    constexpr int EACH = COMBINE_WAVES * R / 64;           // wavefronts' states of a lane
    const int first = (threadIdx.x / R) * EACH;
    M = sh[first][0][lane]; s = sh[first][1][lane]; u = sh[first][2][lane];
#pragma unroll
    for (int w = 1; w < EACH; ++w) combine_merge(M, s, u, sh[first + w][0][lane], sh[first + w][1][lane], sh[first + w][2][lane]);
#pragma unroll
    for (int w = R; w < 64; w *= 2) {
      const float m2 = __shfl_xor(M, w), s2 = __shfl_xor(s, w), u2 = __shfl_xor(u, w);
      combine_merge(M, s, u, m2, s2, u2);
    }
    if ((int)threadIdx.x >= R) return;
  }
  const float LN2 = 0.693147180559945309f, LOG2E = 1.44269504088896341f;
  if (a.partials_out) {      // this shard's state of the row, natural-log units
    if (i < ctl.n_active)
      *reinterpret_cast<float4*>(a.partials_out + (size_t)a.rows[i] * 4) = make_float4(M * LN2, s, u * LN2, a.zy[i] * LN2);
    return;
  }
  float zy = a.zy[i];
  if (a.partials_in) {       // state merged over all shards; padded rows get lse = 0
    M = 0.f; s = 1.f; u = 0.f; zy = 0.f;
    if (i < ctl.n_active) {
      const float4 q = *reinterpret_cast<const float4*>(a.partials_in + (size_t)a.rows[i] * 4);
      M = q.x * LOG2E; s = q.y; u = q.z * LOG2E; zy = q.w * LOG2E;
    }
  }
  const float log2s = __builtin_amdgcn_logf(s);     // v_log_f32: log2
  const float lse2 = M + log2s;
  a.lse2[i] = lse2;
  if (i >= ctl.n_active) {
    if (a.with_loss) { a.coefc[i] = 0.f; a.lossterm[i] = 0.f; }
    return;
  }
  const int row = a.rows[i];
  const float logp = (zy - lse2) * LN2;
  if (a.logp_out) a.logp_out[row] = logp;
  if (a.ent_out) a.ent_out[row] = (log2s - u / s) * LN2;
  if (a.lse_out) a.lse_out[row] = lse2 * LN2;
  if (!a.with_loss) return;
  if (a.with_loss == 2) {            // cross-entropy: l = -logp, dl/dlogp = -1
    a.coefc[i] = -1.f / ctl.norm * a.inv_tau;
    a.lossterm[i] = -logp;
    return;
  }
  const float A = a.a_tok[row], c = a.c_tok[row];
  const float r = a.old_logp ? expf(logp - a.old_logp[row]) : 1.f;
  const float lo = 1.f - a.eps_lo, hi = 1.f + a.eps_hi;
  const float rc = fminf(fmaxf(r, lo), hi);
  float l = -fminf(r * A, rc * A);
  const bool flows = (A >= 0.f && r <= hi) || (A < 0.f && r >= lo);
  float g = flows ? -A * r : 0.f;
  if (r != r) { l = r; g = r; }      // fminf / fmaxf drop a NaN operand: a NaN ratio must reach the loss
  if (A >= 0.f && r > hi) atomicAdd(&a.counters[1], 1ull);
  if (A < 0.f && r < lo) atomicAdd(&a.counters[2], 1ull);
  a.coefc[i] = c * g / ctl.norm * a.inv_tau;
  a.lossterm[i] = c * l;
}
void launch_combine(const CombineArgs& a, hipStream_t s) {
  const int rows = a.blk.cap_t > 0 ? a.blk.cap_t * BN : a.t_cap;
  const bool few = a.t_cap <= COMBINE_FEW_ROWS, settles = a.dh.n > 0 && a.blk.b == 0;
  auto kernel = few ? (settles ? combine_kernel<16, true> : combine_kernel<16, false>) : settles ? combine_kernel<64, true> : combine_kernel<64, false>;
  hipLaunchKernelGGL(kernel, dim3(rows / (few ? 16 : 64)), dim3(64 * COMBINE_WAVES), 0, s, a);
}

// One workgroup of 256, fixed order, fp64: loss = (sum_t c_t l_t) / norm; publishes the counters.  It runs as a
// workgroup of the scatter, the first one there (a launch of its own was 4..17 us).
__device__ __forceinline__ void finish_loss(const FinishArgs& a) {
  __shared__ double sh[256];
  const Ctl ctl = *a.ctl;
  const int tid = threadIdx.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  int i = tid;
  for (; i + 3 * 256 < ctl.n_active; i += 4 * 256)
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] += (double)a.lossterm[i + k * 256];
  for (; i < ctl.n_active; i += 256) acc[0] += (double)a.lossterm[i];
  sh[tid] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) sh[tid] += sh[tid + w];
    __syncthreads();
  }
  if (tid == 0 && a.loss_out) *a.loss_out = (float)(sh[0] / (double)ctl.norm);
  if (tid < 8 && a.counters_out) a.counters_out[tid] = (long long)a.counters[tid];
}

// Adds the slabs of a split dW contraction (dw_split) in order, and the gradient that was there if it accumulates:
// workgroup `group` of `groups` of 256.  With one vocab chunk they are workgroups of the scatter, behind the finish (a launch of
// its own, which a call of few active rows makes for nothing, was 4.6 us).
__device__ __forceinline__ void dw_fold(const DwFoldArgs& a, int group, int groups) {
  const int slabs = dw_split(dw_stages(a.ctl->n_active), a.dw_cap) * a.products;
  if (slabs == 1) return;                           // the contraction wrote dW itself
  for (long long e = ((long long)group * 256 + threadIdx.x) * 4; e < a.n; e += (long long)groups * 256 * 4) {
    f32x4 v = *reinterpret_cast<const f32x4*>(a.slabs + e);
    for (int q = 1; q < slabs; ++q) v += *reinterpret_cast<const f32x4*>(a.slabs + q * a.slab + e);
    if (a.out_bf16) {
      bf16x4* p = reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(a.dW) + e);
      if (a.accumulate) {
        const bf16x4 old = *p;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] += (float)old[r];
      }
      bf16x4 o;
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = (__bf16)v[r];
      *p = o;
    } else {
      f32x4* p = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.dW) + e);
      if (a.accumulate) v += *p;
      *p = v;
    }
  }
}
__global__ __launch_bounds__(256) void dw_fold_kernel(DwFoldArgs a) { dw_fold(a, (int)blockIdx.x, (int)gridDim.x); }
static int dw_fold_groups(const DwFoldArgs& a) {
  const long long groups = (a.n / 4 + 255) / 256;
  return (int)(groups < 2048 ? groups : 2048);
}
void launch_dw_fold(const DwFoldArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(dw_fold_kernel, dim3(dw_fold_groups(a)), dim3(256), 0, s, a);
}

// ------------------------------------------------------------------ dH scatter
// dH[t,:] = accumulated row of its compacted position, or zeros for rows that are not active.
// A thread requests AHEAD slabs at once (one after the other, 16 slabs of 200 rows, d = 5120, took 24.5 us; with seven and the split below 12.4).  FEW: calls of few
// rows.  The slabs go by the active rows, so a call of many rows has as many of them when few are active, but seven at once cost such a launch more for the rows
// that have none.  One / four / seven: 177 of 12352 rows, 2304 x 15669, 27.6 / 18.4 / 23.2 us; 100 of 4000, 1024 x 100000, 22.7 / 11.6 / 12.2; 200 of
// 16000, 1024 x 65536, 32.5 / 23.1 / 23.4; all of 40 000, d = 64, 14.8 / 14.7 / 17.4; all of 20 000, d = 512, 15.0 / 15.5 / 17.1.
// Rows without a slab take a way of their own, to which the wider loop is no burden.  In one way / apart: 780 of 39 013 rows, d = 896, 35.4 / 24.3 us; 760 of
// 37 930, d = 2240, 39.5 / 31.8; 177 of 12 352, d = 2304, 18.7 / 17.4; all of 40 000, d = 64, 14.7 / 15.4.
constexpr int SCATTER_FEW_ROWS = 2048;
template <bool FEW>
__global__ __launch_bounds__(256) void scatter_dh_kernel(ScatterArgs a, FinishArgs fin, DwFoldArgs fold, int fold_groups) {
  const int t = (int)blockIdx.x - 1 - fold_groups;
  if (FEW && t < 0 && blockIdx.y) return;
  if (blockIdx.x == 0) return finish_loss(fin);
  if (t < 0) return dw_fold(fold, (int)blockIdx.x - 1, fold_groups);
  const int p = a.pos[t];
  const float* src = a.acc + (size_t)p * a.d;         // (not followed where there is none)
  const int n_pad = a.ctl->n_pad;
  const int ks = a.ctl->dh_slabs;
  const size_t slab = (size_t)n_pad * a.d;
  if (__builtin_expect(p < 0, 0)) {
    for (int j = ((FEW ? blockIdx.y * 256 : 0) + threadIdx.x) * 4; j < a.d; j += (FEW ? gridDim.y : 1) * (256 * 4)) {
      if (a.out_f32) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.dH) + (size_t)t * a.d + j) = f32x4{};
      else *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(a.dH) + (size_t)t * a.d + j) = bf16x4{};
    }
    return;
  }
  for (int j = ((FEW ? blockIdx.y * 256 : 0) + threadIdx.x) * 4; j < a.d; j += (FEW ? gridDim.y : 1) * (256 * 4)) {
    f32x4 v = *reinterpret_cast<const f32x4*>(src + j);
    constexpr int AHEAD = FEW ? 7 : 4;
    int q = 1;
    for (; q + AHEAD <= ks; q += AHEAD) {               // split-K slabs, added in a fixed order
      f32x4 w[AHEAD];
#pragma unroll
      for (int r = 0; r < AHEAD; ++r) w[r] = *reinterpret_cast<const f32x4*>(src + (q + r) * slab + j);
#pragma unroll
      for (int r = 0; r < AHEAD; ++r) v += w[r];
    }
    for (; q < ks; ++q) v += *reinterpret_cast<const f32x4*>(src + q * slab + j);
    if (a.out_f32) {
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.dH) + (size_t)t * a.d + j) = v;
    } else {
      bf16x4 o;
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = (__bf16)v[r];
      *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(a.dH) + (size_t)t * a.d + j) = o;
    }
  }
}
// ------------------------------------------------------------------ vocab-sharded head
// The reduction operator of the exchange between vocab shards: per row, the softmax states
// (m, s, u) of two disjoint vocab ranges merge by the online-softmax rule and the sampled
// token's logit (held by one shard, 0 elsewhere) by addition.  Rows nobody computed are all
// zeros and stay so.  out may alias a or b.
__global__ void merge_partials_kernel(const float* a, const float* b, float* out, long long T) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const float4 p = *reinterpret_cast<const float4*>(a + t * 4), q = *reinterpret_cast<const float4*>(b + t * 4);
  float4 r;
  if (p.y == 0.f) {          // empty state on one side: the other side unchanged
    r = make_float4(q.x, q.y, q.z, p.w + q.w);
  } else if (q.y == 0.f) {
    r = make_float4(p.x, p.y, p.z, p.w + q.w);
  } else {
    const float mm = fmaxf(p.x, q.x);
    const float a1 = expf(p.x - mm), a2 = expf(q.x - mm);
    r.x = mm;
    r.y = a1 * p.y + a2 * q.y;
    r.z = a1 * (p.z + (p.x - mm) * p.y) + a2 * (q.z + (q.x - mm) * q.y);
    r.w = p.w + q.w;
  }
  *reinterpret_cast<float4*>(out + t * 4) = r;
}
void launch_merge_partials(const float* a, const float* b, float* out, long long T, hipStream_t s) {
  if (T <= 0) return;
  hipLaunchKernelGGL(merge_partials_kernel, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, s, a, b, out, T);
}

__global__ void finish_partials_kernel(const float* parts, long long T, float* logp, float* ent, float* lse) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const float4 p = *reinterpret_cast<const float4*>(parts + t * 4);
  float lp = 0.f, en = 0.f, ls = 0.f;
  if (p.y != 0.f) {
    const float lns = logf(p.y);
    ls = p.x + lns;
    lp = p.w - ls;
    en = lns - p.z / p.y;
  }
  if (logp) logp[t] = lp;
  if (ent) ent[t] = en;
  if (lse) lse[t] = ls;
}
void launch_finish_partials(const float* parts, long long T, float* logp, float* ent, float* lse, hipStream_t s) {
  if (T <= 0) return;
  hipLaunchKernelGGL(finish_partials_kernel, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, s, parts, T, logp, ent, lse);
}

// Few rows: a row's columns over several workgroups, or too few bytes are in flight.  One workgroup a row / 1024 columns each, d = 5120: 512 rows 13.9 / 12.3 us,
// 1013 rows 15.1 / 15.1; d = 4096, 100 rows of 16 slabs 15.3 / 6.2; but 4000 rows 20.6 / 25.9, 16 000 82 / 104.
constexpr int SCATTER_PARTS_ROWS = 512;
void launch_scatter_dh(const ScatterArgs& a, const FinishArgs& fin, const DwFoldArgs& fold, hipStream_t s) {
  if (a.T <= 0) return;
  const int f = dw_fold_groups(fold);
  const int parts = a.T <= SCATTER_PARTS_ROWS ? (a.d + 1023) / 1024 : 1;
  if (a.T <= SCATTER_FEW_ROWS) hipLaunchKernelGGL(scatter_dh_kernel<true>, dim3(a.T + 1 + f, parts), dim3(256), 0, s, a, fin, fold, f);
  else hipLaunchKernelGGL(scatter_dh_kernel<false>, dim3(a.T + 1 + f), dim3(256), 0, s, a, fin, fold, f);
}

// ------------------------------------------------------------------ rewards (Eq. 1, Eq. 6-7)
__global__ void turn_reward_kernel(RewardArgs a) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  double R = 0.0, pr = 0.0;
  if (a.correct[i]) {
    const double speedup = fmin((double)a.t_reference[i] / (double)a.t_kernel[i], (double)a.cap);
    R = 1.0 + speedup;
    if (a.t_generated) {
      pr = (double)a.t_generated[i] / (double)a.t_total[i];
      R += pr;
    }
  }
  a.rewards_out[i] = (float)R;
  if (a.pr_out) a.pr_out[i] = (float)pr;
}
void launch_turn_reward(const RewardArgs& a, hipStream_t s) {
  if (a.n <= 0) return;
  hipLaunchKernelGGL(turn_reward_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s, a);
}

// ------------------------------------------------------------------ PRS (Sec. 5.2, Eq. 8)
// Philox-4x32 with 10 rounds (Salmon et al., SC'11), one block per sample; only the first
// output word is used.
__device__ __forceinline__ uint32_t philox4x32_10_word0(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                       uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c0;
}

__global__ void prs_retain_kernel(PrsArgs a) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const double pr = (double)a.pr[i];
  double p = (pr - (double)a.tau) / (double)a.s;
  p = fmin(fmax(p, 0.0), 1.0);
  bool keep = false;
  if (!a.valid || a.valid[i]) {
    if (a.hard) {
      keep = pr >= (double)a.tau;
    } else {
      const uint32_t x = philox4x32_10_word0((uint32_t)i, (uint32_t)((unsigned long long)i >> 32), 0u, 0u,
                                             (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
      const double u = ((double)x + 0.5) * (1.0 / 4294967296.0);
      keep = u < p;
    }
  }
  a.keep_out[i] = keep ? 1 : 0;
  if (a.p_out) a.p_out[i] = (float)p;
}
void launch_prs_retain(const PrsArgs& a, hipStream_t s) {
  if (a.n <= 0) return;
  hipLaunchKernelGGL(prs_retain_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s, a);
}

// ------------------------------------------------------------------ monitors (Sec. 5.1)
// Stage 1: MON_BLOCKS workgroups; workgroup b sums a fixed, contiguous slice of every input in
// fp64 (tree reduction in a fixed order).  Stage 2: one workgroup folds the partials, again in a
// fixed order, and writes the six monitors.
__device__ __forceinline__ double block_sum_256(double v, double* sh) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) sh[tid] += sh[tid + w];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// Sum of squares of 8 consecutive elements.
template <bool F32>
__device__ __forceinline__ double sumsq8(const void* p, long long u) {
  if constexpr (F32) {
    const f32x4 x = reinterpret_cast<const f32x4*>(p)[u * 2], y = reinterpret_cast<const f32x4*>(p)[u * 2 + 1];
    return ((double)x[0] * x[0] + (double)x[1] * x[1]) + ((double)x[2] * x[2] + (double)x[3] * x[3]) + (((double)y[0] * y[0] + (double)y[1] * y[1]) +
           ((double)y[2] * y[2] + (double)y[3] * y[3]));
  } else {
    const bf16x8 x = reinterpret_cast<const bf16x8*>(p)[u];
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) { const double v = (double)(float)x[e]; acc += v * v; }
    return acc;
  }
}
// Slice b of MON_BLOCKS of n elements, in units of 8 so that loads stay 16-byte aligned, four steps' loads in
// flight: 3.56 GB 606 -> 594 us, 6.0 TB/s.  (Interleaving the workgroups' units over the whole array: 669 us.)
template <bool F32>
__device__ __forceinline__ double sumsq_share(const void* p, long long n, int b, int tid) {
  const long long units = n / 8, per = (units + MON_BLOCKS - 1) / MON_BLOCKS;
  long long u = (long long)b * per + tid;
  const long long u1 = (long long)(b + 1) * per < units ? (long long)(b + 1) * per : units;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (; u + 3 * 256 < u1; u += 4 * 256)
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] += sumsq8<F32>(p, u + k * 256);
  for (; u < u1; u += 256) acc[0] += sumsq8<F32>(p, u);
  if (b == 0 && tid < (int)(n & 7)) {
    const long long e = units * 8 + tid;
    const double v = F32 ? reinterpret_cast<const float*>(p)[e] : (double)(float)reinterpret_cast<const __bf16*>(p)[e];
    acc[1] += v * v;
  }
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}
__device__ __forceinline__ double sumsq_share(const void* p, int is_f32, long long n, int b, int tid) {
  return is_f32 ? sumsq_share<true>(p, n, b, tid) : sumsq_share<false>(p, n, b, tid);
}

__global__ __launch_bounds__(256) void monitors_partial_kernel(MonitorArgs a) {
  __shared__ double sh[256];
  const int b = blockIdx.x, tid = threadIdx.x;
  const long long per = (a.T + MON_BLOCKS - 1) / MON_BLOCKS;
  const long long t0 = (long long)b * per, t1 = t0 + per < a.T ? t0 + per : a.T;
  double s_ent = 0.0, s_tr = 0.0, s_ro = 0.0, s_n = 0.0;
  for (long long t = t0 + tid; t < t1; t += 256) {
    if (a.mask[t]) {
      s_n += 1.0;
      s_tr += (double)a.logp_train[t];
      if (a.logp_rollout) s_ro += (double)a.logp_rollout[t];
      if (a.entropy) s_ent += (double)a.entropy[t];
    }
  }
  const double r0 = block_sum_256(s_ent, sh), r1 = block_sum_256(s_tr, sh), r2 = block_sum_256(s_ro, sh),
               r5 = block_sum_256(s_n, sh);
  const double r3 = a.dH ? block_sum_256(sumsq_share(a.dH, a.dH_f32, a.dH_elems, b, tid), sh) : 0.0;
  const double r4 = a.dW ? block_sum_256(sumsq_share(a.dW, a.dW_f32, a.dW_elems, b, tid), sh) : 0.0;
  if (tid == 0) {
    a.partial[0 * MON_BLOCKS + b] = r0; a.partial[1 * MON_BLOCKS + b] = r1; a.partial[2 * MON_BLOCKS + b] = r2;
    a.partial[3 * MON_BLOCKS + b] = r3; a.partial[4 * MON_BLOCKS + b] = r4; a.partial[5 * MON_BLOCKS + b] = r5;
  }
}

__global__ __launch_bounds__(256) void monitors_final_kernel(MonitorArgs a) {
  __shared__ double sh[256];
  __shared__ double tot[6];
  const int tid = threadIdx.x;
  for (int q = 0; q < 6; ++q) {
    double v = 0.0;
    for (int b = tid; b < MON_BLOCKS; b += 256) v += a.partial[q * MON_BLOCKS + b];
    const double r = block_sum_256(v, sh);
    if (tid == 0) tot[q] = r;
  }
  __syncthreads();
  if (tid == 0) {
    const double n = tot[5], den = n > 0.0 ? n : 1.0;
    a.out[0] = a.entropy ? tot[0] / den : 0.0;
    a.out[1] = exp(-tot[1] / den);
    a.out[2] = a.logp_rollout ? exp(-tot[2] / den) : 0.0;
    a.out[3] = sqrt(tot[3]);
    a.out[4] = sqrt(tot[4]);
    a.out[5] = n;
    a.out[6] = 0.0;
    a.out[7] = 0.0;
  }
}
void launch_monitors(const MonitorArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(monitors_partial_kernel, dim3(MON_BLOCKS), dim3(256), 0, s, a);
  hipLaunchKernelGGL(monitors_final_kernel, dim3(1), dim3(256), 0, s, a);
}

// ------------------------------------------------------------------ RMSNorm in front of the head
// h = x * rstd * gamma, rstd = 1 / sqrt(mean x^2 + eps).  One wavefront per row, 16-byte (bf16) or
// 32-byte (fp32) accesses of 8 consecutive elements per lane and step; fp32 arithmetic, the sum of
// squares reduced in a fixed butterfly order.  Both kernels hold the current row in registers and
// read every element once; they are HBM-bound.
template <bool F32>
__device__ __forceinline__ void load8(const void* p, long long elem, float (&v)[8]) {
  if (F32) {
    const float4 a = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(p) + elem);
    const float4 b = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(p) + elem + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const __bf16*>(p) + elem);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)a[e];
  }
}
template <bool F32, bool NT = false>
__device__ __forceinline__ void store8(void* p, long long elem, const float (&v)[8]) {
  if (F32) {
    const f32x4 a = {v[0], v[1], v[2], v[3]}, b = {v[4], v[5], v[6], v[7]};
    f32x4* q = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p) + elem);
    if (NT) {
      __builtin_nontemporal_store(a, q);
      __builtin_nontemporal_store(b, q + 1);
    } else {
      q[0] = a;
      q[1] = b;
    }
  } else {
    bf16x8 a;
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = (__bf16)v[e];
    bf16x8* q = reinterpret_cast<bf16x8*>(reinterpret_cast<__bf16*>(p) + elem);
    if (NT) __builtin_nontemporal_store(a, q);
    else *q = a;
  }
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int sh = 32; sh >= 1; sh >>= 1) v += __shfl_xor(v, sh);
  return v;
}
// Forward: a lane keeps its (up to) NORM_FC x 8 elements of the row in registers between the sum
// of squares and the scaling, so every element of X is read from memory once.  All loads of the
// row are issued before the first use, so they are in flight together.
constexpr int NORM_FC = NORM_MAX_D / 512;          // 8-column steps per lane

template <bool F32> struct Raw8;
template <> struct Raw8<true> { f32x4 a, b; };
template <> struct Raw8<false> { bf16x8 v; };
__device__ __forceinline__ void raw_load(const void* p, long long elem, Raw8<true>& r) {
  r.a = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p) + elem);
  r.b = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p) + elem + 4);
}
__device__ __forceinline__ void raw_load(const void* p, long long elem, Raw8<false>& r) {
  r.v = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const __bf16*>(p) + elem);
}
// ... past the caches
__device__ __forceinline__ void raw_stream(const void* p, long long elem, Raw8<true>& r) {
  r.a = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p) + elem));
  r.b = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p) + elem + 4));
}
__device__ __forceinline__ void raw_stream(const void* p, long long elem, Raw8<false>& r) {
  r.v = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(reinterpret_cast<const __bf16*>(p) + elem));
}
__device__ __forceinline__ void raw_unpack(const Raw8<true>& r, float (&v)[8]) {
  v[0] = r.a.x; v[1] = r.a.y; v[2] = r.a.z; v[3] = r.a.w; v[4] = r.b.x; v[5] = r.b.y; v[6] = r.b.z; v[7] = r.b.w;
}
__device__ __forceinline__ void raw_unpack(const Raw8<false>& r, float (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (float)r.v[e];
}

// Which of the two stand-alone kernels' accesses go past the caches, from calls in a trainer's order: what writes X, forward, head call,
// backward (X has long left the caches), what reads dX.  Sums of the store's launch and the reader's, plain / past the caches, in us:
//   H, read by the head's gather: bf16 d = 4096, 3000 rows 23.7 / 27.7, 6000 40.5 / 46.4, 14000 86.6 / 84.7, 20000 126.5 / 126.6, 24000 153.7 /
//   149.5; d = 5120, 27000 rows 212 / 195, 43697 351 / 337.  Read in place by a forward-only call (V = 32768): d = 4096, 12000 rows 2345 / 2355,
//   17000 3262 / 3291, 20000 3920 / 3915, 24000 4630 / 4597.  So from about 150 MB on, where X and H no longer share the memory-side cache.
//   dX: 3000 rows 30.5 / 31.8, 12000 97.5 / 103.9, 24000 210.8 / 218.0, 30000 267 / 272; d = 5120, 27000 rows 294 / 278, 43697 485 / 462.  So where
//   dX itself does not fit that cache; X, dH and the forward's X are then read past it too (27000 rows, all five launches: 643 -> 599).
//   fp32: past is never shorter (H 4000 x 1024 18.6 / 21.4, 8000 x 4096 114 / 116, 12000 x 5120 221 / 232; dX 21.3 / 22.3, 145 / 149, 274 / 276).
// (Forward and backward right after each other on one X like stores past the caches at any size, as X then stays for the backward: 20000 rows of
// d = 4096 137 us with all stores past them, 147 to 153 with these lines, 170 with plain ones; 17000 rows 118, 141 and 147; fp32, d = 5120, 8000
// rows 159 with all past them, 170 with none.  That is not the order of a step, so the lines follow the order above.)
constexpr long long NORM_H_PAST_BYTES = 144ll << 20;      // of one bf16 [T, d] matrix
constexpr long long NORM_ALL_PAST_BYTES = 256ll << 20;    // ... the memory-side cache's size

template <bool F32, bool NT_LOAD, bool NT_STORE>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(NormArgs a) {
  const int lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= a.T) return;
  Raw8<F32> raw[NORM_FC];
#pragma unroll
  for (int q = 0; q < NORM_FC; ++q) {
    const int c = lane * 8 + q * 512;
    if (c < a.d) NT_LOAD ? raw_stream(a.X, row * a.d + c, raw[q]) : raw_load(a.X, row * a.d + c, raw[q]);
  }
  float ss = 0.f;
#pragma unroll
  for (int q = 0; q < NORM_FC; ++q) {
    const int c = lane * 8 + q * 512;
    if (c < a.d) {
      float x[8];
      raw_unpack(raw[q], x);
#pragma unroll
      for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
    }
  }
  ss = wave_sum(ss);
  const float rstd = 1.f / sqrtf(ss / (float)a.d + a.eps);
  if (a.rstd_out && lane == 0) a.rstd_out[row] = rstd;
#pragma unroll
  for (int q = 0; q < NORM_FC; ++q) {
    const int c = lane * 8 + q * 512;
    if (c < a.d) {
      float x[8], g[8], h[8];
      raw_unpack(raw[q], x);
      load8<F32>(a.gamma, c, g);
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = x[e] * rstd * g[e];
      store8<F32, NT_STORE>(a.H, row * a.d + c, h);
    }
  }
}
static bool norm_past(const NormArgs& a, long long bytes) { return !a.is_f32 && a.T * a.d * 2 > bytes; }
void launch_rmsnorm_fwd(const NormArgs& a, hipStream_t s) {
  if (a.T <= 0) return;
  const unsigned grid = (unsigned)((a.T + 3) / 4);
  auto kernel = a.is_f32 ? rmsnorm_fwd_kernel<true, false, false>
                : norm_past(a, NORM_ALL_PAST_BYTES) ? rmsnorm_fwd_kernel<false, true, true>
                : norm_past(a, NORM_H_PAST_BYTES) ? rmsnorm_fwd_kernel<false, false, true> : rmsnorm_fwd_kernel<false, false, false>;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, s, a);
}

// Backward: dx = rstd (gamma g - xhat mean(gamma g xhat)), xhat = x rstd; dgamma = sum_rows g xhat.
// Workgroup b takes the rows b, b + NORM_STRIPS, b + 2 NORM_STRIPS, ... (so the workgroups running at
// one time read and write neighbouring rows: 4 % faster than a contiguous strip per workgroup); a thread
// owns the same (up to) 4 x 8 columns of every row, holds x and g of the current row in registers
// (each element is read once) and keeps the dgamma partial sums of its columns in registers.  The
// two row sums (x^2 and gamma g x) are reduced over the workgroup together, in a fixed order.  The
// workgroups' partials are folded by the second kernel.
constexpr int NORM_NC = NORM_MAX_D / 2048;         // 8-column steps per thread at the largest d
static_assert(NORM_NC == 4, "the launcher instantiates 1..4 steps");

__device__ __forceinline__ float block_sum4(float v, float* red, int lane, int wave) {
  v = wave_sum(v);
  if (lane == 0) red[wave] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Keeps the register values of a packed row opaque to the optimiser between the two passes over a row, so that
// the unpacked fp32 copies of the first pass are not kept alive across the reduction (they are unpacked again).
__device__ __forceinline__ void opaque(Raw8<true>& r) { asm volatile("" : "+v"(r.a), "+v"(r.b)); }
__device__ __forceinline__ void opaque(Raw8<false>& r) {
  i32x4 v = __builtin_bit_cast(i32x4, r.v);
  asm volatile("" : "+v"(v));
  r.v = __builtin_bit_cast(bf16x8, v);
}

// NC: 8-column steps per thread, ceil(d / 2048).  Rows stay in registers as loaded (bf16 rows packed) and are
// unpacked on the fly in both passes: with three steps and bf16 rows the kernel fits 4 workgroups on a
// compute unit, each with one row of X and dH in flight ahead of the one it works on.
template <bool F32, int NC, bool PAST>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(NormArgs a) {
  __shared__ float red[2][8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const long long r0 = blockIdx.x, r1 = a.T;      // rows r0, r0 + NORM_STRIPS, ...
  float dg[NC][8];
  Raw8<F32> g_raw[NC] = {};
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = tid * 8 + q * 2048;
#pragma unroll
    for (int e = 0; e < 8; ++e) dg[q][e] = 0.f;
    if (c < a.d) raw_load(a.gamma, c, g_raw[q]);
  }
  const float inv_d = 1.f / (float)a.d;
  // The next row's loads are issued before the current row's workgroup reduction, so a
  // workgroup always has one row of X and dH in flight while it works on the previous one.
  Raw8<F32> xr[NC] = {}, gr_raw[NC] = {}, xn[NC] = {}, gn[NC] = {};
  auto fetch = [&](long long row, Raw8<F32> (&xa)[NC], Raw8<F32> (&ga)[NC]) {
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int c = tid * 8 + q * 2048;
      if (c < a.d) {
        PAST ? raw_stream(a.X, row * a.d + c, xa[q]) : raw_load(a.X, row * a.d + c, xa[q]);
        PAST ? raw_stream(a.dH, row * a.d + c, ga[q]) : raw_load(a.dH, row * a.d + c, ga[q]);
      }
    }
  };
  if (r0 < r1) fetch(r0, xr, gr_raw);
  int parity = 0;
  for (long long row = r0; row < r1; row += NORM_STRIPS, parity ^= 1) {
    if (row + NORM_STRIPS < r1) fetch(row + NORM_STRIPS, xn, gn);
    // sum x^2 and sum gamma g x in one workgroup reduction: mean_j(gamma_j g_j xhat_j) = rstd mean_j(gamma_j g_j x_j)
    float ss = 0.f, sd = 0.f;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int c = tid * 8 + q * 2048;
      if (c < a.d) {
        float x[8], gr[8], g[8];
        raw_unpack(xr[q], x);
        raw_unpack(gr_raw[q], gr);
        raw_unpack(g_raw[q], g);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          ss = fmaf(x[e], x[e], ss);
          sd = fmaf(g[e] * gr[e], x[e], sd);
        }
      }
    }
    ss = wave_sum(ss);
    sd = wave_sum(sd);
    float* rb = red[parity];                // alternating buffers: one barrier per row is enough
    if (lane == 0) { rb[wave] = ss; rb[4 + wave] = sd; }
    __syncthreads();
    const float rstd = 1.f / sqrtf(((rb[0] + rb[1]) + (rb[2] + rb[3])) * inv_d + a.eps);
    const float dot = ((rb[4] + rb[5]) + (rb[6] + rb[7])) * rstd * inv_d;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int c = tid * 8 + q * 2048;
      if (c < a.d) {
        opaque(xr[q]);
        opaque(gr_raw[q]);
        float x[8], gr[8], g[8], dx[8];
        raw_unpack(xr[q], x);
        raw_unpack(gr_raw[q], gr);
        raw_unpack(g_raw[q], g);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float xh = x[e] * rstd;
          dx[e] = rstd * (g[e] * gr[e] - xh * dot);
          dg[q][e] = fmaf(gr[e], xh, dg[q][e]);
        }
        store8<F32, PAST>(a.dX, row * a.d + c, dx);
      }
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) { xr[q] = xn[q]; gr_raw[q] = gn[q]; }
  }
  float* part = a.partial + (size_t)blockIdx.x * a.d;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = tid * 8 + q * 2048;
    if (c < a.d) {
      *reinterpret_cast<float4*>(part + c) = make_float4(dg[q][0], dg[q][1], dg[q][2], dg[q][3]);
      *reinterpret_cast<float4*>(part + c + 4) = make_float4(dg[q][4], dg[q][5], dg[q][6], dg[q][7]);
    }
  }
}

// dgamma[c] = sum over the strips' partials, in a fixed order: workgroup = 32 columns (four per lane) x 32 strip
// groups; group k adds strips k, k + 32, ... in eight interleaved chains, then the groups are folded four, eight at a time.
// Only as many strips as there are rows leave a partial: both calls at 257 rows, d = 5824, fp32 30.0 -> 21.3 us.  Bound by latency: with
// all strips the 32 loads of a lane have no condition and are in flight together, 1024 strips of d = 4096 5.5 us (3 TB/s), of 5120 6.0; eight
// at a time, each with its condition, 11.7 and 13.1; by single floats 11.1 and 12.5.
__global__ __launch_bounds__(256) void rmsnorm_dgamma_kernel(NormArgs a) {
  __shared__ f32x4 sh[32][8];
  const int l4 = threadIdx.x & 7, grp = threadIdx.x >> 3;
  const int c = blockIdx.x * 32 + l4 * 4;
  f32x4 acc[8] = {};
  if (c < a.d && a.strips == NORM_STRIPS) {
#pragma unroll
    for (int b = 0; b < NORM_STRIPS; b += 256)
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] += *reinterpret_cast<const f32x4*>(a.partial + (size_t)(b + grp + 32 * k) * a.d + c);
  } else if (c < a.d) {
    for (int b = grp; b < a.strips; b += 256)
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (b + 32 * k < a.strips) acc[k] += *reinterpret_cast<const f32x4*>(a.partial + (size_t)(b + 32 * k) * a.d + c);
  }
  sh[grp][l4] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  __syncthreads();
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (grp < 8) v = (sh[grp][l4] + sh[grp + 8][l4]) + (sh[grp + 16][l4] + sh[grp + 24][l4]);
  __syncthreads();
  if (grp < 8) sh[grp][l4] = v;
  __syncthreads();
  if (grp == 0 && c < a.d) {
#pragma unroll
    for (int k = 1; k < 8; ++k) v += sh[k][l4];
    // (the caller's: 4-byte aligned, a slice of a flat gradient buffer for instance)
#pragma unroll
    for (int e = 0; e < 4; ++e) a.dgamma[c + e] = v[e];
  }
}
static_assert(NORM_STRIPS % 256 == 0, "strip groups");

template <bool F32, bool PAST>
static void launch_rmsnorm_bwd_rows(const NormArgs& a, hipStream_t s) {
  switch ((a.d + 2047) / 2048) {     // 8-column steps per thread; d <= NORM_MAX_D is checked by the caller
    case 1: hipLaunchKernelGGL((rmsnorm_bwd_kernel<F32, 1, PAST>), dim3(a.strips), dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL((rmsnorm_bwd_kernel<F32, 2, PAST>), dim3(a.strips), dim3(256), 0, s, a); break;
    case 3: hipLaunchKernelGGL((rmsnorm_bwd_kernel<F32, 3, PAST>), dim3(a.strips), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((rmsnorm_bwd_kernel<F32, NORM_NC, PAST>), dim3(a.strips), dim3(256), 0, s, a); break;
  }
}
void launch_rmsnorm_bwd(const NormArgs& args, hipStream_t s) {
  NormArgs a = args;
  a.strips = (int)(a.T < NORM_STRIPS ? a.T : NORM_STRIPS);      // (a strip without a row leaves no partial)
  if (a.strips > 0) {
    if (a.is_f32) launch_rmsnorm_bwd_rows<true, false>(a, s);
    else if (norm_past(a, NORM_ALL_PAST_BYTES)) launch_rmsnorm_bwd_rows<false, true>(a, s);
    else launch_rmsnorm_bwd_rows<false, false>(a, s);
  }
  hipLaunchKernelGGL(rmsnorm_dgamma_kernel, dim3((a.d + 31) / 32), dim3(256), 0, s, a);
}


// ------------------------------------------------------------------ RMSNorm fused around the head
// Forward, fused into the row compaction: one wavefront per compacted row reads the row of X once,
// keeps it in registers between the sum of squares and the scaling (as rmsnorm_fwd_kernel), rounds
// h = x rstd gamma to bf16 (fp32 inputs: splits it into bf16 hi + lo parts, [hi | hi | lo] along k) and
// writes it as the head's compacted operand row; rows that are not active are never read.
template <bool F32>
__global__ __launch_bounds__(256) void norm_gather_kernel(GatherArgs a, NormFuse n) {
  const Ctl ctl = *a.ctl;
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= ctl.n_pad) return;
  const bool live = i < ctl.n_active;
  const int t = live ? a.rows[i] : 0;
  if (lane == 0) {
    int yl = -1;
    if (live) {
      yl = a.y[t] - a.y_offset;
      if (yl < 0 || yl >= a.V) yl = -1;
    }
    a.yc[i] = yl;
  }
  Raw8<F32> raw[NORM_FC];
  if (live) {
#pragma unroll
    for (int q = 0; q < NORM_FC; ++q) {
      const int c = lane * 8 + q * 512;
      if (c < a.d) raw_load(n.X, (long long)t * a.d + c, raw[q]);
    }
  }
  float ss = 0.f;
  if (live) {
#pragma unroll
    for (int q = 0; q < NORM_FC; ++q) {
      const int c = lane * 8 + q * 512;
      if (c < a.d) {
        float x[8];
        raw_unpack(raw[q], x);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
      }
    }
  }
  ss = wave_sum(ss);
  const float rstd = live ? 1.f / sqrtf(ss / (float)a.d + n.eps) : 0.f;
  if (lane == 0) n.rstd_c[i] = rstd;
  const int ldh = F32 ? 3 * a.d : a.d;
#pragma unroll
  for (int q = 0; q < NORM_FC; ++q) {
    const int c = lane * 8 + q * 512;
    if (c < a.d) {
      float h[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (live) {
        float x[8], g[8];
        raw_unpack(raw[q], x);
        load8<F32>(n.gamma, c, g);
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = x[e] * rstd * g[e];
      }
      __bf16* o = a.Hc + (size_t)i * ldh + c;
      if (F32) {
        bf16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) { __bf16 x, y; split_bf16(h[e], x, y); hi[e] = x; lo[e] = y; }
        *reinterpret_cast<bf16x8*>(o) = hi;
        *reinterpret_cast<bf16x8*>(o + a.d) = hi;
        *reinterpret_cast<bf16x8*>(o + 2 * a.d) = lo;
      } else {
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (__bf16)h[e];
        *reinterpret_cast<bf16x8*>(o) = v;
      }
    }
  }
}

// HcT[j, i] = Hc[i, j] for d columns of row stride ldh (the bf16 operand; the hi or the lo parts of a split fp32 one).
__global__ __launch_bounds__(256) void transpose_hc_kernel(const __bf16* Hc, int ldh, __bf16* HcT, int ld_t, const Ctl* ctlp) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[64 * TT_LD];
  const int i0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
  if (i0 >= ctlp->n_pad) return;
  const int tid = threadIdx.x, chunk = tid & 7;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int r = (tid >> 3) + 32 * p;
    tt_put(tile, r, chunk, *reinterpret_cast<const i32x4*>(Hc + (size_t)(i0 + r) * ldh + j0 + chunk * 8));
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int jj = (tid >> 3) + 32 * p;
    *reinterpret_cast<i32x4*>(HcT + (size_t)(j0 + jj) * ld_t + i0 + chunk * 8) = tt_get(tile, jj, chunk);
  }
}

void launch_transpose_hc(const __bf16* Hc, int ldh, __bf16* HcT, const GatherArgs& g, hipStream_t s) {
  hipLaunchKernelGGL(transpose_hc_kernel, dim3(g.t_cap / 64, g.d / 64), dim3(256), 0, s, Hc, ldh, HcT, g.ld_t, g.ctl);
}

void launch_norm_gather(const GatherArgs& g, const NormFuse& n, hipStream_t s) {
  if (g.is_f32) hipLaunchKernelGGL(norm_gather_kernel<true>, dim3(g.t_cap / 4), dim3(256), 0, s, g, n);
  else hipLaunchKernelGGL(norm_gather_kernel<false>, dim3(g.t_cap / 4), dim3(256), 0, s, g, n);
  if (g.HcT) launch_transpose_hc(g.Hc, g.is_f32 ? 3 * g.d : g.d, g.HcT, g, s);
  if (g.HcT_lo) launch_transpose_hc(g.Hc + 2 * g.d, 3 * g.d, g.HcT_lo, g, s);
}

// Backward, fused into the scatter of dH: workgroup b takes the T-rows b, b + NORM_STRIPS, ... (as
// rmsnorm_bwd_kernel) and a thread the same (up to) 4 x 8 columns of every row.  For an active row
// the accumulated fp32 gradient g of its compacted position (split-K slabs added in order) and the
// row of X are read once, rstd comes from the forward,
//   dx = rstd (gamma g - xhat mean_j(gamma_j g_j xhat_j)),  xhat = x rstd,
// and g xhat is added to the thread's dgamma partial sums; rows that are not active are written as
// zeros and nothing of theirs is read.  The workgroups' partials are folded by rmsnorm_dgamma_kernel.
template <bool F32, int NC>
__global__ __launch_bounds__(256) void scatter_dx_norm_kernel(ScatterArgs a, NormFuse n, FinishArgs fin, DwFoldArgs fold) {
  if (blockIdx.x == NORM_STRIPS) return finish_loss(fin);
  if (blockIdx.x > NORM_STRIPS) return dw_fold(fold, (int)blockIdx.x - NORM_STRIPS - 1, (int)gridDim.x - NORM_STRIPS - 1);
  __shared__ float red[2][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const long long T = a.T;
  const int n_pad = a.ctl->n_pad;
  const int ks = a.ctl->dh_slabs;
  const size_t slab = (size_t)n_pad * a.d;
  float dg[NC][8];
  Raw8<F32> gam_raw[NC] = {};
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = tid * 8 + q * 2048;
#pragma unroll
    for (int e = 0; e < 8; ++e) dg[q][e] = 0.f;
    if (c < a.d) raw_load(n.gamma, c, gam_raw[q]);
  }
  // Slabs requested at once, before the next row's inputs are.  More, or two in a bf16 head of two column groups, take registers that cost a compute unit
  // wavefronts (4000 rows of d = 4096, one slab, two at once 35.2 -> 38.1 us).
  // One / two at once: 189 of 3192 rows, 7360 x 39365, 48.3 / 38.7 us; 200 rows, 5120 x 151936, 21.1 / 17.3; 1738 of 8855, 320 x 11839, 41.5 / 30.6; 681 of
  // 7834, 256 x 3145, 25.4 / 18.4; one slab, 20 000 rows of d = 1024 45.4 / 45.2.
  constexpr int AHEAD = !F32 && NC == 2 ? 1 : 2;
  const float inv_d = 1.f / (float)a.d;
  // Row r of the workgroup is T-row blockIdx.x + r NORM_STRIPS; the inputs of the next one (its compacted
  // position, rstd, the row of X and the first slab of the accumulator) are requested before the current
  // row's reduction.  An inactive row (position < 0) needs no input.
  Raw8<F32> xc[NC] = {}, xn[NC] = {};
  Raw8<true> gc[NC] = {}, gn[NC] = {};
  auto fetch = [&](long long row, Raw8<F32> (&xa)[NC], Raw8<true> (&ga)[NC], int& p, float& rstd) {
    p = a.pos[row];                                 // uniform over the workgroup
    if (p < 0) return;
    rstd = n.rstd_c[p];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int c = tid * 8 + q * 2048;
      if (c < a.d) {
        raw_load(n.X, row * a.d + c, xa[q]);
        raw_load(a.acc, (long long)p * a.d + c, ga[q]);
      }
    }
  };
  int pc = -1, parity = 0;
  float rc = 0.f;
  long long row = blockIdx.x;
  if (row < T) fetch(row, xc, gc, pc, rc);
  for (; row < T; row += NORM_STRIPS) {
    if (ks > 1 && pc >= 0) {                        // split-K slabs, added in a fixed order
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int c = tid * 8 + q * 2048;
        if (c >= a.d) continue;
        const float* src = a.acc + (size_t)pc * a.d + c;
        int k = 1;
        for (; k + AHEAD <= ks; k += AHEAD) {
          Raw8<true> w[AHEAD];
#pragma unroll
          for (int r = 0; r < AHEAD; ++r) raw_load(src, (long long)((k + r) * slab), w[r]);
#pragma unroll
          for (int r = 0; r < AHEAD; ++r) { gc[q].a += w[r].a; gc[q].b += w[r].b; }
        }
        for (; k < ks; ++k) {
          Raw8<true> w;
          raw_load(src, (long long)(k * slab), w);
          gc[q].a += w.a; gc[q].b += w.b;
        }
      }
    }
    int pn = -1;
    float rn = 0.f;
    if (row + NORM_STRIPS < T) fetch(row + NORM_STRIPS, xn, gn, pn, rn);
    if (pc < 0) {
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int c = tid * 8 + q * 2048;
        const float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (c < a.d) store8<F32>(a.dH, row * a.d + c, z);
      }
    } else {
      const float rstd = rc;
      float dot = 0.f;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int c = tid * 8 + q * 2048;
        if (c < a.d) {
          float x[8], g[8], gam[8];
          raw_unpack(xc[q], x);
          raw_unpack(gc[q], g);
          raw_unpack(gam_raw[q], gam);
#pragma unroll
          for (int e = 0; e < 8; ++e) dot = fmaf(gam[e] * g[e], x[e] * rstd, dot);
        }
      }
      dot = wave_sum(dot);
      float* rb = red[parity];                      // alternating buffers: one barrier per row is enough
      parity ^= 1;
      if (lane == 0) rb[wave] = dot;
      __syncthreads();
      dot = ((rb[0] + rb[1]) + (rb[2] + rb[3])) * inv_d;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int c = tid * 8 + q * 2048;
        if (c < a.d) {
          opaque(xc[q]);
          float x[8], g[8], gam[8], dx[8];
          raw_unpack(xc[q], x);
          raw_unpack(gc[q], g);
          raw_unpack(gam_raw[q], gam);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float xh = x[e] * rstd;
            dx[e] = rstd * (gam[e] * g[e] - xh * dot);
            dg[q][e] = fmaf(g[e], xh, dg[q][e]);
          }
          store8<F32>(a.dH, row * a.d + c, dx);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) { xc[q] = xn[q]; gc[q] = gn[q]; }
    pc = pn; rc = rn;
  }
  float* part = n.partial + (size_t)blockIdx.x * a.d;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = tid * 8 + q * 2048;
    if (c < a.d) {
      *reinterpret_cast<float4*>(part + c) = make_float4(dg[q][0], dg[q][1], dg[q][2], dg[q][3]);
      *reinterpret_cast<float4*>(part + c + 4) = make_float4(dg[q][4], dg[q][5], dg[q][6], dg[q][7]);
    }
  }
}

template <bool F32>
static void launch_scatter_dx_norm_rows(const ScatterArgs& a, const NormFuse& n, const FinishArgs& fin, const DwFoldArgs& fold, hipStream_t s) {
  const dim3 grid(NORM_STRIPS + 1 + dw_fold_groups(fold));
  switch ((a.d + 2047) / 2048) {     // 8-column steps per thread; d <= NORM_MAX_D is checked by the caller
    case 1: hipLaunchKernelGGL((scatter_dx_norm_kernel<F32, 1>), grid, dim3(256), 0, s, a, n, fin, fold); break;
    case 2: hipLaunchKernelGGL((scatter_dx_norm_kernel<F32, 2>), grid, dim3(256), 0, s, a, n, fin, fold); break;
    case 3: hipLaunchKernelGGL((scatter_dx_norm_kernel<F32, 3>), grid, dim3(256), 0, s, a, n, fin, fold); break;
    default: hipLaunchKernelGGL((scatter_dx_norm_kernel<F32, NORM_NC>), grid, dim3(256), 0, s, a, n, fin, fold); break;
  }
}
void launch_scatter_dx_norm(const ScatterArgs& a, const NormFuse& n, const FinishArgs& fin, const DwFoldArgs& fold, hipStream_t s) {
  if (a.out_f32) launch_scatter_dx_norm_rows<true>(a, n, fin, fold, s);
  else launch_scatter_dx_norm_rows<false>(a, n, fin, fold, s);
  NormArgs f{};
  f.d = a.d; f.partial = n.partial; f.dgamma = n.dgamma; f.strips = NORM_STRIPS;
  hipLaunchKernelGGL(rmsnorm_dgamma_kernel, dim3((a.d + 31) / 32), dim3(256), 0, s, f);
}

}  // namespace pg
