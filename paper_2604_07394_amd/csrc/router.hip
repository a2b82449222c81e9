// flux_router: Layer Router in its inference form (Sec. 3.1): prefix/suffix pooling of the first
// and last `pool` token rows (App. C.1) -> Context Encoder Linear+SiLU -> Router Head Linear ->
// argmax (tie to FA).  Everything after the bf16 loads is fp32; nothing is rounded in between.
//
// Two launches (three where there are many sequences), tiny and latency-bound:
//  1. router_pool: partial column sums of the pooled rows.  grid (column blocks, row splits, batch);
//     a lane owns 8 adjacent columns (one 16-byte load per row), the 4 waves of a workgroup take
//     different rows and are merged in LDS.  Row splits keep whole-sequence pooling (pool = 0) spread
//     over the chip; with pool > 0 the cost is independent of the sequence length.
//  2. router_mlp: grid (inner/8, batch); each wave produces two hidden units (dot of a bf16 W1 row
//     with the pooled fp32 vector held in LDS) and applies SiLU; the workgroup that finishes a sequence's
//     hidden vector turns it into the two logits and the decision (in launches of many workgroups a third kernel does).
// Batch 4, hidden 4096, inner 256, pool 100: 17.4 us per call with the head as a
// third launch and the loads of a column block waiting for those of the one before, 12.8 without, 11.9 with the counters of
// the sequences on lines of their own (16 sequences 23.4 and 19.6), 11.5 and 17.1 with two row splits instead of seven.
#include "flux_internal.h"

namespace flux {

struct PoolArgs {
  const __bf16* x;
  const int32_t* cu;
  int hidden, pool, splits;
  float* psum;            // [batch, splits, hidden]
};

constexpr int kPoolRows = 8;            // rows per lane that are asked for at once where 16 lanes share a row
constexpr int kPoolOnce = 16 * kPoolRows;   // rows of a split then

// pooled row number t (0-based among the pooled rows) -> row of the sequence
__device__ __forceinline__ int pooled_row(int t, int n_rows, int pool, bool all) {
  return (all || t < pool) ? t : n_rows - 2 * pool + t;
}

// CL: lanes that share a row, 8 columns each.  64 (a wave per row) for whole sequences, which are streamed.  16 for pools: a
// workgroup reads what it would read otherwise, but as 128 rows of 128 columns, all asked for at once, so that a quarter of
// the row splits hold them all.  The MLP workgroups each read the sums of all splits of their sequence, next to 64 KB of
// weights: 16 KB per split at hidden 4096, of which pools of 100 + 100 rows had seven (us per call
// with seven / two, inner 256: batch 1 11.5 / 11.0, 4 12.4 / 11.5, 8 14.4 / 12.7, 16 19.9 / 17.1, 64 46.9 / 41.9; 512
// sequences of hidden 256 21.5 / 17.1, hidden 1024, inner 64, batch 4 8.2 either way; with rows and weights not in any cache batch 1
// 14.0 / 12.4, 4 14.6 / 12.8, 16 22.6 / 18.4, 64 57 / 45.5, hidden 1024, inner 64, batch 4 10.5 / 9.5.  One split of two rounds 12.3
// at batch 4, four 12.0).
template <int CL>
__global__ __launch_bounds__(256) void router_pool_kernel(PoolArgs a) {
  constexpr int RL = 256 / CL;                              // rows that the workgroup reads side by side
  constexpr int COLS = 8 * CL;
  constexpr int FLY = CL == 64 ? 4 : kPoolRows;             // rows per lane in flight
  __shared__ float red[4][COLS];
  const int tid = threadIdx.x, w = tid >> 6;
  const int cl = tid % CL;
  const int col = blockIdx.x * COLS + cl * 8;
  const int split = blockIdx.y, b = blockIdx.z;
  const int r0 = a.cu[b];
  const int n_rows = a.cu[b + 1] - r0;
  const bool all = a.pool <= 0 || n_rows <= 2 * a.pool;
  const int n_pooled = all ? n_rows : 2 * a.pool;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto add = [&](const u32x4& v) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[2 * i] += bf16_lo(v[i]);
      acc[2 * i + 1] += bf16_hi(v[i]);
    }
  };
  if (col < a.hidden) {
    const __bf16* xc = a.x + (int64_t)r0 * a.hidden + col;
    const int step = RL * a.splits;
    int t = split * RL + tid / CL;
    // several rows per round, so that independent 16-byte loads are in flight per lane; every row is
    // read once, hence nontemporal
    for (; CL == 64 ? t + (FLY - 1) * step < n_pooled : t < n_pooled; t += FLY * step) {
      u32x4 v[FLY];
#pragma unroll
      for (int u = 0; u < FLY; ++u) {
        const int tu = CL == 64 ? t + u * step : min(t + u * step, n_pooled - 1);   // (rows past the last one are not added)
        v[u] = __builtin_nontemporal_load((const u32x4*)(xc + (int64_t)pooled_row(tu, n_rows, a.pool, all) * a.hidden));
      }
#pragma unroll
      for (int u = 0; u < FLY; ++u)
        if (CL == 64 || t + u * step < n_pooled) add(v[u]);
    }
    if constexpr (CL == 64)
      for (; t < n_pooled; t += step) add(*(const u32x4*)(xc + (int64_t)pooled_row(t, n_rows, a.pool, all) * a.hidden));
  }
  if constexpr (CL == 16) {                                 // the four rows of a wave meet in its first 16 lanes
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] = sum_across_halves(acc[i]);
      acc[i] += __shfl_xor(acc[i], 16);
    }
  }
  if (CL == 64 || (tid & 63) < 16) {
#pragma unroll
    for (int i = 0; i < 8; ++i) red[w][cl * 8 + i] = acc[i];
  }
  __syncthreads();
  for (int c = tid; c < COLS; c += 256) {
    const int cc = blockIdx.x * COLS + c;
    if (cc < a.hidden)
      a.psum[((int64_t)b * a.splits + split) * a.hidden + cc] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
  }
}

struct MlpArgs {
  const float* psum;      // [batch, splits, hidden]
  const int32_t* cu;
  const __bf16* w1;
  const __bf16* b1;
  const __bf16* w2;
  const __bf16* b2;
  float* hbuf;            // [batch, inner]
  int batch, hidden, inner, pool, splits;
  uint32_t* arrived;      // [batch][stride] arrival counters, zero between calls (nullptr: the head is a launch of its own)
  int arrived_stride;
  uint8_t* mode_out;
  float* logits_out;
};

// Router Head: two dot products of length `inner` and the hard decision of one sequence, by one wave.  DEV: the hidden
// vector was written by workgroups of this launch (device-scope reads).
template <bool DEV>
__device__ __forceinline__ void router_head(const float* h, const __bf16* w2, const __bf16* b2, int inner, int l, uint8_t* mode_out,
                                            float* logits_out) {
  float s0 = 0.f, s1 = 0.f;
#pragma unroll 4
  for (int j = l; j < inner; j += 64) {
    const float hv = DEV ? __hip_atomic_load(h + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : h[j];
    s0 = __builtin_fmaf((float)w2[j], hv, s0);
    s1 = __builtin_fmaf((float)w2[inner + j], hv, s1);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_xor(s0, off);
    s1 += __shfl_xor(s1, off);
  }
  if (l == 0) {
    if (b2) {
      s0 += (float)b2[0];
      s1 += (float)b2[1];
    }
    *mode_out = s0 >= s1 ? 1 : 0;                            // argmax, tie -> index 0 = FA
    if (logits_out) {
      logits_out[0] = s0;
      logits_out[1] = s1;
    }
  }
}

// Bound by latencies: what a workgroup reads (8 weight rows, the partial sums of one sequence) is asked for in two rounds
// per BLK columns, the weights first, since they wait for nothing; then everything is summed in a fixed order (the same
// for every BLK).
template <int BLK>                                           // columns per round
__global__ __launch_bounds__(256, BLK > 2048 ? 2 : (BLK > 1024 ? 3 : 5)) void router_mlp_kernel(MlpArgs a) {
  extern __shared__ float pvec[];                           // hidden floats
  constexpr int NW = BLK / 512, NQ = BLK / 1024;             // 16-byte loads of a weight row and of a split's sums per lane
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int b = blockIdx.y;
  // two hidden units per wave, their weight rows streamed together
  const int j0 = blockIdx.x * 8 + w * 2;
  const bool one = j0 < a.inner, two = j0 + 1 < a.inner;
  const __bf16* wrow0 = a.w1 + (int64_t)(one ? j0 : 0) * a.hidden;
  const __bf16* wrow1 = wrow0 + (two ? a.hidden : 0);
  const int n_rows = a.cu[b + 1] - a.cu[b];
  const bool all = a.pool <= 0 || n_rows <= 2 * a.pool;
  const int n_pooled = all ? n_rows : 2 * a.pool;
  const float inv = n_pooled > 0 ? 1.0f / (float)n_pooled : 0.f;
  float acc0 = 0.f, acc1 = 0.f;
  for (int c0 = 0; c0 < a.hidden; c0 += BLK) {
    u32x4 v0[NW], v1[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const int c = c0 + 512 * k + l * 8;
      const int cc = c < a.hidden ? c : 0;                   // (columns past the end are not used)
      v0[k] = *(const u32x4*)(wrow0 + cc);
      v1[k] = *(const u32x4*)(wrow1 + cc);
    }
    // pooled mean: the row-split partial sums are added in split order (fixed, so the result is reproducible); 4
    // columns per thread and 1024, the loads of two or eight splits in flight together
    f32x4 s[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) s[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* p = a.psum + (int64_t)b * a.splits * a.hidden;
    auto add_splits = [&](int sp, auto n) __attribute__((always_inline)) {
      constexpr int N = decltype(n)::value;
      f32x4 v[N][NQ];
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const int c = c0 + 1024 * q + 4 * tid;
          v[i][q] = *(const f32x4*)(p + (int64_t)min(sp + i, a.splits - 1) * a.hidden + (c < a.hidden ? c : 0));
        }
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (sp + i < a.splits) {
#pragma unroll
          for (int q = 0; q < NQ; ++q) s[q] += v[i][q];
        }
    };
    if (a.splits <= 2) add_splits(0, std::integral_constant<int, 2>());
    else
      for (int sp = 0; sp < a.splits; sp += 8) add_splits(sp, std::integral_constant<int, 8>());
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int c = c0 + 1024 * q + 4 * tid;
      if (c < a.hidden) *(f32x4*)(pvec + c) = s[q] * inv;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const int c = c0 + 512 * k + l * 8;
      if (c < a.hidden) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc0 = __builtin_fmaf(bf16_lo(v0[k][i]), pvec[c + 2 * i], acc0);
          acc0 = __builtin_fmaf(bf16_hi(v0[k][i]), pvec[c + 2 * i + 1], acc0);
          acc1 = __builtin_fmaf(bf16_lo(v1[k][i]), pvec[c + 2 * i], acc1);
          acc1 = __builtin_fmaf(bf16_hi(v1[k][i]), pvec[c + 2 * i + 1], acc1);
        }
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    acc0 += __shfl_xor(acc0, off);
    acc1 += __shfl_xor(acc1, off);
  }
  if (one && l < 2 && (l == 0 || two)) {
    float acc = l == 0 ? acc0 : acc1;
    const int j = j0 + l;
    if (a.b1) acc += (float)a.b1[j];
    // (device scope: the workgroup that reads it may sit on another XCD)
    __hip_atomic_store(a.hbuf + (int64_t)b * a.inner + j, acc / (1.0f + expf(-acc)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // SiLU
  }
  if (!a.arrived) return;
  // ---- the workgroup that finishes a sequence's hidden vector runs its head: counted once its own values have been
  // acknowledged at device scope
  __shared__ int is_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) is_last = __hip_atomic_fetch_add(a.arrived + b * a.arrived_stride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  __syncthreads();
  if (is_last && w == 0) {
    if (l == 0) a.arrived[b * a.arrived_stride] = 0;                            // ready for the next call on this stream
    router_head<true>(a.hbuf + (int64_t)b * a.inner, a.w2, a.b2, a.inner, l, a.mode_out + b, a.logits_out ? a.logits_out + 2 * b : nullptr);
  }
}

// The head as a launch of its own (launches of many workgroups).
__global__ __launch_bounds__(64) void router_head_kernel(MlpArgs a) {
  const int b = blockIdx.x;
  router_head<false>(a.hbuf + (int64_t)b * a.inner, a.w2, a.b2, a.inner, threadIdx.x, a.mode_out + b, a.logits_out ? a.logits_out + 2 * b : nullptr);
}

// Columns per round: wide rounds wait for memory fewer times, but take the registers of most of a CU's waves and load what
// lies past the last column for nothing, so they are for wide layers and launches that leave the chip room.  us per call,
// hidden 4096, inner 256, rounds of 4096 / 1024: batch 1 10.8 / 11.7, 8 14.8 / 15.7, 16 22.4 / 22.5, 24 32.2 / 27.1, 64
// 61.9 / 51; hidden 2048, batch 16, rounds of 4096 / 2048 13.9 / 13.4; hidden 256, 512 sequences, 4096 / 1024 35.9 / 21.7;
// hidden 64 6.4 / 5.6.  From there on the head is a launch of its own as well: what every workgroup pays for counting
// itself is more than a launch (hidden 4096, batch 24 27.1 / 24.2, 32 32.5 / 28.8, 64 50.7 / 47.1).
constexpr int kMlpFew = 512;   // workgroups of a launch up to which rounds are as wide as the layer, and the last one runs the head
static_assert(kMlpFew <= kRouterCounters, "a counter per sequence");

hipError_t launch_router(const Ctx& c, const void* x, const int32_t* cu_seqlens, int batch, int hidden, int pool,
                         const void* w1, const void* b1, const void* w2, const void* b2, int inner,
                         uint8_t* mode_out, float* logits_out, hipStream_t s) {
  // row splits: kPoolOnce pooled rows per workgroup when the count is known, 64 splits for whole-sequence
  // pooling, bounded by the scratch region
  int splits = pool > 0 ? (2 * pool + kPoolOnce - 1) / kPoolOnce : 64;
  const size_t per_split = (size_t)batch * hidden * sizeof(float);
  const size_t hbytes = (size_t)batch * inner * sizeof(float);
  size_t room = kSmallBytes - hbytes;
  if ((size_t)splits * per_split > room) splits = (int)(room / per_split);
  if (splits < 1) return hipErrorInvalidValue;              // flux_router has checked the sizes
  float* psum = c.small;
  float* hbuf = c.small + (size_t)splits * batch * hidden;

  PoolArgs pa{(const __bf16*)x, cu_seqlens, hidden, pool, splits, psum};
  if (pool > 0) hipLaunchKernelGGL(router_pool_kernel<16>, dim3((hidden + 127) / 128, splits, batch), dim3(256), 0, s, pa);
  else hipLaunchKernelGGL(router_pool_kernel<64>, dim3((hidden + 511) / 512, splits, batch), dim3(256), 0, s, pa);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;

  MlpArgs ma;
  ma.psum = psum;
  ma.cu = cu_seqlens;
  ma.w1 = (const __bf16*)w1;
  ma.b1 = (const __bf16*)b1;
  ma.w2 = (const __bf16*)w2;
  ma.b2 = (const __bf16*)b2;
  ma.hbuf = hbuf;
  ma.batch = batch;
  ma.hidden = hidden;
  ma.inner = inner;
  ma.pool = pool;
  ma.splits = splits;
  const dim3 grid((inner + 7) / 8, batch);
  const bool few = (long long)grid.x * batch <= kMlpFew;
  ma.arrived = few ? c.router_counters : nullptr;
  // (counts on one line of memory are taken one after the other, some 10 ns each: a line per sequence where they fit)
  ma.arrived_stride = batch <= kRouterLines ? kCounterStride : 1;
  ma.mode_out = mode_out;
  ma.logits_out = logits_out;
  const size_t lds = hidden * sizeof(float);
  if (few && hidden > 2048) hipLaunchKernelGGL(router_mlp_kernel<4096>, grid, dim3(256), lds, s, ma);
  else if (few && hidden > 1024) hipLaunchKernelGGL(router_mlp_kernel<2048>, grid, dim3(256), lds, s, ma);
  else hipLaunchKernelGGL(router_mlp_kernel<1024>, grid, dim3(256), lds, s, ma);
  e = hipGetLastError();
  if (e != hipSuccess) return e;

  if (ma.arrived) return hipSuccess;
  hipLaunchKernelGGL(router_head_kernel, dim3(batch), dim3(64), 0, s, ma);
  return hipGetLastError();
}

}  // namespace flux
