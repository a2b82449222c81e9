// flux_kv_append: copy new K/V rows to the tail of each sequence's cache, then bump the lengths.
// flux_kv_append_ring / flux_kv_compact_ring: the same copy into the sink + ring layout a sparse layer
// keeps for decode (Sec. 3.3): position p sits in row p for p < n_sink, else in row
// n_sink + (p - n_sink) % window.
//
// One launch.  Every workgroup reads the old lengths, copies its share of 16-byte chunks, and the
// workgroup that finishes last (arrival counter) writes the new lengths, so no copy can observe a
// bumped length.  Pure HBM copy: 16 bytes per lane per access, rows are contiguous on both sides.
#include "flux_internal.h"

namespace flux {

struct AppendArgs {
  const u32x4* k_new;
  const u32x4* v_new;
  const int32_t* cu_new;
  u32x4* kc;
  u32x4* vc;
  int64_t stride_b, stride_h, stride_t;   // in 16-byte chunks
  int32_t* kv_len;
  int batch, capacity, hkv, cpr_shift;     // 1 << cpr_shift chunks per row
  int total_new;
  int ring, n_sink, window;                // ring != 0: sink + ring rows, lengths are logical
  uint32_t* counter;                       // workgroups (or words of `gather` whose workgroups) that have arrived
  uint32_t* gather;                        // kAppendGather words that workgroups count themselves on
  uint32_t* status;
};

constexpr int kAppendTable = 1024;          // sequences whose lengths fit the table in LDS

// The thread that calls counts its workgroup; true for the last one of the launch.
template <bool ONE>
__device__ __forceinline__ bool count_arrival(const AppendArgs& a) {
  const uint32_t n = gridDim.x;
  if (!ONE) {
    const uint32_t x = blockIdx.x & (kAppendGather - 1);
    uint32_t* word = a.gather + x * kCounterStride;
    if (atomicAdd(word, 1u) != (n - x + kAppendGather - 1) / kAppendGather - 1) return false;
    *word = 0;                                               // ready for the next launch on this stream
  }
  return atomicAdd(a.counter, 1u) == (ONE ? n : kAppendGather) - 1;
}

__device__ __forceinline__ int length_after(const AppendArgs& a, int len, int n) {
  len += n > 0 ? n : 0;
  return !a.ring && len > a.capacity ? a.capacity : len;
}

// Where token row t goes, of a sequence of length len0 whose n new rows begin with `first`; -1: nowhere.
__device__ __forceinline__ int64_t row_place(const AppendArgs& a, int b, int len0, int first, int n, int t) {
  const int pos = len0 + (t - first);
  int row = pos;
  bool keep = pos >= 0 && pos < a.capacity;
  if (a.ring) {
    // only rows that are still resident after the whole call are written: the sinks and the last
    // `window` positions (an earlier row of this call may share a ring row with a later one)
    keep = pos >= 0 && (pos < a.n_sink || pos >= len0 + n - a.window);
    row = pos < a.n_sink ? pos : a.n_sink + (pos - a.n_sink) % a.window;
  }
  return keep ? (int64_t)b * a.stride_b + (int64_t)row * a.stride_t : -1;
}

// What bounds it: the copy where there is much to copy, else latencies.  Workgroups that count themselves on one word do
// so one after the other, some 10 ns each, which 512 of them waited 5 us for; so each counts itself on one of 16 words, and
// who completes a word on the last one (up to 64 workgroups the second step takes longer than it saves).  With that a token
// row per thread and as many workgroups as that takes are fastest up to 4096 of them.  Longer copies keep four rows per
// thread in flight and read the lengths into LDS once, where a row's sequence is looked up.  (Batches up to 64 are
// copied by kv_append_few_kernel below.)  us on one word with at most
// 256 such workgroups, and 512 of four rows / now, 8 KV heads of 128: 256 tokens 4.9 / 4.2, 512 6.4 / 4.4, 1195 tokens of 4
// sequences 7.6 / 5.8, 2000 9.3 / 6.9, 6466 of 5 17.0 / 14.5, 8192 20.0 / 15.8 (4.3 TB/s), 600 of one token 8.4 / 6.0; 16384
// 32.5 and 32768 56 (4.8 TB/s) as before.
// U: token rows a thread has in flight (with one, lengths are looked up in global memory); ONE: the workgroups count
// themselves on one word
template <int U, bool ONE>
__global__ __launch_bounds__(256) void kv_append_kernel(AppendArgs a) {
  __shared__ int is_last;
  __shared__ int s_cu[kAppendTable + 1], s_len[kAppendTable];
  const int cpt = a.hkv << a.cpr_shift;                      // 16-byte chunks per token
  const int lanes = cpt < 256 ? cpt : 256;                   // threads that share one token
  const int tpi = 256 / lanes;                               // tokens per workgroup iteration and row in flight
  const int tid = threadIdx.x;
  const int trow = tid / lanes, c0 = tid - trow * lanes;
  const bool table = U > 1 && a.batch <= kAppendTable;
  if (table) {
    for (int i = tid; i <= a.batch; i += 256) {
      s_cu[i] = a.cu_new[i];
      if (i < a.batch) s_len[i] = a.kv_len[i];
    }
    __syncthreads();
  }
  auto cu = [&](int i) { return table ? s_cu[i] : a.cu_new[i]; };
  bool overflow = false;
  if (trow < tpi) {
    for (int64_t t0 = (int64_t)blockIdx.x * tpi * U + trow; t0 < a.total_new; t0 += (int64_t)gridDim.x * tpi * U) {
      int64_t dst0[U];                                       // where the row goes, -1: nowhere
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t tt = t0 + u * tpi;
        dst0[u] = -1;
        if (tt >= a.total_new) continue;
        const int t = (int)tt;
        // sequence of token row t: largest b with cu_new[b] <= t
        int lo = 0, hi = a.batch;
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (cu(mid) <= t) lo = mid; else hi = mid;
        }
        const int len0 = table ? s_len[lo] : a.kv_len[lo];
        dst0[u] = row_place(a, lo, len0, cu(lo), a.ring ? cu(lo + 1) - cu(lo) : 0, t);
        overflow |= dst0[u] < 0 && !a.ring;
      }
      for (int c = c0; c < cpt; c += lanes) {
        const int h = c >> a.cpr_shift, cc = c - (h << a.cpr_shift);
        const int64_t off = (int64_t)h * a.stride_h + cc;
        // ordinary loads and stores: the appended rows are read again at once by the attention call
        // that follows (nontemporal accesses measured 10 % slower here)
        u32x4 k[U], v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (dst0[u] >= 0) {
            const int64_t src = (t0 + u * tpi) * cpt + c;
            k[u] = a.k_new[src];
            v[u] = a.v_new[src];
          }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (dst0[u] >= 0) {
            a.kc[dst0[u] + off] = k[u];
            a.vc[dst0[u] + off] = v[u];
          }
      }
    }
  }
  if (overflow) atomicOr(a.status, (uint32_t)FLUX_DEV_KV_OVERFLOW);

  // The last workgroup to arrive bumps the lengths.  The others only READ kv_len, and a thread's loads
  // have returned (waited for here) before the barrier lets thread 0 count the arrival, so no
  // fence is needed for this read-before-write order.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) is_last = count_arrival<ONE>(a);
  __syncthreads();
  if (is_last) {
    for (int b = tid; b < a.batch; b += blockDim.x) {
      a.kv_len[b] = length_after(a, a.kv_len[b], a.cu_new[b + 1] - a.cu_new[b]);
    }
    if (tid == 0) *a.counter = 0;   // ready for the next launch on this stream
  }
}

// Up to 64 sequences: one token row per thread, a single pass, as many workgroups as that takes (kAppendMost at most).  What
// bounds it: short copies memory latencies one behind the other, long ones the memory (6.1 TB/s at 32768 tokens, read and
// written).  The general kernel waits for the lengths, the new rows, the acknowledgement of the stores, the arrival count and the lengths once more.  Here every wave
// asks for the lengths, a sequence per lane, and right behind them for the new rows, whose place in the input does not depend on
// them; a row's sequence is looked up in the registers, the stores are not waited for, and the last workgroup holds the
// lengths already.  Nothing is shared by the workgroup, so new ones start while others drain, which workgroups that stay for several rows
// do not make up for by having four in flight.  us with the general kernel / now: 16 tokens
// 3.8 / 3.4, 256 4.25 / 3.8, 1000 4.95 / 4.5, 2000 6.0 / 5.4, 6466 tokens of 5 sequences 13.0 / 11.2, 8192 13.5 / 12.1, 16384
// 25.4 / 23.1, 32768 47.6 / 44.3, 65536 107 / 97, 32 x 2048 109 / 95 (8 KV heads of 128), one token of 16 rings (4 heads) 4.3 /
// 3.65.  In the general kernel's body the same changes cost its long copies 3 %, so these have a kernel of their own.
// LATE: the new rows are asked for when their place is known, and only those that have one (ring appends that drop rows, see
// plan_append).
template <bool ONE, bool LATE>
__global__ __launch_bounds__(256) void kv_append_few_kernel(AppendArgs a) {
  const int cpt = a.hkv << a.cpr_shift;
  const int lanes = cpt < 256 ? cpt : 256;
  const int tpi = 256 / lanes;
  const int tid = threadIdx.x;
  const int trow = tid / lanes, c0 = tid - trow * lanes;
  const uint32_t at = blockIdx.x * (uint32_t)tpi + trow;      // (below 2^31 + 256, and the launch below 2^30 threads)
  const int t = (int)at;
  const bool valid = trow < tpi && at < (uint32_t)a.total_new;
  const int own = min(tid & 63, a.batch - 1);                // the sequence whose lengths this lane holds
  const int my_cu = a.cu_new[own], my_end = a.cu_new[own + 1], my_len = a.kv_len[own];
  __builtin_amdgcn_sched_barrier(0);
  u32x4 k = {0, 0, 0, 0}, v = {0, 0, 0, 0};
  if (!LATE && valid) {
    k = a.k_new[(int64_t)t * cpt + c0];
    v = a.v_new[(int64_t)t * cpt + c0];
  }
  __builtin_amdgcn_sched_barrier(0);
  const int my_n = my_end - my_cu;
  int b = 0;                                                 // largest b with cu_new[b] <= t (all lanes take part)
  for (int step = a.batch > 1 ? 1 << (31 - __builtin_clz(a.batch - 1)) : 0; step > 0; step >>= 1) {
    const int first = __shfl(my_cu, b + step);
    if (b + step < a.batch && first <= t) b += step;
  }
  const int len0 = __shfl(my_len, b), first = __shfl(my_cu, b), n = __shfl(my_n, b);
  if (valid) {
    const int64_t dst = row_place(a, b, len0, first, n, t);
    if (dst < 0 && !a.ring) atomicOr(a.status, (uint32_t)FLUX_DEV_KV_OVERFLOW);
    for (int c = c0; c < cpt && dst >= 0; c += lanes) {
      const int h = c >> a.cpr_shift;
      const int64_t off = dst + (int64_t)h * a.stride_h + (c - (h << a.cpr_shift));
      if (LATE || c != c0) {
        k = a.k_new[(int64_t)t * cpt + c];
        v = a.v_new[(int64_t)t * cpt + c];
      }
      a.kc[off] = k;
      a.vc[off] = v;
    }
  }
  // as above: a wave has its lengths before its thread passes the barrier, and only then is the workgroup counted
  asm volatile("" : : "v"(my_len), "v"(my_n) : "memory");
  __syncthreads();
  if (tid >= 64) return;
  const int last = tid == 0 && count_arrival<ONE>(a) ? 1 : 0;
  if (__builtin_amdgcn_readfirstlane(last) == 0) return;
  if (tid < a.batch) a.kv_len[tid] = length_after(a, my_len, my_n);
  if (tid == 0) *a.counter = 0;
}

hipError_t launch_kv_append(const Ctx& c, const flux_kv_cache& cache, int hkv, int d, const void* k_new,
                            const void* v_new, const int32_t* cu_new, int total_new, int max_new, int ring, int n_sink,
                            int window, hipStream_t s) {
  AppendArgs a;
  a.k_new = (const u32x4*)k_new;
  a.v_new = (const u32x4*)v_new;
  a.cu_new = cu_new;
  a.kc = (u32x4*)cache.k;
  a.vc = (u32x4*)cache.v;
  a.stride_b = cache.stride_b / 8;
  a.stride_h = cache.stride_h / 8;
  a.stride_t = cache.stride_t / 8;
  a.kv_len = cache.kv_len;
  a.batch = cache.batch;
  a.capacity = cache.capacity;
  a.hkv = hkv;
  a.cpr_shift = d == 128 ? 4 : 3;
  a.total_new = total_new;
  a.ring = ring;
  a.n_sink = n_sink;
  a.window = window;
  a.counter = c.counters + 0;
  a.gather = c.append_counters;
  a.status = c.status;
  const AppendPlan p = plan_append(cache.batch, hkv, d, total_new, max_new, ring, window);
  const dim3 grid(p.wgs), block(256);
  if (p.form == kAppendWide) hipLaunchKernelGGL((kv_append_kernel<kAppendTokens, false>), grid, block, 0, s, a);
  else if (p.form == kAppendSingle && p.one_word) hipLaunchKernelGGL((kv_append_kernel<1, true>), grid, block, 0, s, a);
  else if (p.form == kAppendSingle) hipLaunchKernelGGL((kv_append_kernel<1, false>), grid, block, 0, s, a);
  else if (p.form == kAppendEarly && p.one_word) hipLaunchKernelGGL((kv_append_few_kernel<true, false>), grid, block, 0, s, a);
  else if (p.form == kAppendEarly) hipLaunchKernelGGL((kv_append_few_kernel<false, false>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((kv_append_few_kernel<false, true>), grid, block, 0, s, a);
  return hipGetLastError();
}

// ---- compaction of a full cache into a ring cache: list entry p of sequence b (p < n_sink: sink p;
// else the (p - n_sink)-th position of the window tail) is copied to its ring row.
struct CompactArgs {
  const u32x4* ks;
  const u32x4* vs;
  int64_t s_stride_b, s_stride_h, s_stride_t;   // in 16-byte chunks
  const int32_t* s_len;
  int s_capacity;
  u32x4* kd;
  u32x4* vd;
  int64_t d_stride_b, d_stride_h, d_stride_t;
  int32_t* d_len;
  int batch, hkv, chunks_per_row, n_sink, window;
};

__global__ __launch_bounds__(256) void kv_compact_ring_kernel(CompactArgs a) {
  const int cpt = a.hkv * a.chunks_per_row;                  // 16-byte chunks per position
  const int lanes = cpt < 256 ? cpt : 256;
  const int tpi = 256 / lanes;
  const int tid = threadIdx.x;
  const int c0 = tid % lanes, trow = tid / lanes;
  const int b = blockIdx.y;
  int len = a.s_len[b];
  len = len < 0 ? 0 : (len > a.s_capacity ? a.s_capacity : len);
  const int n_keep = len < a.n_sink + a.window ? len : a.n_sink + a.window;
  const int tail0 = len - a.window - a.n_sink;               // list entry p >= n_sink is position p + tail0 (if len is longer than the ring)
  if (trow < tpi) {
    for (int p = blockIdx.x * tpi + trow; p < n_keep; p += gridDim.x * tpi) {
      const int pos = (p < a.n_sink || tail0 <= 0) ? p : p + tail0;
      const int row = pos < a.n_sink ? pos : a.n_sink + (pos - a.n_sink) % a.window;
      const int64_t src0 = (int64_t)b * a.s_stride_b + (int64_t)pos * a.s_stride_t;
      const int64_t dst0 = (int64_t)b * a.d_stride_b + (int64_t)row * a.d_stride_t;
      for (int c = c0; c < cpt; c += lanes) {
        const int h = c / a.chunks_per_row, cc = c - h * a.chunks_per_row;
        a.kd[dst0 + (int64_t)h * a.d_stride_h + cc] = a.ks[src0 + (int64_t)h * a.s_stride_h + cc];
        a.vd[dst0 + (int64_t)h * a.d_stride_h + cc] = a.vs[src0 + (int64_t)h * a.s_stride_h + cc];
      }
    }
  }
  if (blockIdx.x == 0 && tid == 0) a.d_len[b] = len;
}

hipError_t launch_kv_compact_ring(const flux_kv_cache& src, const flux_kv_cache& dst, int hkv, int d, int n_sink,
                                  int window, hipStream_t s) {
  CompactArgs a;
  a.ks = (const u32x4*)src.k;
  a.vs = (const u32x4*)src.v;
  a.s_stride_b = src.stride_b / 8;
  a.s_stride_h = src.stride_h / 8;
  a.s_stride_t = src.stride_t / 8;
  a.s_len = src.kv_len;
  a.s_capacity = src.capacity;
  a.kd = (u32x4*)dst.k;
  a.vd = (u32x4*)dst.v;
  a.d_stride_b = dst.stride_b / 8;
  a.d_stride_h = dst.stride_h / 8;
  a.d_stride_t = dst.stride_t / 8;
  a.d_len = dst.kv_len;
  a.batch = src.batch;
  a.hkv = hkv;
  a.chunks_per_row = d / 8;
  a.n_sink = n_sink;
  a.window = window;
  const int cpt = hkv * (d / 8);
  const int tpi = 256 / (cpt < 256 ? cpt : 256);
  long long blocks = ((long long)n_sink + window + tpi - 1) / tpi;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(kv_compact_ring_kernel, dim3((unsigned)blocks, src.batch), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace flux
