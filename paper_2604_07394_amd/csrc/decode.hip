// flux_attn_decode: split-K streaming attention for one query row per sequence (Eq. 1 / Eq. 2 with
// one query; the decode step of Sec. 3.3 / App. B.3).
//
// Decode is bound by reading the K and V rows of the cache once from HBM.  The work of one
// (sequence, KV head) pair is the VISIBLE key list (FA: all positions; SA: the sinks followed by the
// window tail, so the hidden middle of the cache is never addressed), taken in blocks of 128 keys that
// go round the pair's units.  One 256-thread workgroup is one unit and serves all query heads of the GQA
// group at once, so every K/V row is fetched exactly once per step.
//
// The split is taken ON THE DEVICE from the lengths and mode bytes the call finds there: the chunk
// size (the keys one unit takes) is the one that cuts the visible keys of the whole batch into about
// kTargetUnits workgroups, a pair of nv visible keys gets ceil(nv / chunk) units, and workgroup u finds
// its (sequence, KV head, unit of the pair) by a prefix sum over the batch.  Every
// workgroup with work therefore sits at the front of the grid whatever the mix of lengths and
// modes in the batch, and a ragged batch fills the chip like a uniform one (a grid shaped by the
// longest sequence leaves most workgroups of the short ones empty and the rest badly spread).
//
// Per wave, 32 keys at a time:
//   S^T[key][q]  = K[key][:] . Q[q][:]       4 (D=128) MFMA 16x16x32 bf16 per 16 keys; the A operand
//                                            (8 consecutive d of one key row per lane) is loaded
//                                            straight from global memory, 64 contiguous bytes per row
//                                            and instruction
//   online softmax in the MFMA accumulator layout (one query per lane column, 4 keys per lane)
//   O^T[d][q]   += V^T[d][key] . P^T[key][q] the P operand is the accumulator layout itself; the
//                                            V operand needs keys along the lane's registers, so V
//                                            rows are staged in wave-private LDS and read back with
//                                            the transposing LDS read
// The four waves keep private (m, l, O) and are merged through LDS at the end; the unit's
// unnormalised result goes to the workspace and a second small kernel merges the units of a pair in a fixed
// order (deterministic, no float atomics).
#include "flux_internal.h"

namespace flux {

// What both kernels read to agree on the split.
struct SplitArgs {
  const int32_t* kv_len;
  const uint8_t* mode;
  int batch, capacity;
  int ring;               // != 0: the cache is a sink + ring store of a sparse layer, kv_len is logical, no mode bytes
  int sink_lim, win_blocks, blk_shift;   // SA geometry (see sa_geom)
  int max_keys;           // the host's bound on the keys any sequence attends to
  int pps;                // (KV head, query block) pairs per sequence = hkv * qblocks
  int bump;               // 1: the call also appends one row per sequence, so every list is one key longer than kv_len says
};

struct DecodeArgs {
  const __bf16* q;        // [B, Hq, D]
  const __bf16* k;
  const __bf16* v;
  int64_t stride_b, stride_h, stride_t;   // elements
  SplitArgs sp;
  int hq, hkv, group;     // group = hq / hkv
  int qblocks;            // ceil(group / 16)
  int rpu;                // partial rows per unit = min(group, 16)
  float scale_log2;       // softmax scale * log2(e)
  float* partials;        // per pair [rpu, chunks of the pair, D + 2], pairs in unit order
  int* table;             // [batch][2]: first unit and chunks per pair of every sequence, for the merge kernel
  uint32_t* status;       // sticky device status word
  // the fused decode step only: the row each sequence appends at position kv_len[b], [B, Hkv, D]
  const __bf16* k_new;
  const __bf16* v_new;
  // calls merged in place only (see SMALL below)
  uint32_t* arrived;      // [0]: workgroups that have read the lengths; [1 + pair]: units of a pair that have left their rows
  int32_t* kv_len_rw;
  void* out;
  int out_fp32;
};

// Number of keys the query at position n - 1 attends to.  The visible list is the sinks [0, s_end)
// followed by the window tail [tail_start, n); `sparse` says whether anything lies hidden between them.
__device__ __forceinline__ int visible_len(int n, int md, int sink_lim, int win_blocks, int shift, bool& sparse,
                                           int& s_end, int& tail_start) {
  s_end = n < sink_lim ? n : sink_lim;
  const int lo = n > 0 ? window_start(n - 1, shift, win_blocks) : 0;
  tail_start = lo > s_end ? lo : s_end;
  sparse = ((md & 1) == 0) && (tail_start > s_end);          // bit 0 of md: 1 = FA
  return sparse ? s_end + (n - tail_start) : n;
}

constexpr int kResidentUnits = 768;             // workgroups the chip holds at once: three per CU (at head dimension 64 four would fit; the round is the same)
constexpr int kLongCall = 32768;                // 128-key pieces of all pairs from which a round of two workgroups per CU is no longer better

// Length and mode of sequence b under the clamp: a length the host could not see (negative, or past the
// capacity of a full cache) is cut and reported through `bad`.
// With s.bump the length returned counts the row the call appends, and bit 1 of md says that it does (a full cache
// drops the row).
__device__ __forceinline__ void load_seq(const SplitArgs& s, int b, int& len, int& md, bool& bad) {
  len = s.kv_len[b];
  md = s.ring ? 0 : s.mode[b];
  bad = len < 0 || (!s.ring && len > s.capacity);
  len = len < 0 ? 0 : ((!s.ring && len > s.capacity) ? s.capacity : len);
  md = md != 0 ? 1 : 0;
  if (s.bump && len < s.capacity) {
    ++len;
    md |= 2;
  }
}

// Visible keys of a sequence of `len` rows in mode `md`, cut at the host's bound (reported through `bad`).
__device__ __forceinline__ int seq_visible(const SplitArgs& s, int len, int md, bool& bad, bool& sparse, int& s_end,
                                           int& tail_start) {
  int nv = visible_len(len, md, s.sink_lim, s.win_blocks, s.blk_shift, sparse, s_end, tail_start);
  if (nv > s.max_keys) {
    bad = true;
    nv = s.max_keys;
  }
  return nv;
}

// The split of one call, as every wave of both kernels computes it from the lengths and mode bytes.
struct Split {
  int chunk;        // keys per unit: the visible keys of all pairs, counted in 128-key pieces, divided over
                    // kTargetUnits (at least kMinChunk); the units then number at most kTargetUnits + batch * pps
  int b;            // the sequence found (-1: the unit lies past the last one)
  int first_unit;   // first unit of that sequence
  int nc;           // its chunks per (KV head, query block) pair
  int len, md;      // its clamped length and mode
  bool any_bad;     // this lane saw a clamp trip
  unsigned long long empty;   // (calls merged in place) sequences without keys
};

// chunks that a list of `pieces` takes at `c` pieces each
__device__ __forceinline__ int chunks_of(int pieces, int c, float inv_c) { return pieces > 0 ? div_small(pieces - 1, c, inv_c) + 1 : 0; }

// Find the sequence whose units contain `unit`.
// Lane i of the wave looks after sequences i, i + 64, ...; a batch of up to 64 takes one load per lane.
__device__ __forceinline__ Split find_split(const SplitArgs& s, int lane, int unit) {
  Split r;
  r.b = -1;
  r.first_unit = r.nc = r.len = 0;
  r.md = 1;
  r.any_bad = false;
  r.empty = 0;
  bool sparse;
  int s_end, tail_start;
  int len0 = 0, md0 = 1, pc0 = 0;                          // block 0 stays in registers for the second pass
  int pieces = 0;
  for (int b0 = 0; b0 < s.batch; b0 += 64) {
    int len = 0, md = 1, nv = 0;
    if (b0 + lane < s.batch) {
      bool bad;
      load_seq(s, b0 + lane, len, md, bad);
      nv = seq_visible(s, len, md, bad, sparse, s_end, tail_start);
      r.any_bad |= bad;
    }
    const int pc = (nv + 127) >> 7;
    if (b0 == 0) {
      len0 = len;
      md0 = md;
      pc0 = pc;
    }
    pieces += __builtin_amdgcn_readlane(wave_inclusive_sum(pc), 63);
  }
  const long long total = (long long)pieces * s.pps;
  const long long c128 = (total + (kTargetUnits - 1)) / kTargetUnits;
  int c = c128 < kMinChunk / 128 ? kMinChunk / 128 : (int)c128;
  // If a larger chunk cuts the batch into one nearly full round of workgroups, it is taken: a single round of equal
  // workgroups pays the start and the merge of a workgroup once instead of twice.  Uniform batches do; a ragged one usually
  // spills a few units into a second round, and a short list (a sparse layer) leaves much of the round empty: both keep
  // the smaller chunk.  A round of 512 (two per CU) is better than one of 768 (all that fit) while the lists are short
  // (1 x 32768 keys 29.6 against 33.1 us, 1 x 131072 84.7 / 89.3, 8 x 32768 168.7 / 169.3; 8 x 131072 665 / 656).
  if (s.batch <= 64) {
    auto round_of = [&](int slots, int least) __attribute__((always_inline)) {
      const int big = max((int)((float)total * (1.0f / (float)slots)) + 1, kMinChunk / 128);
      const int units = __builtin_amdgcn_readlane(wave_inclusive_sum(s.pps * chunks_of(pc0, big, 1.0f / (float)big)), 63);
      return units <= slots && units > least ? big : 0;
    };
    const int two = total < kLongCall ? round_of(512, 512 - 512 / 20) : 0;
    const int big = two > 0 ? two : round_of(kResidentUnits, kResidentUnits - kResidentUnits / 10);
    if (big > 0) c = big;
  }
  r.chunk = 128 * c;
  const float inv_c = 1.0f / (float)c;

  for (int b0 = 0, base = 0; b0 < s.batch; b0 += 64) {
    int len = len0, md = md0, pc = pc0;
    if (b0 > 0) {
      len = 0, md = 1, pc = 0;
      if (b0 + lane < s.batch) {
        bool bad;
        load_seq(s, b0 + lane, len, md, bad);
        pc = (seq_visible(s, len, md, bad, sparse, s_end, tail_start) + 127) >> 7;
      }
    }
    const int nc = chunks_of(pc, c, inv_c);
    const int incl = wave_inclusive_sum(s.pps * nc);        // units up to and including this lane's sequence
    const int total_b = __builtin_amdgcn_readlane(incl, 63);
    if (unit < base + total_b) {                            // wave-uniform
      const int sidx = __builtin_amdgcn_readfirstlane(__builtin_popcountll(__builtin_amdgcn_ballot_w64(base + incl <= unit)));
      r.b = b0 + sidx;
      r.first_unit = base + (sidx > 0 ? __builtin_amdgcn_readlane(incl, sidx - 1) : 0);
      r.nc = __builtin_amdgcn_readlane(nc, sidx);
      r.len = __builtin_amdgcn_readlane(len, sidx);
      r.md = __builtin_amdgcn_readlane(md, sidx);
      break;
    }
    base += total_b;
  }
  return r;
}

// The split of a call merged in place: a lane per sequence, always the smallest chunk.
__device__ __forceinline__ Split find_split_small(const SplitArgs& s, int lane, int unit) {
  Split r;
  bool sparse, bad = false;
  int s_end, tail_start, len = 0, md = 1, nv = 0;
  if (lane < s.batch) {
    load_seq(s, lane, len, md, bad);
    nv = seq_visible(s, len, md, bad, sparse, s_end, tail_start);
  }
  r.any_bad = bad;
  r.empty = __builtin_amdgcn_ballot_w64(lane < s.batch && nv == 0);
  r.chunk = kMinChunk;
  const int nc = (nv + kMinChunk - 1) / kMinChunk;
  const int incl = wave_inclusive_sum(s.pps * nc);
  const int total = __builtin_amdgcn_readlane(incl, 63);
  r.b = -1;
  r.first_unit = r.nc = r.len = 0;
  r.md = 1;
  if (unit < total) {                                       // wave-uniform
    r.b = __builtin_amdgcn_readfirstlane(__builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= unit)));
    r.nc = __builtin_amdgcn_readlane(nc, r.b);
    r.first_unit = __builtin_amdgcn_readlane(incl, r.b) - s.pps * r.nc;
    r.len = __builtin_amdgcn_readlane(len, r.b);
    r.md = __builtin_amdgcn_readlane(md, r.b);
  }
  return r;
}

// The split as a table, for the merge kernel: entry b = (first unit, chunks per pair) of sequence b.  One wave writes
// it (lane i looks after sequences i, i + 64, ...), with the same arithmetic as find_split.
__device__ __forceinline__ void write_split_table(const SplitArgs& s, int lane, int chunk, int* table) {
  bool sparse, bad;
  int s_end, tail_start;
  for (int b0 = 0, base = 0; b0 < s.batch; b0 += 64) {
    int len = 0, md = 1, nv = 0;
    if (b0 + lane < s.batch) {
      load_seq(s, b0 + lane, len, md, bad);
      nv = seq_visible(s, len, md, bad, sparse, s_end, tail_start);
    }
    const int nc = chunks_of((nv + 127) >> 7, chunk >> 7, 1.0f / (float)(chunk >> 7));
    const int incl = wave_inclusive_sum(s.pps * nc);
    if (b0 + lane < s.batch) {
      table[2 * (b0 + lane)] = base + incl - s.pps * nc;
      table[2 * (b0 + lane) + 1] = nc;
    }
    base += __builtin_amdgcn_readlane(incl, 63);
  }
}

// Merge every STEP-th chunk, from `first` on, of one column of a head's rows [chunk][D + 2]: num = sum_c w_c O_c[d],
// den = sum_c w_c l_c with w_c = exp(m_c - m), m = max m_c.  N chunks at a time, so that their loads are in flight
// together.  DEV: the rows were written by workgroups of this launch (device-scope reads).
struct Merged {
  float m, num, den;
};
template <int D, bool DEV, int STEP, int N>
__device__ __forceinline__ Merged merge_rows(const float* base, int nc, float scale_log2, int d, int first) {
  constexpr int RED = D + 2;
  auto ld = [](const float* p) { return DEV ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p; };
  Merged r = {-INFINITY, 0.f, 0.f};
  for (int c0 = first; c0 < nc; c0 += N * STEP) {
    float mc[N], lc[N], oc[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const float* row = base + (int64_t)min(c0 + u * STEP, nc - 1) * RED;  // (the last chunk again where there are fewer)
      mc[u] = ld(row + D);
      lc[u] = ld(row + D + 1);
      oc[u] = ld(row + d);
    }
    float m_new = r.m;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      mc[u] = c0 + u * STEP < nc ? mc[u] : -INFINITY;
      m_new = fmaxf(m_new, mc[u]);
    }
    const float al = fast_exp2((r.m - m_new) * scale_log2);                 // 0 for the first chunks (each holds a key)
    r.num *= al;
    r.den *= al;
    r.m = m_new;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const float w = fast_exp2((mc[u] - m_new) * scale_log2);
      r.num += w * oc[u];
      r.den += w * lc[u];
    }
  }
  return r;
}

// FUSED: the call is a whole decode step of the layer (Sec. 3.3): it also appends the row k_new / v_new of every
// sequence at position kv_len[b].  The unit that owns the end of a list stores the row in the cache; the units that
// attend to it take it from k_new / v_new, so no read waits for that store.  The lengths are moved on by the merge
// kernel, after every workgroup of both kernels has read them.  Two launches instead of three.
//
// SMALL: a call of few short lists (see decode_small), which is bound by latencies and not by bytes: one launch instead
// of two.  Eight waves per workgroup, so that each has one block of 32 keys and no second wait for memory; the unit that
// arrives last at its pair merges the pair's rows.  The rows pass between workgroups that may sit on different XCDs:
// they are written and read with device-scope accesses (past the L2s, which are not coherent with each other), and a
// unit counts itself only after its own stores have been acknowledged.  ROWS: the same eight waves and chunks, but the rows
// are left for the merge kernel, as in the two-launch form: for callers without arrival counters (the static scratch).
// The merge takes the same sums in the same order, so the results are those of the one-launch form bit for bit.
// Three workgroups per CU are asked for: left alone the compiler keeps the accumulators in a second register file (192
// registers, two workgroups per CU) although 160 do: SA layer of 8 x 131072 32.6 -> 31.1 us, 32 ragged sequences of 513 to
// 8400 keys at 28/4 heads 44.5 -> 39.7 us.  (Very long calls stream at the rate of the memory with two as well, up to 1 %
// faster, but the host cannot tell them from short lists under a large bound, which lose 10 %: with a bound of 65536 the
// 32 ragged sequences take 38.0 us, 41.9 with two; 8 x 131072 651.7 and 650.5.)
template <int D, bool NT, bool FUSED, bool SMALL = false, bool ROWS = false>
__global__ __launch_bounds__(SMALL ? 512 : 256, SMALL ? 2 : 3) void decode_splitk_kernel(DecodeArgs a) {
  constexpr int W = SMALL ? 8 : 4;    // waves per workgroup
  constexpr bool IN_PLACE = SMALL && !ROWS;   // the unit that arrives last merges its pair
  constexpr int KC = D / 32;          // MFMA k-steps over the head dimension
  constexpr int DB = D / 16;          // 16-wide output blocks over the head dimension
  constexpr int VL = D / 16;          // 16-byte V loads per lane per 32-key block
  constexpr int CPR = D / 8;          // 16-byte chunks per row
  constexpr int VROW = D + 8;         // padded LDS row (elements)
  constexpr int RED = D + 2;

  __shared__ __attribute__((aligned(16))) char smem[W * 32 * VROW * 2];

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int g = l >> 4, n = l & 15;
  const int unit = blockIdx.x;

  // ---- the split: chunk size from the whole batch, then the sequence whose units contain `unit`
  const Split sp = SMALL ? find_split_small(a.sp, l, unit) : find_split(a.sp, l, unit);
  if (unit == 0 && w == 0 && sp.any_bad) atomicOr(a.status, (uint32_t)FLUX_DEV_BAD_LENGTH);
  // SMALL and FUSED: every workgroup counts itself once all its waves hold the lengths; the one that finds all others
  // counted moves the lengths on, when it has nothing else to do (nobody reads them any more).
  uint32_t order = 0;
  if constexpr (SMALL && FUSED) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) order = __hip_atomic_fetch_add(a.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  auto finish = [&]() __attribute__((always_inline)) {
    if constexpr (SMALL && FUSED) {
      if (w == 0 && __builtin_amdgcn_readfirstlane(order) == gridDim.x - 1) {
        if (l < a.sp.batch) {
          int len = a.kv_len_rw[l];
          len = len < 0 ? 0 : (len > a.sp.capacity ? a.sp.capacity : len);
          a.kv_len_rw[l] = len < a.sp.capacity ? len + 1 : len;
        }
        if (l == 0) a.arrived[0] = 0;                       // ready for the next call on this stream
      }
    }
  };
  // the last workgroup of the grid (idle unless the host's bound on the units is met exactly) leaves the split
  // behind for the merge kernel, which then needs neither the lengths nor the scan
  if (!IN_PLACE && unit == (int)gridDim.x - 1 && w == 0) write_split_table(a.sp, l, sp.chunk, a.table);
  if (IN_PLACE && unit == (int)gridDim.x - 1) {             // sequences without keys have no units: their rows are zero
    for (unsigned long long left = sp.empty; left != 0; left &= left - 1) {
      const int64_t off = (int64_t)__builtin_ctzll(left) * a.hq * D;
      for (int i = tid; i < a.hq * D; i += 64 * W) {
        if (a.out_fp32) ((float*)a.out)[off + i] = 0.f;
        else ((__bf16*)a.out)[off + i] = (__bf16)0.f;
      }
    }
  }
  if (sp.b < 0) {                                           // past the last unit: uniform for the whole workgroup
    finish();
    return;
  }
  const int b = sp.b;
  const int local = unit - sp.first_unit;                   // < pps * nc, chunk index fastest
  const float inv_nc = 1.0f / (float)sp.nc;
  const int pair = __builtin_amdgcn_readfirstlane(div_small(local, sp.nc, inv_nc));
  const int ci = local - pair * sp.nc;
  const int kvh = a.qblocks == 1 ? pair : pair / a.qblocks;
  const int qb = a.qblocks == 1 ? 0 : pair % a.qblocks;

  bool bad_b = false, sparse;
  int s_end, tail_start;
  const int n_vis = seq_visible(a.sp, sp.len, sp.md, bad_b, sparse, s_end, tail_start);
  // The chunk size fixes how many units a pair has (sp.nc); the pair's 128-key blocks then go round its units: unit ci
  // takes the blocks ci, ci + nc, ci + 2 nc, ...  Every unit of a pair gets the same number of blocks to within one
  // (chunks of consecutive keys leave the last unit of every pair a remainder, which costs a ragged batch a tenth of
  // its time), and the units of a pair, which run side by side, read one moving window of consecutive rows.
  const int c0 = ci * 128;
  const int c1 = n_vis;
  const int pstep = 128 * sp.nc;
  const int tail0 = tail_start - s_end;                     // list index p >= s_end maps to key p + tail0
  // ring store (s_end = sink_lim when sparse): that key sits in row sink_lim + (p + tail0 - sink_lim) % ring_window
  //                                                               = sink_lim + (p - sink_lim + ring0) % ring_window
  const int ring_window = a.sp.win_blocks << a.sp.blk_shift;
  const int ring0 = (a.sp.ring && sparse) ? tail0 % ring_window : 0;

  const __bf16* kbase = a.k + (int64_t)b * a.stride_b + (int64_t)kvh * a.stride_h;
  const __bf16* vbase = a.v + (int64_t)b * a.stride_b + (int64_t)kvh * a.stride_h;

  // FUSED: the appended row is position sp.len - 1, the last key of every list (none when the cache was full).
  int new_key = -1;
  const __bf16* knew = nullptr;
  const __bf16* vnew = nullptr;
  if constexpr (FUSED) {
    if (sp.md & 2) {                                         // the sequence takes its row
      new_key = sp.len - 1;
      knew = a.k_new + ((int64_t)b * a.hkv + kvh) * D;
      vnew = a.v_new + ((int64_t)b * a.hkv + kvh) * D;
      const int last_piece = (n_vis - 1) >> 7;
      if (ci == last_piece - div_small(last_piece, sp.nc, inv_nc) * sp.nc && qb == 0 && tid < 2 * CPR) {   // this unit owns the list's last block: it stores the row
        const int c = tid % CPR;
        const __bf16* src = (tid < CPR ? knew : vnew) + 8 * c;
        __bf16* dst = const_cast<__bf16*>(tid < CPR ? kbase : vbase) + (int64_t)new_key * a.stride_t + 8 * c;
        *(u32x4*)dst = *(const u32x4*)src;
      }
    } else if (ci == 0 && pair == 0 && tid == 0) {
      atomicOr(a.status, (uint32_t)FLUX_DEV_KV_OVERFLOW);
    }
  }

  // ---- Q operand: lane (n, g) holds d = 32*kc + 8*g .. +7 of query head kvh*group + 16*qb + n
  const int qh = 16 * qb + n;
  bf16x8 qf[KC];
  {
    const u32x4 zero = {0, 0, 0, 0};
    const __bf16* qrow = a.q + ((int64_t)b * a.hq + (int64_t)kvh * a.group + (qh < a.group ? qh : 0)) * D;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      u32x4 t = *(const u32x4*)(qrow + 32 * kc + 8 * g);
      qf[kc] = __builtin_bit_cast(bf16x8, qh < a.group ? t : zero);
    }
  }

  auto key_of = [&](int p) -> int64_t {
    p = p < c1 ? p : c1 - 1;                                // keep every address inside the list
    if (!sparse || p < s_end) return (int64_t)p;
    if (!a.sp.ring) return (int64_t)p + tail0;
    const int x = p - s_end + ring0;                        // < 2 * ring_window
    return (int64_t)s_end + (x >= ring_window ? x - ring_window : x);
  };

  // A 32-key block whose keys are 32 consecutive cache rows (every block of an FA chunk, and all but the
  // few SA blocks that contain the sink / tail seam, the ring wrap or the end of the list) is addressed as
  // a wave-uniform row pointer plus per-lane offsets fixed for the whole kernel: no per-lane multiplies.
  // The lane's offset is the same for every load of a block (one register for K, one for V); what differs between
  // the loads, 16 rows per K half and 64 / CPR rows per V load, is added to the uniform row pointer.
  constexpr int RPL = 64 / CPR;                             // V rows per wave-wide load
  const int k_lane = n * (int)a.stride_t + 8 * g;           // element offsets inside a block of consecutive rows
  const int v_lane = (l / CPR) * (int)a.stride_t + (l % CPR) * 8;

  // Rows that are read once and evicted before the next step (the launcher decides by the bytes of the call) are
  // fetched with nontemporal loads (NT), which measurably raise the streaming rate of this access shape
  // (6.2 -> 7.1 TB/s in isolation).
  auto ld = [](const u32x4* p) -> u32x4 { return NT ? __builtin_nontemporal_load(p) : *p; };
  u32x4 kreg[2][KC], vreg[VL];
  auto load_block = [&](int p0) {                           // p0 is wave-uniform
    const int64_t r0 = key_of(p0);
    // (FUSED: the block that holds the appended row takes the per-lane path, where that row comes from k_new / v_new)
    const bool linear = p0 + 32 <= c1 && key_of(p0 + 31) - r0 == 31 && !(FUSED && new_key >= 0 && r0 + 31 >= new_key);
    if (linear) {
      const __bf16* kb0 = kbase + r0 * a.stride_t;
      const __bf16* vb0 = vbase + r0 * a.stride_t;
#pragma unroll
      for (int sb = 0; sb < 2; ++sb)
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) kreg[sb][kc] = ld((const u32x4*)(kb0 + 16 * sb * a.stride_t + k_lane + 32 * kc));
#pragma unroll
      for (int i = 0; i < VL; ++i) vreg[i] = ld((const u32x4*)(vb0 + i * RPL * a.stride_t + v_lane));
    } else {
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        const int64_t key = key_of(p0 + 16 * sb + n);
        const __bf16* row = (FUSED && key == new_key) ? knew : kbase + key * a.stride_t;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) kreg[sb][kc] = ld((const u32x4*)(row + 32 * kc + 8 * g));
      }
#pragma unroll
      for (int i = 0; i < VL; ++i) {
        const int e = i * 64 + l;
        const int64_t key = key_of(p0 + e / CPR);
        const __bf16* row = (FUSED && key == new_key) ? vnew : vbase + key * a.stride_t;
        vreg[i] = ld((const u32x4*)(row + (e % CPR) * 8));
      }
    }
  };

  FLUX_LDS __bf16* vs = (FLUX_LDS __bf16*)smem + w * 32 * VROW;

  float m_run = -INFINITY, l_run = 0.f;
  f32x4 o[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};

  // (eight waves: the upper four take every other block of the unit)
  int p0 = c0 + (SMALL ? (w >> 2) * pstep : 0) + 32 * (w & 3);
  if (p0 < c1) load_block(p0);
  while (p0 < c1) {
    // ---- stage this block's V rows in LDS and take K into MFMA operands
#pragma unroll
    for (int i = 0; i < VL; ++i) {
      const int e = i * 64 + l;
      *(FLUX_LDS u32x4*)(vs + (e / CPR) * VROW + (e % CPR) * 8) = vreg[i];
    }
    bf16x8 kf[2][KC];
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) kf[sb][kc] = __builtin_bit_cast(bf16x8, kreg[sb][kc]);
    const int pnext = p0 + (SMALL ? 2 * pstep : pstep);
    // ---- scores: s[sb][i] is key p0 + 16*sb + 4*g + i against query n
    f32x4 s[2];
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
      s[sb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < KC; ++kc)
        s[sb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[sb][kc], qf[kc], s[sb], 0, 0, 0);
    }
    // the next block is asked for once the score MFMAs have taken this block's K registers, which the loads then
    // reuse (asked for before them, the block in flight needs registers of its own: 30 more per lane)
    __builtin_amdgcn_sched_barrier(0);
    if (pnext < c1) load_block(pnext);
    __builtin_amdgcn_sched_barrier(0);
    if (p0 + 32 > c1) {
#pragma unroll
      for (int sb = 0; sb < 2; ++sb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (p0 + 16 * sb + 4 * g + i >= c1) s[sb][i] = -INFINITY;
    }
    // ---- online softmax (row maximum over the 4 lane groups of this query)
    float mloc = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                       fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
    mloc = fmaxf(mloc, __shfl_xor(mloc, 16));
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
    const float m_new = fmaxf(m_run, mloc);                 // finite: the block holds a valid key
    const float alpha = fast_exp2((m_run - m_new) * a.scale_log2);
    const float mneg = -m_new * a.scale_log2;
    m_run = m_new;
    uint32_t pk[4];
    float psum = 0.f;
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
      const float p0f = fast_exp2(__builtin_fmaf(s[sb][0], a.scale_log2, mneg));
      const float p1f = fast_exp2(__builtin_fmaf(s[sb][1], a.scale_log2, mneg));
      const float p2f = fast_exp2(__builtin_fmaf(s[sb][2], a.scale_log2, mneg));
      const float p3f = fast_exp2(__builtin_fmaf(s[sb][3], a.scale_log2, mneg));
      pk[2 * sb] = pack_bf16(p0f, p1f);
      pk[2 * sb + 1] = pack_bf16(p2f, p3f);
      // the denominator sums the same rounded weights the numerator uses
      psum += (bf16_lo(pk[2 * sb]) + bf16_hi(pk[2 * sb])) + (bf16_lo(pk[2 * sb + 1]) + bf16_hi(pk[2 * sb + 1]));
    }
    l_run = l_run * alpha + psum;
    const bf16x8 pf = __builtin_bit_cast(bf16x8, u32x4{pk[0], pk[1], pk[2], pk[3]});
    // ---- O^T += V^T P^T
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      o[db] *= alpha;
      FLUX_LDS __bf16* src = vs + (4 * g + (n >> 2)) * VROW + 16 * db + 4 * (n & 3);
      const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((FLUX_LDS bf16x4*)src);
      const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((FLUX_LDS bf16x4*)(src + 16 * VROW));
      const bf16x8 vf = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
      o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o[db], 0, 0, 0);
    }
    p0 = pnext;
  }

  auto store_out = [&](int qi, int d, float r) __attribute__((always_inline)) {
    const int64_t off = ((int64_t)b * a.hq + (int64_t)kvh * a.group + 16 * qb + qi) * D + d;
    if (a.out_fp32) ((float*)a.out)[off] = r;
    else ((__bf16*)a.out)[off] = (__bf16)r;
  };
  // ---- merge the waves through LDS: red[w][n][0..D-1] = O, [D] = m, [D+1] = l
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  __syncthreads();                                          // every wave is done with its V staging
  FLUX_LDS float* red = (FLUX_LDS float*)smem;
  static_assert(W * 16 * RED * 4 <= W * 32 * VROW * 2, "merge buffer must fit the staging buffer");
  {
    FLUX_LDS float* mine = red + (w * 16 + n) * RED;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) mine[16 * db + 4 * g + i] = o[db][i];
    if (g == 0) {
      mine[D] = m_run;
      mine[D + 1] = l_run;
    }
  }
  __syncthreads();
  const int nq = min(16, a.group - 16 * qb);
  if (IN_PLACE && sp.nc == 1) {                             // the only unit of its pair: nothing to merge with
    for (int idx = tid; idx < nq * D; idx += 64 * W) {
      const int qi = idx / D, d = idx % D;
      float m = -INFINITY, num = 0.f, den = 0.f;
#pragma unroll
      for (int ww = 0; ww < W; ++ww) m = fmaxf(m, red[(ww * 16 + qi) * RED + D]);
#pragma unroll
      for (int ww = 0; ww < W; ++ww) {
        const float wgt = fast_exp2((red[(ww * 16 + qi) * RED + D] - m) * a.scale_log2);
        num += wgt * red[(ww * 16 + qi) * RED + d];
        den += wgt * red[(ww * 16 + qi) * RED + D + 1];
      }
      store_out(qi, d, num / den);
    }
    finish();
    return;
  }
  for (int idx = tid; idx < nq * RED; idx += 64 * W) {
    const int qi = idx / RED, e = idx % RED;
    float mw[W], m = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < W; ++ww) {
      mw[ww] = red[(ww * 16 + qi) * RED + D];
      m = fmaxf(m, mw[ww]);
    }
    float val;
    if (e == D) {
      val = m;
    } else {
      val = 0.f;
#pragma unroll
      for (int ww = 0; ww < W; ++ww) {
        const float wgt = fast_exp2((mw[ww] - m) * a.scale_log2);   // exp2(-inf) = 0 for idle waves
        val += wgt * red[(ww * 16 + qi) * RED + e];                 // e == D+1 merges l the same way
      }
    }
    // the units of one pair are consecutive: inside their block the rows run [query head][chunk], so that the merge
    // reads one head's chunks as one contiguous run
    float* dst = a.partials + (((int64_t)(unit - ci) * a.rpu) + (int64_t)qi * sp.nc + ci) * RED + e;
    if constexpr (IN_PLACE) __hip_atomic_store(dst, val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *dst = val;
  }
  if constexpr (IN_PLACE) {
    // ---- the unit that arrives last merges the pair
    __shared__ int last_of_pair;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // this wave's rows have reached the point all XCDs see
    __syncthreads();
    uint32_t* count = a.arrived + 1 + b * a.sp.pps + pair;
    if (tid == 0) last_of_pair = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(sp.nc - 1);
    __syncthreads();
    if (last_of_pair) {
      if (tid == 0) *count = 0;                             // ready for the next call on this stream
      const float* rows = a.partials + (int64_t)(unit - ci) * a.rpu * RED;
      for (int idx = tid; idx < nq * D; idx += 64 * W) {
        const int qi = idx / D, d = idx % D;
        const Merged r = merge_rows<D, true, 1, 8>(rows + (int64_t)qi * sp.nc * RED, sp.nc, a.scale_log2, d, 0);
        store_out(qi, d, r.num / r.den);
      }
    }
    finish();
  }
}

// Merge the chunks of one (sequence, query head): out = sum_c w_c O_c / sum_c w_c l_c,
// w_c = exp(m_c - max m), chunks taken in index order.
struct CombineArgs {
  const float* partials;
  const int* table;       // the split the first kernel took: [batch][2] = first unit, chunks per pair
  int hq, group, qblocks, rpu, out_fp32;
  float scale_log2;
  void* out;
  // the fused decode step only (bump = 1): the lengths, which this kernel moves on.  Nothing reads them any more
  // at that point: the first kernel has ended and this one takes the split from the table.
  int bump, capacity;
  int32_t* kv_len_rw;
};

// G groups of D threads per (sequence, query head), each with every G-th chunk; the partial results meet in LDS.
// Bound by latencies (the split table, then the rows): all rows of up to 8 G chunks are asked for at once (with maximum,
// weights and sums as three dependent passes over the rows a layer took 0.9 - 1.3 us longer).  One group is enough where
// a list has few chunks, and four times the threads cost 0.7 us where there are a thousand heads to merge.
template <int D, int G>
__global__ __launch_bounds__(G * D) void decode_combine_kernel(CombineArgs a) {
  constexpr int RED = D + 2;
  const int tid = threadIdx.x, d = tid % D, grp = tid / D, head = blockIdx.x, b = blockIdx.y;
  const int first_unit = a.table[2 * b], nc = a.table[2 * b + 1];
  const int kvh = head / a.group, hh = head - kvh * a.group;
  const int64_t unit0 = first_unit + (int64_t)(kvh * a.qblocks + hh / 16) * nc;
  const float* base = a.partials + (unit0 * a.rpu + (int64_t)(hh % 16) * nc) * RED;
  Merged r = merge_rows<D, false, G, 8>(base, nc, a.scale_log2, d, grp);
  if constexpr (G > 1) {
    __shared__ Merged part[G][D];
    part[grp][d] = r;
    __syncthreads();
    r = {-INFINITY, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < G; ++i) r.m = fmaxf(r.m, part[i][d].m);
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const float w = fast_exp2((part[i][d].m - r.m) * a.scale_log2);       // exp2(-inf) = 0 for a group without chunks
      r.num += w * part[i][d].num;
      r.den += w * part[i][d].den;
    }
  }
  if (grp == 0) {
    const float x = nc > 0 ? r.num / r.den : 0.f;                           // an empty cache yields zeros
    const int64_t off = ((int64_t)b * a.hq + head) * D + d;
    if (a.out_fp32) ((float*)a.out)[off] = x;
    else ((__bf16*)a.out)[off] = (__bf16)x;
  }
  if (a.bump && head == 0 && tid == 0) {
    int len = a.kv_len_rw[b];
    len = len < 0 ? 0 : (len > a.capacity ? a.capacity : len);
    a.kv_len_rw[b] = len < a.capacity ? len + 1 : len;
  }
}

// c.small_counters may be null: a call of few short lists then takes two launches.
hipError_t launch_decode(const Ctx& c, const flux_attn_cfg& cfg, const void* q, int max_kv_len,
                         const flux_kv_cache& cache, const uint8_t* mode, int ring, const void* k_new,
                         const void* v_new, void* out, hipStream_t s) {
  const bool fused = k_new != nullptr;                       // append + attend + merge in one launch
  const DecodePlan plan = plan_decode(cfg, cache.batch, max_kv_len);
  const float scale = cfg.softmax_scale != 0.f ? cfg.softmax_scale : 1.0f / sqrtf((float)cfg.head_dim);
  DecodeArgs a;
  a.q = (const __bf16*)q;
  a.k = (const __bf16*)cache.k;
  a.v = (const __bf16*)cache.v;
  a.stride_b = cache.stride_b;
  a.stride_h = cache.stride_h;
  a.stride_t = cache.stride_t;
  const SaGeom geom = sa_geom(cfg);
  a.sp.kv_len = cache.kv_len;
  a.sp.mode = mode;
  a.sp.batch = cache.batch;
  a.sp.capacity = cache.capacity;
  a.sp.ring = ring;
  a.sp.sink_lim = geom.sink_lim;
  a.sp.win_blocks = geom.win_blocks;
  a.sp.blk_shift = geom.shift;
  a.sp.max_keys = max_kv_len;
  a.sp.pps = plan.pps;
  a.sp.bump = fused ? 1 : 0;
  a.k_new = (const __bf16*)k_new;
  a.v_new = (const __bf16*)v_new;
  a.hq = cfg.n_q_heads;
  a.hkv = cfg.n_kv_heads;
  a.group = cfg.n_q_heads / cfg.n_kv_heads;
  a.qblocks = (a.group + 15) / 16;
  a.rpu = plan.rpu;
  a.scale_log2 = scale * kLog2e;
  a.table = (int*)c.partials;                                // the split table sits in front of the partial rows
  a.partials = c.partials + plan.table_floats;
  a.status = c.status;
  const dim3 grid(plan.units);
  // K and V bytes one call may read.  A call of a model whose layers together stream more than the 256 MB last-level
  // cache finds none of its rows there, whatever its own size (an SA layer reads 138 MB of a 4 GB cache): from 64 MB
  // on the rows are fetched with nontemporal loads (SA layer 34.5 -> 33.4 us, FA layers as before); smaller calls are
  // bound by their launches either way.
  const bool nt = 4.0 * cache.batch * cfg.n_kv_heads * cfg.head_dim * (double)max_kv_len > 64.0 * 1024 * 1024;
  a.arrived = c.small_counters;
  a.kv_len_rw = cache.kv_len;
  a.out = out;
  a.out_fp32 = cfg.out_dtype;
  const bool small = decode_small(cfg, cache.batch, max_kv_len) && (c.small_counters || !fused);
  if (small && c.small_counters) {
    if (cfg.head_dim == 128) {
      if (fused) hipLaunchKernelGGL((decode_splitk_kernel<128, false, true, true>), grid, dim3(512), 0, s, a);
      else hipLaunchKernelGGL((decode_splitk_kernel<128, false, false, true>), grid, dim3(512), 0, s, a);
    } else {
      if (fused) hipLaunchKernelGGL((decode_splitk_kernel<64, false, true, true>), grid, dim3(512), 0, s, a);
      else hipLaunchKernelGGL((decode_splitk_kernel<64, false, false, true>), grid, dim3(512), 0, s, a);
    }
    return hipGetLastError();
  }
  auto launch = [&](auto d, auto f) {
    constexpr int D = decltype(d)::value;
    constexpr bool FU = decltype(f)::value;
    if (small) {
      if constexpr (!FU) hipLaunchKernelGGL((decode_splitk_kernel<D, false, false, true, true>), grid, dim3(512), 0, s, a);
    } else if (nt) hipLaunchKernelGGL((decode_splitk_kernel<D, true, FU>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((decode_splitk_kernel<D, false, FU>), grid, dim3(256), 0, s, a);
  };
  if (cfg.head_dim == 128) {
    if (fused) launch(std::integral_constant<int, 128>(), std::true_type());
    else launch(std::integral_constant<int, 128>(), std::false_type());
  } else {
    if (fused) launch(std::integral_constant<int, 64>(), std::true_type());
    else launch(std::integral_constant<int, 64>(), std::false_type());
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;

  CombineArgs ca;
  ca.partials = a.partials;
  ca.table = a.table;
  ca.hq = cfg.n_q_heads;
  ca.group = a.group;
  ca.qblocks = a.qblocks;
  ca.rpu = plan.rpu;
  ca.out_fp32 = cfg.out_dtype;
  ca.scale_log2 = a.scale_log2;
  ca.out = out;
  ca.bump = a.sp.bump;
  ca.capacity = cache.capacity;
  ca.kv_len_rw = cache.kv_len;
  const dim3 cgrid(cfg.n_q_heads, cache.batch);
  // chunks of the longest list, as far as the host can tell: the bound, or about twice a pair's share of the units
  const long long pairs = (long long)cache.batch * plan.pps;
  const bool few = small || max_kv_len <= 8 * kMinChunk || 2 * kTargetUnits <= 8 * pairs;
  if (cfg.head_dim == 128) {
    if (few) hipLaunchKernelGGL((decode_combine_kernel<128, 1>), cgrid, dim3(128), 0, s, ca);
    else hipLaunchKernelGGL((decode_combine_kernel<128, 4>), cgrid, dim3(512), 0, s, ca);
  } else {
    if (few) hipLaunchKernelGGL((decode_combine_kernel<64, 1>), cgrid, dim3(64), 0, s, ca);
    else hipLaunchKernelGGL((decode_combine_kernel<64, 4>), cgrid, dim3(256), 0, s, ca);
  }
  return hipGetLastError();
}

}  // namespace flux
