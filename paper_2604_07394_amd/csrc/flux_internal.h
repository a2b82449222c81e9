// Internal declarations shared by the translation units of libflux (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/flux.h"

// The host-only build that checks the C ABI under sanitizers compiles flux_api.hip as plain C++ (no device pass):
// there the few device-side spellings it meets are given host meanings.
#ifndef __HIP__
#ifndef __device__
#define __device__
#endif
#ifndef __align__
#define __align__(n) __attribute__((aligned(n)))
#endif
#ifndef HIP_SYMBOL
#define HIP_SYMBOL(x) x
#endif
#endif

namespace flux {

// ---- vector types for MFMA operands and packed memory access --------------------------------
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;

#define FLUX_LDS __attribute__((address_space(3)))
#define FLUX_GLOBAL __attribute__((address_space(1)))
#define FLUX_CONSTANT __attribute__((address_space(4)))

constexpr float kLog2e = 1.4426950408889634f;

// The context: a device workspace carved into fixed regions.
struct Ctx {
  int device;              // < 0: no device (argument checking only)
  char* ws;                // device workspace base (256-byte aligned)
  size_t ws_bytes;         // as given: the counters that have lines of their own come on top
  // carved regions (device pointers)
  uint32_t* status;        // sticky status word
  uint32_t* counters;      // kCounters zero-initialised arrival counters; users reset them to zero
  uint32_t* append_counters;  // kAppendGather of the same kind, kCounterStride apart
  uint32_t* decode_counters;  // kDecodeCounters of the same kind; null: decode calls take two launches
  uint32_t* router_counters;  // kRouterCounters of the same kind, one per sequence of a router call
  float* small;            // router scratch: pooled vectors and hidden activations
  float* partials;         // split-K partial results
  size_t partials_bytes;
};

// The SA visible set in block units (App. C.3): positions are grouped into blocks of 2^shift; the sinks
// are the positions below sink_lim (whole blocks), the window of query position i starts at
// window_start(i).  shift = 0 is the token-exact rule: sink_lim = n_sink, window_start(i) = i - window + 1.
struct SaGeom {
  int shift, sink_lim, win_blocks;
};
inline SaGeom sa_geom(const flux_attn_cfg& cfg) {
  int b = cfg.sa_block > 1 ? cfg.sa_block : 1, sh = 0;
  while ((1 << sh) < b) ++sh;
  SaGeom g;
  g.shift = sh;
  // rounded up in 64 bits and cut at the largest int: n_sink or window near INT32_MAX ("SA sees everything",
  // Eq. 2 degenerating to Eq. 1) must not wrap.  Positions are below INT32_MAX, so the cut changes nothing.
  const long long sink_lim = (((long long)cfg.n_sink + b - 1) >> sh) << sh;
  const long long win_blocks = ((long long)cfg.window + b - 1) >> sh;
  g.sink_lim = sink_lim > 0x7FFFFFFFll ? 0x7FFFFFFF : (int)sink_lim;
  g.win_blocks = win_blocks > (0x7FFFFFFFll >> sh) ? (0x7FFFFFFF >> sh) : (int)win_blocks;
  return g;
}
#ifdef __HIP__   // device helpers: absent from the host-only build that checks the C ABI under sanitizers
__device__ __forceinline__ int window_start(int i, int shift, int win_blocks) {
  const int lo = ((i >> shift) - win_blocks + 1) << shift;
  return lo > 0 ? lo : 0;
}
#endif

constexpr int kCounters = 64;
constexpr int kRouterCounters = 512;
constexpr int kRouterLines = 24;              // router calls of at most so many sequences have each counter on a line of its own
// Arrival counters of the decode calls, each on a line of its own (counts on one line are taken one after the other, some
// 10 ns each): words whose workgroups have all read the lengths; the words that workgroups count themselves on; one per
// workgroup, for the pair that begins in its range and goes on behind it.
constexpr int kCounterStride = 32;            // words
constexpr int kDecodeGather = 32;
constexpr int kDecodeOneWord = 128;           // workgroups of eight waves up to which all count themselves on the first word
constexpr int kDecodeWgsShift = 8, kDecodeAlignedShift = 9;
constexpr int kDecodeCounters = 1 + kDecodeGather + (1 << kDecodeAlignedShift);
constexpr int kAppendGather = 16;             // words that the workgroups of an append count themselves on, each on a line of its own
constexpr size_t kSmallBytes = 8u << 20;      // router: batch * (splits * hidden + inner) floats; decode: the rows of parts
constexpr size_t kHeaderBytes = 4096;         // status + counters
// The counters that have lines of their own lie between the header and the router scratch, and are not taken from the bytes
// that the caller gives a context: a workspace of a given size holds the partials that it held before there were any.
constexpr size_t kDecodeCountersAt = kHeaderBytes;   // bytes
constexpr size_t kAppendCountersAt = kDecodeCountersAt + kDecodeCounters * kCounterStride * 4;
constexpr size_t kCountersBytes = (kAppendCountersAt + kAppendGather * kCounterStride * 4 - kHeaderBytes + 4095) / 4096 * 4096;

// What launches an append (see the kernels in kv_append.hip).
enum AppendForm {
  kAppendEarly,    // up to kAppendLanes sequences: a token row per thread, asked for before its place is known
  kAppendLate,     // the same, asked for when its place is known, and if it has one
  kAppendSingle,   // a token row per thread, lengths looked up in memory
  kAppendWide,     // kAppendTokens rows per thread in flight, lengths looked up in LDS, workgroups that stay
};
struct AppendPlan {
  AppendForm form;
  unsigned wgs;
  bool one_word;   // all workgroups count themselves on one word
};
constexpr int kAppendLanes = 64;
constexpr int kAppendTokens = 4;
constexpr int kAppendFew = 4096;
constexpr int kAppendResident = 2048;       // workgroups that the chip holds at once
constexpr int kAppendMost = 1 << 22;        // workgroups of a launch with a row per thread (from 2^24 on it would be refused: 2^32 threads)
constexpr unsigned kAppendOneWord = 64;     // workgroups up to which all count themselves on one word
static_assert(kAppendResident >= (int)kAppendOneWord, "kAppendLate counts on several words");
static_assert(kAppendOneWord >= kAppendGather && 512 / kAppendTokens > kAppendOneWord, "every word of a launch that counts on several is used");
// Up to 64 sequences take one pass of as many workgroups as there are rows (see kv_append_few_kernel), up to kAppendMost.  More of them:
// one token row per thread up to 4096 workgroups (us with four and the table / with one: 1195 tokens 6.9 / 5.8, 6466 15.0 /
// 14.5, 32 x 200 15.0 / 14.5).  Many sequences take longer to look up in global memory, so there the table serves from 512
// on.  Four rows per thread: 1024 workgroups where that is one or two rounds (8192 tokens of 128 to 1024 sequences), 512 for more (32768
// tokens 56.0, with 1024 56.7).
// A ring append of more workgroups than the chip holds at once does not ask for the rows that it drops (128 + 4096 keys of 8 heads of 128
// stay of 131072 rows: 105 to 109 us with every row read, 52 to 54 as here); a smaller one waits for latencies, and all its rows are on
// their way together (us as kAppendEarly / kAppendLate, 64 + 2048 rows of 8 heads of 128 stay: 3000 rows 5.8 / 6.2, 4096 6.35 / 6.65,
// 5000 6.8 / 7.0, 6000 7.55 / 7.3, 8192 9.15 / 8.55; 64 + 64 stay: 2000 rows 4.6 / 4.7, 4096 5.5 / 5.4, 8192 7.7 / 7.4).
// Workgroups that only find that their rows are dropped cost less than looking up the sequence of a row, which one or two sequences
// have little need of, and which shows where they are many (us as kAppendWide / kAppendLate: 8192 rows 8.8 / 8.3, 14000 9.3 / 10.7,
// 32768 17.6 / 19.0, 2 x 60000 58.6 / 57.9 to 61.3, 3 x 40000 65 / 60 to 63, 8 x 8000 52 / 42 to 45, 64 x 5000 326 / 255 to 262).
inline AppendPlan plan_append(int batch, int hkv, int d, int total_new, int max_new, int ring, int window) {
  const int cpt = hkv * (d / 8), tpi = 256 / (cpt < 256 ? cpt : 256);
  const long long single = ((long long)total_new + tpi - 1) / tpi;
  AppendPlan p;
  const bool late = ring && max_new > window && single > kAppendResident;
  if (batch <= kAppendLanes && single <= kAppendMost && !(late && batch <= 2 && single > kAppendFew)) {
    p.form = late ? kAppendLate : kAppendEarly;
    p.wgs = (unsigned)single;
  } else if (single <= (batch <= 128 ? kAppendFew : 512)) {
    p.form = kAppendSingle;
    p.wgs = (unsigned)single;
  } else {
    const long long blocks = (single + kAppendTokens - 1) / kAppendTokens, most = blocks < 2048 ? 1024 : 512;
    p.form = kAppendWide;
    p.wgs = (unsigned)(blocks < most ? blocks : most);
  }
  p.one_word = p.form != kAppendWide && p.wgs <= kAppendOneWord;
  return p;
}

// ---- launchers (each validates nothing: flux_api.hip has done it) ---------------------------
hipError_t launch_kv_append(const Ctx& c, const flux_kv_cache& cache, int hkv, int d, const void* k_new,
                            const void* v_new, const int32_t* cu_new, int total_new, int max_new, int ring, int n_sink,
                            int window, hipStream_t s);
hipError_t launch_kv_compact_ring(const flux_kv_cache& src, const flux_kv_cache& dst, int hkv, int d, int n_sink,
                                  int window, hipStream_t s);

// Decode shares the visible keys of a call out over 2^kDecodeWgsShift workgroups, one per CU, in equal ranges (two per CU
// where there are many lists); calls of at most 2^kDecodeAlignedShift times 128 keys take one workgroup per 128 keys of a
// list, and few keys eight waves per workgroup.  The cut itself is taken on the device; the host only bounds it.  A CU takes in about 27 bytes per ns from memory, whatever its workgroups have asked for, which is
// its even share of what the memory delivers: a call takes as long as the CU with the most keys.  (Units of whole chunks of a
// list left the fullest CU 18 % over the mean in a batch of 32 ragged lists and 44 % in 16 lists of 2112 keys, and the third
// workgroup of a CU, whose lengths are asked for behind the others' keys, began to stream when those were done.)  Two
// workgroups per CU take no more in, start later and leave twice the rows to merge: us with two / one, 32/8 heads of 128,
// weights of one bf16 term: 8 x 4224 keys 29.7 / 28.1, 1 x 100000 69.8 / 65.0, 8 x 131072 652.5 / 644.9, 32 ragged lists of
// 28/4 heads 37.4 / 36.8 (one, with two terms: 29.4, 37.9 for the first and the last).
struct DecodePlan {
  int units;        // what the scratch is sized by: the units of a cut into chunks of kMinChunk keys and more
  int pps;          // (KV head, query block) pairs per sequence
  int rpu;          // partial rows of a unit
  int table_floats; // two 4-byte words per sequence (rounded to 256 B), which the documented size of the scratch counts
  int table_words;  // calls of two launches: words in front of the rows that hold the cut as a table (rounded to 256 B)
  int wgs;          // workgroups launched
  int waves;        // of a workgroup
  int most_by_four; // calls of eight waves: workgroups up to which merged lists are taken by 128 keys
  int aligned_shift;   // log2 of the most where every one takes its keys from one list; < 0: never
  int block_shift;  // log2 of the keys of a block
  bool in_partials; // the rows of parts need the partials region (they fit the small one otherwise)
};
// Calls that two workgroups per CU can hold at 256 keys each are bound by latencies and take eight waves per workgroup, so that
// each has one block of 32 keys and no second wait for memory (us with four / eight, 32/8 heads of 128 unless said: 3 lists of
// 144 keys 8.8 / 7.0, 8 of 100 7.5 / 6.4, 5 of 61 to 210 at head dimension 64 7.4 / 5.9, 16 of 250 at 16/8 heads 9.8 / 8.6, 1 x
// 8000 13.8 / 12.6; with at most 256 workgroups / 512: 5 of 420 to 6881 at 8/2 heads of 64 20.0 / 18.1 for two layers).  Where
// lists are merged they take 128 keys each while that leaves at most 1024 rows, as a CU takes in its keys no faster than its
// even share (256 / 128 keys: 1 x 2001 9.8 / 8.5, 11 lists of 66 to 503 38.3 / 34.7 for four layers, 16 of 49 to 710 at 28/4
// heads 39.6 / 35.0; with eight rows and more per list there is more to merge than to win: 2 lists of 16 heads 11.1 / 12.4).
constexpr int kDecodeFewWgs = 512;
constexpr int kDecodeFewRows = 1024;
constexpr int kTargetUnits = 1024;
constexpr int kMinChunk = 256;
inline DecodePlan plan_decode(const flux_attn_cfg& cfg, int batch, int max_kv_len) {
  DecodePlan p;
  const int group = cfg.n_q_heads / cfg.n_kv_heads;
  p.pps = cfg.n_kv_heads * ((group + 15) / 16);
  p.rpu = group < 16 ? group : 16;
  const long long pairs = (long long)batch * p.pps, keys = max_kv_len > 0 ? max_kv_len : 1;
  const long long by_len = pairs * ((keys + kMinChunk - 1) / kMinChunk);
  const long long by_target = kTargetUnits + pairs;
  p.units = (int)(by_len < by_target ? by_len : by_target);
  if (p.units < 1) p.units = 1;
  p.table_floats = (2 * batch + 63) / 64 * 64;
  p.table_words = (2 * batch + 5 + 63) / 64 * 64;            // (two per sequence and five behind them, see write_cut_table)
  // a range leaves rows in two places at most (see part_place); never fewer workgroups than share the keys out otherwise
  static_assert(kDecodeAlignedShift > kDecodeWgsShift, "halved below");
  const long long by_four = pairs * ((keys + 127) / 128);
  auto bytes = [&](long long wgs) { return 2 * wgs * p.rpu * (cfg.head_dim + 2) * (long long)sizeof(float); };
  p.aligned_shift = kDecodeAlignedShift;
  p.wgs = (int)(by_four < (1 << p.aligned_shift) ? by_four : (1 << p.aligned_shift));
  const long long by_eight = pairs * ((keys + 255) / 256);
  p.waves = 4;
  p.most_by_four = kDecodeFewRows / p.rpu < kDecodeFewWgs ? kDecodeFewRows / p.rpu : kDecodeFewWgs;
  const long long few = by_eight > p.most_by_four ? by_eight : (by_four < p.most_by_four ? by_four : p.most_by_four);
  if (few <= kDecodeFewWgs && bytes(few) <= (long long)kSmallBytes) {
    p.waves = 8;
    p.wgs = (int)few;
  }
  p.in_partials = false;
  if (bytes(p.wgs) > (long long)kSmallBytes) {
    if (2ll * p.wgs <= p.units) {
      p.in_partials = true;
    } else {
      --p.aligned_shift;
      p.wgs = 1 << p.aligned_shift;
    }
  }
  // blocks are counted in 32 bits: where the bounds allow more of them, they are larger; and in calls of very many lists they
  // are counted as they are (a list may be counted as up to 15 blocks more otherwise)
  const bool rounded = pairs <= 1 << 20;
  if (!rounded) p.aligned_shift = -1;
  p.block_shift = 5;
  while (pairs * ((keys >> p.block_shift) + (rounded ? 16 : 1)) > 0x7FFFFFFFll && p.block_shift < 30) ++p.block_shift;
  return p;
}
inline size_t decode_partials_bytes(const flux_attn_cfg& cfg, const DecodePlan& p) {
  return ((size_t)p.table_floats + (size_t)p.units * p.rpu * (cfg.head_dim + 2)) * sizeof(float);
}
// Where the rows of parts begin in the partials, in floats: behind the table, which only calls of two launches leave there.
// (A call of one launch that keeps its rows there takes at most `units` of them, all that decode_partials_bytes counts.)
inline size_t decode_rows_at(const DecodePlan& p, bool two_launches) { return two_launches ? p.table_words : 0; }
// Bytes of the static scratch that a call takes: the documented size, and what the table and the rows of parts take.
inline size_t decode_static_bytes(const flux_attn_cfg& cfg, const DecodePlan& p) {
  const size_t said = decode_partials_bytes(cfg, p);
  const size_t used = (decode_rows_at(p, true) + (size_t)2 * p.wgs * p.rpu * (cfg.head_dim + 2)) * sizeof(float);
  return said > used ? said : used;
}
// k_new / v_new != nullptr: the fused decode step (append one row per sequence, then attend: one launch instead of
// two); needs c.decode_counters and a cache that is not a ring.
hipError_t launch_decode(const Ctx& c, const flux_attn_cfg& cfg, const void* q, int max_kv_len,
                         const flux_kv_cache& cache, const uint8_t* mode, int ring, const void* k_new,
                         const void* v_new, void* out, hipStream_t s);

// Keep flags of the block-sparse prefill: [batch, heads, n_qblocks, n_kblocks] bytes, heads = 1 or n_q_heads.
struct BlockMask {
  const uint8_t* flags;
  int heads, n_qblocks, n_kblocks;
};
hipError_t launch_prefill(const Ctx& c, const flux_attn_cfg& cfg, const void* q, const int32_t* cu_q,
                          int max_q_len, int max_kv_len, const flux_kv_cache& cache, const uint8_t* mode,
                          const BlockMask* bm /*nullptr: the sink + window form*/, void* out, hipStream_t s);

// XA block selection: LDS of one workgroup (partial tiles + the masses of 8 query blocks), and the launcher
constexpr int kXaMaxKBlocks = 4096;           // key blocks a prompt may have (262144 positions): the masses live in LDS
constexpr int kXaSingleWalkMaxKBlocks = 1024; // up to here the (square row, key block) table of one workgroup fits LDS (144 KB)
inline size_t xa_select_lds_bytes(int n_kblocks) {
  const size_t table = n_kblocks <= kXaSingleWalkMaxKBlocks ? (size_t)32 * n_kblocks : (size_t)8 * n_kblocks;
  return (size_t)2 * 4 * 512 * 4 + table * 4;
}
hipError_t launch_xa_select(const Ctx& c, const flux_attn_cfg& cfg, const void* q, const int32_t* cu_q, int max_q_len,
                            const flux_kv_cache& cache, float threshold, uint8_t* mask, int n_qblocks, int n_kblocks,
                            hipStream_t s);

hipError_t launch_router(const Ctx& c, const void* x, const int32_t* cu_seqlens, int batch, int hidden, int pool,
                         const void* w1, const void* b1, const void* w2, const void* b2, int inner,
                         uint8_t* mode_out, float* logits_out, hipStream_t s);

// ---- small device helpers -------------------------------------------------------------------
#ifdef __HIP__
__device__ __forceinline__ float bf16_bits_to_float(uint32_t bits16) {
  return __builtin_bit_cast(float, bits16 << 16);
}
__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __builtin_bit_cast(float, packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __builtin_bit_cast(float, packed & 0xFFFF0000u); }

// two fp32 -> packed bf16 pair (round to nearest even), low half = a
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  bf16x2 r;
  r[0] = (__bf16)a;
  r[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, r);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max over the two half-waves: lane l and lane l^32 end up with the same value
__device__ __forceinline__ float max_across_halves(float x) {
  uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ float sum_across_halves(float x) {
  uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

// Inclusive prefix sum over the 64 lanes with data-parallel-primitive moves (add within rows of 16 by
// shifts of 1, 2, 4, 8, then carry lane 15 of each row into the next row and lane 31 into the upper half);
// lanes without a source keep the 0 passed as the old value.  Lane 63 ends up with the total.
__device__ __forceinline__ int wave_inclusive_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

// Quotients of small numbers (below 2^24) through a reciprocal, put right by one step.
__device__ __forceinline__ int div_small(int x, int y, float inv_y) {
  int q = (int)((float)x * inv_y);
  q += (q + 1) * y <= x ? 1 : (q * y > x ? -1 : 0);
  return q;
}

// One wave-wide direct global -> LDS transfer: every lane fetches its own 16 bytes, the 64 pieces land
// at lds_base + 16 * lane.  Issued as inline assembly so that the compiler does not serialise later LDS
// reads of the OTHER stage behind it; completion is awaited explicitly with vmcnt(0) before the barrier.
// M0 (the LDS base of the transfer) is written here and declared as clobbered.
__device__ __forceinline__ void lds_copy16(const char* base /*uniform*/, int lane_off, uint32_t lds_base /*uniform*/) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_off), "s"(base), "s"(lds_base) : "memory", "m0");
}

#endif  // __HIP__

}  // namespace flux
