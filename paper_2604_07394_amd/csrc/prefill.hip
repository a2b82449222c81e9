// flux_attn_prefill: tiled causal GQA attention on bf16 MFMA, Full (Eq. 1) or Sparse (Eq. 2 with the
// sink + window subset of Sec. 4.1 / App. C.3), chosen per sequence by the cached mode byte.
//
// Shape of the computation (one workgroup = 128 query rows, 4 waves x 32 rows = 2 column blocks of 16 queries;
// launches of few tiles 4 waves x 16 rows; which rows these are, see the kernel):
//   for each VISITED 64-key block (FA: all blocks up to the diagonal; SA: the sink blocks and the
//   blocks that intersect the tile's window, nothing else: hidden blocks are skipped, not masked)
//     S^T[key][q]  = K[key][:] . Q[q][:]     MFMA 16x16x32 bf16, A = K rows from LDS, B = Q in registers
//     online softmax along keys.  S is kept TRANSPOSED: a query column belongs to the 4 lanes
//     (n, g = 0..3), each holding 4 of a 16-key block's scores in its accumulator registers, so the
//     running reference is a per-lane scalar and the row sum a per-lane partial that is only combined
//     across the 4 lanes at the end.
//     O^T[d][q]   += V^T[d][key] . P^T[key][q]   the accumulator layout of two 16-key blocks of S^T is the
//     B-operand layout of this product for 32 keys (keys taken in the order 4g..4g+3, 16+4g..16+4g+3), so
//     P never moves between lanes; V^T comes from row-major LDS through the transposing LDS read, its
//     keys in the same order.
// The 16x16x32 form is used because it is the one this chip sustains: a loop of nothing but MFMAs on
// random bf16 data reaches 2030-2280 TFLOP/s with it and 1170-1450 with 32x32x16, whatever the number of
// independent accumulators.
// Only blocks that straddle the causal diagonal or a window / sink edge evaluate the element mask.
//
// flux_attn_prefill_blocksparse is the same kernel (template flag BS) with another list of visited blocks: a
// sequence whose mode byte is 0 visits the key blocks that a caller-given keep matrix marks for the query
// blocks of the workgroup's tile (Eq. 2 over an arbitrary set of 64-position blocks, App. C.3: the block is
// the minimum unit of sparsity), found by scanning the matrix 64 key blocks at a time; blocks that no row of
// the tile keeps are never loaded.
#include <type_traits>

#include "flux_internal.h"

namespace flux {

typedef __attribute__((__vector_size__(4 * sizeof(int32_t)))) int32_t i32x4;

// Quotients by a divisor that the host knows, by the round-up method of Granlund and Montgomery (Division by invariant integers using
// multiplication, 1994): n / d = (mulhi(n, mul) + n) >> shift for n < 2^31 (mul = floor(2^32 (2^shift - d) / d) + 1 with 2^shift >= d).
struct Divisor {
  uint32_t mul, shift;
};

inline Divisor divisor(uint32_t d) {
  uint32_t shift = 0;
  while (shift < 31 && (1ull << shift) < d) ++shift;
  return {(uint32_t)(((((uint64_t)1 << shift) - d) << 32) / d + 1), shift};
}

__device__ __forceinline__ int quotient(int n, const Divisor& d) { return (int)(((uint32_t)(((uint64_t)(uint32_t)n * d.mul) >> 32) + (uint32_t)n) >> d.shift); }

struct PrefillArgs {
  const __bf16* q;        // [T, Hq, D]
  const int32_t* cu_q;    // [B + 1]
  const __bf16* k;
  const __bf16* v;
  int64_t stride_b, stride_h, stride_t;
  const int32_t* kv_len;
  const uint8_t* mode;
  int capacity;
  int hq, hkv, group, batch;
  int xcd_map;            // 0 plain, 1 pairs-per-XCD, 2 XCDs-per-pair, 3 planned on the device (see the kernel)
  int sink_lim, win_blocks, blk_shift;   // SA geometry (see sa_geom)
  int n_qtiles, n_wg;
  Divisor by_group, by_hkv, by_qtiles;
  int turn;               // block-sparse form: query tiles after which the pairs of a round change XCD
  float scale_log2;
  int out_fp32;
  void* out;
  uint32_t* status;       // sticky device status word
  // block-sparse form only: keep flags [batch, bm_heads, bm_qblocks, bm_kblocks], one byte per (query block, key
  // block) pair of 64 x 64 positions; row 0 is the block that holds the call's first query of that sequence
  const uint8_t* bmask;
  int bm_heads, bm_qblocks, bm_kblocks;
  // planned launches only: a tile's key blocks may be shared out over several workgroups
  int split_units;        // 0: never; else the units a launch may have beyond one per tile
  int part_units;         // units whose partial results the workspace holds
  float* part_o;          // unnormalised outputs of a unit, [unit][BM][D] (sequences whose tiles are split have the first units)
  float* part_ml;         // reference (score units) and weight sum of its rows, [unit][BM][2]
  i32x4* tile_info;       // [batch][n_kv_heads][n_qtiles]: first unit, unit stride, units of the tile; behind them, per sequence, the most of them that a tile of it has
  int merge_rows, merge_wgs;   // merge launch: rows of a tile per workgroup, workgroups that the tiles of a sequence are shared by
};

constexpr float kWeightGuard = 1073741824.0f;   // 2^30: a block whose weights sum past this moves the softmax reference

// All transfers of one wave for one whole tile in a single statement (four for K and four for V, or two and two):
// the LDS destination of transfer t is the uniform base plus a compile-time offset, so M0 is produced by one
// scalar add, and nothing is scheduled between the transfers.  A transfer keeps the issuing wave for about 64
// cycles whatever surrounds it (measured: the vector memory port of a SIMD takes one lane's 16 bytes per cycle),
// so their place in the iteration does not matter; they sit right behind the barrier, where the stage is free.
#define FLUX_DMA_ONE(v, p, o) "s_add_u32 m0, %[lds], %[" o "]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[" v "], %[" p "]\n\t"
template <int OFF, int KT>   // OFF: LDS offset of the stage; KT: bytes from the K tile to the V tile of a stage
__device__ __forceinline__ void dma_tile4(const char* kt, const char* vt, const int (&ko)[4], const int (&vo)[4],
                                          uint32_t lds_base) {
  asm volatile(FLUX_DMA_ONE("k0", "kt", "o0") FLUX_DMA_ONE("k1", "kt", "o1") FLUX_DMA_ONE("k2", "kt", "o2")
               FLUX_DMA_ONE("k3", "kt", "o3") FLUX_DMA_ONE("v0", "vt", "o4") FLUX_DMA_ONE("v1", "vt", "o5")
               FLUX_DMA_ONE("v2", "vt", "o6") FLUX_DMA_ONE("v3", "vt", "o7")
               : : [k0] "v"(ko[0]), [k1] "v"(ko[1]), [k2] "v"(ko[2]), [k3] "v"(ko[3]), [v0] "v"(vo[0]), [v1] "v"(vo[1]),
                   [v2] "v"(vo[2]), [v3] "v"(vo[3]), [kt] "s"(kt), [vt] "s"(vt), [lds] "s"(lds_base), [o0] "i"(OFF),
                   [o1] "i"(OFF + 4096), [o2] "i"(OFF + 8192), [o3] "i"(OFF + 12288), [o4] "i"(OFF + KT),
                   [o5] "i"(OFF + KT + 4096), [o6] "i"(OFF + KT + 8192), [o7] "i"(OFF + KT + 12288)
               : "memory", "m0", "scc");
}
template <int OFF, int KT>
__device__ __forceinline__ void dma_tile2(const char* kt, const char* vt, const int (&ko)[2], const int (&vo)[2],
                                          uint32_t lds_base) {
  asm volatile(FLUX_DMA_ONE("k0", "kt", "o0") FLUX_DMA_ONE("k1", "kt", "o1") FLUX_DMA_ONE("v0", "vt", "o4")
               FLUX_DMA_ONE("v1", "vt", "o5")
               : : [k0] "v"(ko[0]), [k1] "v"(ko[1]), [v0] "v"(vo[0]), [v1] "v"(vo[1]), [kt] "s"(kt), [vt] "s"(vt),
                   [lds] "s"(lds_base), [o0] "i"(OFF), [o1] "i"(OFF + 4096), [o4] "i"(OFF + KT), [o5] "i"(OFF + KT + 4096)
               : "memory", "m0", "scc");
}

// ---- the plan of a launch, taken on the device
// Every wave of a planned launch (2 to 64 sequences, or one whose tiles may be split; lane b looks after sequence b) finds
// out from the lengths and mode bytes which unit of work its workgroup is: the tiles of the sequences with the longest key
// lists first, no empty workgroups between them (a grid shaped by the host's bounds leaves most workgroups of short
// sequences empty, and long ones late).  Where the host allows it (split_units), the key blocks of a tile are shared out
// over several units, so that a few query rows behind long contexts fill the chip as well; their partial results are
// merged by a second kernel.  The plan is latency at the start of every workgroup: those past the last unit leave as soon
// as the units are summed (8192 + 63 x 100 tokens, 32/8 heads: 1324 us with all workgroups ranking first, 605 now, 616
// without a plan), and sequences that are all alike need no ranking.
constexpr int kMinSplitBlocks = 16;             // lists of at most so many key blocks are never split (a unit has about half of it at least)
constexpr int kResident128 = 512;               // workgroups of four waves the chip holds at once: two per CU, at head dimension
constexpr int kResident64 = 768;                // 64 three
constexpr int kPlanTiles = 512;                 // batches of at least so many tiles by the host's bounds are planned: a smaller
                                                // one is resident at once, and the plan only delays it (us without / with
                                                // it: 8 x 100 tokens 7.65 / 9.1, 4 x 64 at 8/2 heads of 64 4.7 / 5.0)
constexpr int kSplitUnits = 1024;               // units a launch that splits may have beyond one per tile
constexpr int kSplitFewTiles = 448;             // merges of at most so many tiles give a row to every thread; batches of at most so
                                                // many by the host's bounds may split from 40 key blocks on
constexpr int kSplitMaxTiles = 16384;           // ... and of at most so many where the lists may be long for so many tiles (see launch_prefill)

// Whether it pays to share out the keys of so many tiles, the longest of which walks so many key blocks: what the idle
// part of the chip can take of the walk has to be worth the plan, the partial results and the second launch.  us whole /
// split, one sequence of 32/8 heads of 128 (a tile is 32 tokens of a KV head): 128 tiles, 18, 24 and 32 blocks 24.8 /
// 30.7, 31.2 / 33.0, 39.7 / 37.1; 250 tiles, 32, 47 and 64 blocks 31.5 / 37.7, 56.1 / 57.1, 74.8 / 70.9; 320 tiles, 64 and
// 96 blocks 86 / 91, 128 / 125; 376 tiles, 256 blocks 365 / 389; 8 tiles, 18 blocks 22.7 / 18.8.  8/2 heads of 64: 2
// tiles, 18 blocks 16.2 / 14.6; 32 tiles, 18 and 32 blocks 17.5 / 20.2, 27.7 / 20.8.
__host__ __device__ __forceinline__ bool split_pays(int tiles, int blocks, int resident) {
  const float t = (float)tiles;
  return 3 * tiles <= 2 * resident && (float)blocks * (1.0f - t / (float)resident) >= (resident <= kResident128 ? 15.0f + t / 18.0f : 16.0f + t / 8.0f);
}

// Place of the j-th of the nj workgroups of an XCD in the order from long to short.  Consecutive workgroups of an XCD go
// round its 32 CUs, and a launch of at most two per CU is resident at once: its second half is handed out in reverse, so
// that the longest share a CU with the shortest.
__device__ __forceinline__ int pair_long_with_short(int j, int nj) { return nj > 32 && nj <= 64 && j >= 32 ? 32 + nj - 1 - j : j; }

struct PrefillUnit {
  int b;                  // sequence, -1: past the last unit
  int kvh, tile;
  int chunk;              // key blocks a unit takes at most
  int ci;                 // which part of its tile's blocks this unit takes
  int slot0, slot_step;   // unit numbers for the partial results of this tile
  int q_begin, n_q, len;
  bool sa;
};

// resident: workgroups of the launch that the chip holds at once
template <bool PACK>
__device__ __forceinline__ PrefillUnit prefill_plan(const PrefillArgs& a, int wg, int l, int bm, int resident) {
  PrefillUnit u;
  // this lane's sequence: lengths under the clamps, tiles, key blocks of its longest tile (an upper bound for SA)
  int q_begin = 0, n_q = 0, len = 0, tiles = 0, nb = 0;
  bool sa = false, bad = false;
  if (l < a.batch) {
    q_begin = a.cu_q[l];
    n_q = a.cu_q[l + 1] - q_begin;
    len = a.kv_len[l];
    sa = a.mode[l] == 0;
    bad = n_q < 0 || len < 0 || len > a.capacity || n_q > len;
    len = len < 0 ? 0 : (len > a.capacity ? a.capacity : len);
    n_q = n_q < 0 ? 0 : (n_q > len ? len : n_q);
    tiles = PACK ? min((int)(((int64_t)n_q * a.group + bm - 1) / bm), a.n_qtiles) : min((n_q + bm - 1) / bm, a.n_qtiles) * a.group;
    nb = (len + 63) >> 6;
    if (sa) {
      const int64_t win = min((int64_t)a.win_blocks << a.blk_shift, (int64_t)len);
      nb = min(nb, ((min(a.sink_lim, len) + 63) >> 6) + (int)((win + bm) >> 6) + 2);
    }
  }
  if (wg == 0 && threadIdx.x < 64 && bad) atomicOr(a.status, (uint32_t)FLUX_DEV_BAD_LENGTH);
  u.chunk = 0x7FFFFFFF;
  int nc = tiles > 0 ? 1 : 0;
  float share = 0.f;
  bool worth = false;                                        // this lane's lists are a reason to split
  if (PACK && a.split_units > 0) {
    const int t = __builtin_amdgcn_readlane(wave_inclusive_sum(tiles), 63) * a.hkv;
    share = (float)(__builtin_amdgcn_readlane(wave_inclusive_sum(tiles * nb), 63) * a.hkv) / (float)resident;
    // few tiles; or enough of them, but a list that takes twice as long as its share of the chip
    worth = tiles > 0 && nb > kMinSplitBlocks && (3 * t <= 2 * resident ? split_pays(t, nb, resident) : nb >= 64 && (float)nb > 2.0f * share);
  }
  if (PACK && __builtin_amdgcn_ballot_w64(worth) != 0) {
    // Key blocks a unit takes at most: every lane works out one candidate, around the share of one of the workgroups
    // the chip holds, by a model in units of one block: the longest unit, or that share plus half a unit of
    // unevenness where there is more than one round, plus 0.02 for writing and merging the partial result of a unit
    // (66 KB each way; a block takes 1.65 us).
    const int cand = l == 63 ? 0x3FFFFFFF : max(kMinSplitBlocks, (int)(share * (float)(l + 4) * (1.0f / 16.0f)) + 1);
    const float inv = 1.0f / (float)cand;
    int units = 0, parts = 0, longest = 0;
    for (int j = 0; j < a.batch; ++j) {
      const int tj = __builtin_amdgcn_readlane(tiles, j) * a.hkv, nbj = __builtin_amdgcn_readlane(nb, j);
      int n = (int)((float)(nbj - 1) * inv);                                 // parts of its tiles: (nb - 1) / cand, then + 1
      n += (n + 1) * cand <= nbj - 1 ? 1 : (n * cand > nbj - 1 ? -1 : 0);
      n = tj > 0 ? n + 1 : 0;
      units += tj * n;
      parts += n > 1 ? tj * n : 0;
      longest = max(longest, n > 0 ? (int)((float)nbj / (float)n) + 1 : 0);
    }
    float cost = units <= resident ? (float)longest : fmaxf((float)longest, share + 0.5f * (float)longest);
    cost += 0.02f * (float)parts;
    if (units + 8 * a.batch > a.n_wg || parts + 8 * a.batch > a.part_units) cost = 1e30f;   // (never the last: it splits nothing)
    int best = (__builtin_bit_cast(int, cost) & ~63) | l;                     // (positive floats order like their bits)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) best = min(best, __shfl_xor(best, off));
    u.chunk = __builtin_amdgcn_readlane(cand, __builtin_amdgcn_readfirstlane(best) & 63);
    nc = tiles > 0 ? (nb + u.chunk - 1) / u.chunk : 0;
  }
  const bool parts = __builtin_amdgcn_ballot_w64(nc > 1) != 0;
  if (PACK && a.split_units > 0 && wg == 0 && threadIdx.x < a.batch) a.tile_info[a.batch * a.hkv * a.n_qtiles + threadIdx.x] = i32x4{nc, 0, 0, 0};
  u.b = -1;
  const int t0 = __builtin_amdgcn_readlane(tiles, 0);
  const bool alike = __builtin_amdgcn_ballot_w64(l < a.batch && (tiles != t0 || nb != __builtin_amdgcn_readlane(nb, 0))) == 0;
  if (!parts && alike) {
    // Nothing is split and the sequences are as long as each other: a unit per (KV head, tile), found without a ranking.
    // Workgroups go to the 8 XCDs by id mod 8, and the units of one KV head walk the same K/V rows: they get ids of one
    // residue, or of 8 / hkv residues.  q: the unit's place among those of its head
    const int total = t0 * a.batch;
    int q, nj = total;                                       // nj: units of this XCD
    const int x = wg & 7;
    int j = wg >> 3;
    if ((a.hkv & 7) == 0) {
      nj = total * (a.hkv >> 3);
      if (j >= nj) return u;
      if (resident >= 512) j = pair_long_with_short(j, nj);
      const int o = a.hkv == 8 ? 0 : j / total;
      u.kvh = 8 * o + x;
      q = j - o * total;
    } else if (a.hkv < 8 && (a.hkv & (a.hkv - 1)) == 0) {
      const int sh = a.hkv == 1 ? 3 : (a.hkv == 2 ? 2 : 1);
      nj = (total + (1 << sh) - 1) >> sh;
      if (j >= nj) return u;
      if (resident >= 512) j = pair_long_with_short(j, nj);
      u.kvh = x & (a.hkv - 1);
      q = (j << sh) + (x >> (3 - sh));
      if (q >= total) return u;                              // padding of the last round
    } else {
      if (wg >= total * a.hkv) return u;
      u.kvh = wg / total;
      q = wg - u.kvh * total;
    }
    // Few rounds: the sequences take turns, heaviest tiles first (28/4 heads, 4 x 1000 tokens 41 us, one sequence after
    // the other 49).  Many rounds, or a sequence that fills a round by itself: one after the other, for the L2 (4 x 8192
    // 1806, in turn 1816; 16 x 700 99, in turn 102)
    int tt;
    if (t0 < 64 && nj < resident / 2) {
      tt = __builtin_amdgcn_readfirstlane(div_small(q, a.batch, 1.0f / (float)a.batch));
      u.b = q - tt * a.batch;
    } else {
      u.b = __builtin_amdgcn_readfirstlane(div_small(q, t0, 1.0f / (float)t0));
      tt = q - u.b * t0;
    }
    u.tile = t0 - 1 - tt;
    u.ci = u.slot0 = u.slot_step = 0;
    u.q_begin = __builtin_amdgcn_readlane(q_begin, u.b);
    u.n_q = __builtin_amdgcn_readlane(n_q, u.b);
    u.len = __builtin_amdgcn_readlane(len, u.b);
    u.sa = __builtin_amdgcn_readlane((int)sa, u.b) != 0;
    return u;
  }
  // units of the sequence: one per (KV head, part, tile).  Workgroups go to the 8 XCDs by id mod 8, and the units of one
  // (KV head, part) walk the same K/V rows: they get ids of one residue (or of 8 / groups residues).
  const int groups = a.hkv * nc;
  const int share_sh = groups == 1 ? 3 : (groups == 2 ? 2 : (groups == 4 ? 1 : 0));
  const int units = share_sh > 0 ? ((tiles + (1 << share_sh) - 1) >> share_sh) * 8 : groups * tiles;
  int units_s = units, idx_s = l;
  int incl = wave_inclusive_sum(units);
  const int total_units = __builtin_amdgcn_readlane(incl, 63);
  int id = wg;
  if (id >= total_units) return u;                           // (most workgroups, where the host's bounds are far above the lengths)
  // longest first, if they are not all alike: rank by (key blocks, index), then the units in that order
  if (a.batch > 1) {
    const int key = (nb << 6) | (63 - l);                    // no two alike; lanes without a sequence hold the lowest
    int rank = 0;
    for (int j = 0; j < a.batch; j += 8) {
#pragma unroll
      for (int v = 0; v < 8; ++v) rank += __builtin_amdgcn_readlane(key, j + v) > key ? 1 : 0;
    }
    rank = l < a.batch ? rank : l;
    units_s = __builtin_amdgcn_ds_permute(4 * rank, units);
    idx_s = __builtin_amdgcn_ds_permute(4 * rank, l);
    incl = wave_inclusive_sum(units_s);
  }
  if (resident >= 512) id = 8 * pair_long_with_short(id >> 3, (total_units - (id & 7) + 7) >> 3) + (id & 7);
  const int at = __builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= id));
  u.b = __builtin_amdgcn_readlane(idx_s, at);
  const int before = __builtin_amdgcn_readlane(incl, at) - __builtin_amdgcn_readlane(units_s, at);
  const int local = id - before;
  const int n_t = __builtin_amdgcn_readlane(tiles, u.b), n_g = __builtin_amdgcn_readlane(groups, u.b), sh = __builtin_amdgcn_readlane(share_sh, u.b);
  int grp, tt;
  if (sh > 0) {
    const int x = local & 7;
    grp = x & (n_g - 1);
    tt = ((local >> 3) << sh) + (x >> (3 - sh));
  } else if ((n_g & 7) == 0) {
    tt = (local >> 3) % n_t;
    grp = ((local >> 3) / n_t) * 8 + (local & 7);
  } else {
    tt = local % n_t;
    grp = local / n_t;
  }
  grp = __builtin_amdgcn_readfirstlane(grp);
  tt = __builtin_amdgcn_readfirstlane(tt);
  if (tt >= n_t) {                                           // padding of the last round
    u.b = -1;
    return u;
  }
  u.ci = quotient(grp, a.by_hkv);
  u.kvh = grp - u.ci * a.hkv;
  u.tile = n_t - 1 - tt;                                     // heaviest first
  u.slot0 = before + u.kvh * n_t + u.tile;
  u.slot_step = a.hkv * n_t;
  u.q_begin = __builtin_amdgcn_readlane(q_begin, u.b);
  u.n_q = __builtin_amdgcn_readlane(n_q, u.b);
  u.len = __builtin_amdgcn_readlane(len, u.b);
  u.sa = __builtin_amdgcn_readlane((int)sa, u.b) != 0;
  return u;
}

// A tile is BM = 16 * QB * NW rows.  PACK: they are the query rows of ALL heads of the group, token by token: row R is head
// R % group of token R / group.  Short runs of queries then fill their tiles (16 new tokens of a group of 4 are half a
// tile, not an eighth of four), a tile spans few tokens, so that little of what the diagonal or a window's start cuts is
// worked out for nothing, and its query rows are contiguous in memory.  Otherwise a tile is 128 tokens of one head:
// finding the rows costs a workgroup about a microsecond, more than that saves where tiles are full (8 x 2048 tokens
// packed 3 % slower), and in the block-sparse form the keep matrix differs between heads.
// QB: column blocks of 16 rows per wave, 1 in launches of few tiles (where that pays, see launch_prefill)
// (Eight waves and 256 rows per workgroup, one per CU, which transfer every tile once for twice the rows, were 1 to 3 % faster from
// 32768 tokens on until the loop lost its taken branches; us with eight / with four since: 32768 tokens 7013 / 6767, 28/4 heads
// 6063 / 5894, 65536 tokens 27328 / 27320, sparse layers 1752 / 1750 and 3637 / 3632, 16384 tokens behind 16384 5073 / 5017.)
template <int D, bool BS, bool PLAN = false, bool PACK = false, int QB = 2>
__global__ __launch_bounds__(256, 2) void prefill_kernel(PrefillArgs a) {
  constexpr int NW = 4;                   // waves, two workgroups per CU
  constexpr bool SPLIT = PLAN && PACK;    // tiles may be split
  constexpr int WR = 16 * QB;             // query rows per wave
  constexpr int BM = WR * NW;             // query rows per workgroup
  constexpr int BN = 64;                  // keys per iteration: two halves of 32, the K dimension of one PV MFMA
  constexpr int KC = D / 32;              // MFMA k-steps over the head dimension (QK^T)
  constexpr int DB = D / 16;              // 16-wide output blocks over the head dimension (PV)
  constexpr int KB = BN / 16;             // 16-key blocks of S^T per iteration
  constexpr int KS = BN / 32;             // 32-key steps of the PV product per iteration
  constexpr int CPR = D / 8;              // 16-byte chunks per row
  constexpr int ROWB = D * 2;             // bytes per K/V row
  // K tile: unpadded rows, the 16-byte chunk index XOR-swizzled by the row (D = 128: row & 15; D = 64, two
  // rows per 64 banks: (row >> 1) & 7).  A wave-wide 16-byte LDS read is served in four passes of 16 lanes,
  // and within lanes 0..31 the passes are {0-3, 12-15, 20-27} and {4-11, 16-19, 28-31} (measured with the
  // bank conflict counter).  With lane (n, g) reading row n, chunk 4*kc + g, a pass holds rows {0-3, 12-15}
  // at one chunk and rows {4-11} at the chunk next to it; both row sets are closed under XOR with 1, 2 and
  // 3, so the swizzled chunks of a pass are a permutation of all 16 and every pass covers 64 distinct banks.
  // (Rows padded by one chunk give two-way conflicts with this mapping, by two chunks none.)
  constexpr int KPITCH = ROWB;
  constexpr int NKI = BN * CPR / 64;         // wave-wide 1 KB transfers per K tile
  constexpr int NVI = BN * CPR / 64;         // wave-wide 1 KB transfers per V tile
  constexpr int KTILE = BN * ROWB;
  constexpr int VTILE = BN * ROWB;        // V tile: unpadded rows, 32-byte units XOR-swizzled by the row
  constexpr int STAGE = KTILE + VTILE;
  constexpr int KPW = NKI / NW;               // K transfers per wave
  constexpr int VPW = NVI / NW;               // V transfers per wave
  constexpr int RPI = 64 / CPR;              // V rows per transfer
  static_assert(BN * CPR % 64 == 0, "V tile must split into whole wave transfers");
  static_assert(NKI % NW == 0 && NVI % NW == 0 && (KPW == 4 || KPW == 2) && VPW == KPW, "every wave issues the same transfers");

  __shared__ __attribute__((aligned(1024))) char smem[2 * STAGE];
  // Planned launches: what only the end of the kernel needs waits in LDS (kept in scalar registers it pushes values of the
  // loop out of them).
  __shared__ struct { int rows, rem0, grp, hq, slot, out_fp32; int64_t tile_off; FLUX_GLOBAL void* out; FLUX_GLOBAL float* part_o; FLUX_GLOBAL float* part_ml; } fin;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave of the workgroup
  const int l = tid & 63;
  const int g = l >> 4, n = l & 15;
  const int grp = PACK ? a.group : 1;                        // heads whose rows share a tile
  // (the arguments that a workgroup's start needs, asked for together: tied to its number.  Not where tiles may be split, where the
  // scalar registers are short as it is and it gains nothing, nor in batches of head dimension 64 (us with / without, 32/8 heads: 1325 and
  // 2914 tokens behind 2685 and 1017 106.4 / 104.6, 4 x 4000 268.5 / 264.3, 3000, 700 and 5000 151.3 / 150.2, 8 x 700 25.7 / 25.9;
  // at head dimension 128 8192 and 63 x 100 tokens 597 / 603, 2782, 35, 64 and 802 71.1 / 71.8))
  int i = blockIdx.x;
  if constexpr (!PLAN || (!PACK && D == 128)) asm("" : "+s"(i) : "s"(a.q), "s"(a.cu_q), "s"(a.k), "s"(a.v), "s"(a.stride_b), "s"(a.stride_h), "s"(a.stride_t), "s"(a.kv_len), "s"(a.mode),
      "s"(a.capacity), "s"(a.hq), "s"(a.hkv), "s"(a.group), "s"(a.batch), "s"(a.xcd_map), "s"(a.sink_lim), "s"(a.win_blocks),
      "s"(a.blk_shift), "s"(a.n_qtiles), "s"(a.n_wg), "s"(a.by_group), "s"(a.by_hkv), "s"(a.by_qtiles));
  // ---- which (sequence, KV head, tile) this workgroup owns.  Workgroups go to the 8 XCDs round-robin
  // by linear id, and each XCD has its own L2.  The workgroups that an XCD holds at one time are therefore
  // given neighbouring query tiles of one (sequence, KV head) pair, heaviest tiles first,
  // so that they walk the same K/V rows at the same time and the rows come from
  // HBM once per XCD and round instead of once per workgroup.
  int qt, kvh, h, b;                                         // h: first query head of the tile
  int q_begin, n_q, len, ci = 0, chunk = 0x7FFFFFFF, slot0 = 0, slot_step = 0;
  bool sa;
  if constexpr (PLAN) {
    const PrefillUnit u = prefill_plan<PACK>(a, i, l, BM, D == 64 ? kResident64 : kResident128);
    if (u.b < 0) return;                                     // uniform for the workgroup
    b = u.b;
    kvh = u.kvh;
    h = u.kvh * a.group;
    qt = u.tile;
    if constexpr (!PACK) {                                   // tiles of one head: the heads of a group next to each other
      qt = quotient(u.tile, a.by_group);
      h += u.tile - qt * a.group;
    }
    q_begin = u.q_begin;
    n_q = u.n_q;
    len = u.len;
    sa = u.sa;
    ci = u.ci;
    chunk = u.chunk;
    slot0 = u.slot0;
    slot_step = u.slot_step;
    if (len < 1) return;
  } else {
    const int n_pairs = a.batch * a.hkv;
    const int gw = a.group;                                  // workgroups per (pair, query tile)
    if (a.xcd_map == 1) {                                    // n_pairs a multiple of 8: eight pairs at a time, one per XCD
      const int x = i & 7;
      int j = i >> 3;
      if (!BS) j = pair_long_with_short(j, a.n_wg >> 3);
      // An XCD takes its pairs one after the other (all tiles of a pair, heaviest first, the heads of a tile next to
      // each other).  Interleaving the pairs tile by tile looks more even, but in a ragged batch the tiles past a
      // short sequence's end are empty workgroups, and at fixed places of a short period they keep falling to the
      // same CUs (consecutive workgroups go round the CUs of an XCD), leaving the others idle: measured 1.5 - 2 x.
      // Two rotations even out work that differs between heads (block-sparse launches whose heads keep different
      // shares), at no cost where it does not: the heads of a tile change places from tile to tile, so that a CU
      // (which sees every 32nd workgroup of its XCD) meets all heads of the group; and the eight pairs of a round
      // change XCD every 16 tiles (one round of resident workgroups), so that every XCD works through two rounds of
      // every pair instead of all rounds of one.  A round streams its K/V rows from behind the L2 anyway.  Shorter prompts of
      // the block-sparse form have fewer tiles than make that even, so their pairs change sooner (launch_prefill).
      const int jg = quotient(j, a.by_group), r = quotient(jg, a.by_qtiles), qtd = jg - r * a.n_qtiles;
      const int g = j + qtd - quotient(j + qtd, a.by_group) * gw;
      const int pair = ((x + qtd / (BS ? a.turn : 16)) & 7) + 8 * r;
      b = quotient(pair, a.by_hkv);
      kvh = pair - b * a.hkv;
      h = kvh * gw + g;
      qt = a.n_qtiles - 1 - qtd;
    } else if (a.xcd_map == 2) {                             // n_pairs divides 8: 8 / n_pairs XCDs share a pair
      const int x = i & 7, j = i >> 3, sh = n_pairs >> 1;    // n_pairs = 2^sh: 1, 2 or 4
      const int pair = x & (n_pairs - 1), jg = quotient(j, a.by_group);
      const int qtd = (jg << (3 - sh)) + (x >> sh);
      b = quotient(pair, a.by_hkv);
      kvh = pair - b * a.hkv;
      h = kvh * gw + j - jg * gw;
      qt = a.n_qtiles - 1 - qtd;
      if (qt < 0) return;                                    // padding of the last round (uniform)
    } else {                                                 // any other shape: plain order, heavy tiles first
      const int row = quotient(i, a.by_qtiles);
      qt = a.n_qtiles - 1 - (i - row * a.n_qtiles);
      const int head = quotient(row, a.by_group);            // KV head, counted over the sequences
      b = quotient(head, a.by_hkv);
      kvh = head - b * a.hkv;
      h = row - b * a.hq;
    }
    // (the lengths and the mode byte, all asked for before any of them is looked at)
    int q_end = a.cu_q[b + 1], mode = a.mode[b];
    q_begin = a.cu_q[b];
    len = a.kv_len[b];
    asm("" : "+s"(q_begin) : "s"(q_end), "s"(len), "v"(mode));
    const int n_q_given = q_end - q_begin;
    // lengths the host could not see: negative, past the capacity, or more queries than cached positions;
    // they are clamped below, and reported once per sequence
    if (qt == a.n_qtiles - 1 && h == 0 && tid == 0 && (n_q_given < 0 || len < 0 || len > a.capacity || n_q_given > len))
      atomicOr(a.status, (uint32_t)FLUX_DEV_BAD_LENGTH);
    len = len > a.capacity ? a.capacity : len;
    if (len < 1) return;                                     // nothing cached: nothing to attend
    // the queries are the last n_q cached positions, so there cannot be more of them than positions: the
    // surplus rows of an inconsistent call are not computed (every key tile then starts inside the cache)
    n_q = n_q_given < len ? n_q_given : len;
    sa = __builtin_amdgcn_readfirstlane(mode) == 0;
  }
  const int64_t n_rows = (int64_t)n_q * grp;                 // rows of the pair (of the head, in the block-sparse form)
  if ((int64_t)qt * BM >= n_rows) return;                    // uniform for the workgroup
  const int pos0 = len - n_q;                                // position of the first query
  // rows are counted from the tile's first one: row x of the tile belongs to token tok0 + (rem0 + x) / grp, head
  // (rem0 + x) % grp of the group.  (x is small: the quotient is taken through floats)
  const int rows = (int)min((int64_t)BM, n_rows - (int64_t)qt * BM);
  const int tok0 = PACK ? (int)((uint32_t)(qt * BM) / (uint32_t)grp) : qt * BM, rem0 = qt * BM - tok0 * grp;
  const float inv_grp = __builtin_amdgcn_rcpf((float)grp);
  auto tok_of = [&](int x) { return !PACK ? x : (int)(((float)(rem0 + x) + 0.5f) * inv_grp); };   // from tok0 on

  // query rows of the tile / of this wave, as absolute positions
  const int i_tile_min = pos0 + tok0;
  const int i_tile_max = i_tile_min + __builtin_amdgcn_readfirstlane(tok_of(rows - 1));
  const int r_w0 = WR * w;                                   // first row of this wave, within the tile
  const bool wave_active = r_w0 < rows;
  const int i_w_min = i_tile_min + __builtin_amdgcn_readfirstlane(tok_of(r_w0));
  const int i_w_max = wave_active ? i_tile_min + __builtin_amdgcn_readfirstlane(tok_of(min(r_w0 + WR - 1, rows - 1))) : i_w_min - 1;
  // where row x lies in q and out
  const int64_t tile_off = ((int64_t)(q_begin + tok0) * a.hq + h) * D;
  auto row_off = [&](int x) {
    const int t = tok_of(x);
    return tile_off + (t * a.hq + (PACK ? rem0 + x - t * grp : 0)) * D;
  };
  // ---- block-sparse form: the visited key blocks come from the keep matrix.  The tile's 128 rows lie in up
  // to three 64-position query blocks (two when the first query sits on a block boundary); a key block is
  // visited when any of them keeps it.  The matrix is scanned 64 key blocks at a time: lane l of every wave reads
  // the flag of key block win + l for each of the tile's query blocks, a ballot turns them into one 64-bit word
  // per query block, and the blocks are taken from the lowest set bit up.  Every wave runs the same scan (all of
  // it in scalar registers), so no exchange is needed.  A query block always keeps its own (diagonal) block, and
  // never a later one; an FA sequence (mode byte 1) keeps everything.
  const int rb0 = i_tile_min >> 6;                           // absolute index of the tile's first query block
  const int n_rb = (i_tile_max >> 6) - rb0 + 1;              // 1 .. 3
  int scan_win = -64;                                        // first key block of the 64 being scanned
  unsigned long long scan_bits[3] = {0, 0, 0};               // what is left of them, per query block of the tile
  int cur_kb = -1, cur_rows = 0;                             // the block of this iteration, and which query blocks keep it
  // The flags of a window are asked for one window ahead, those of the first one in front of the query rows (they come back in
  // the order they were asked for in; 8 % of the blocks kept, 16384 tokens 222 -> 220 us, 32768 686 -> 674, 65536 2405 -> 2369).
  // Every lane reads a flag of the matrix, whatever it needs: no branch differs between lanes, see weights_guarded.
  const int rq0 = rb0 - (pos0 >> 6);                         // row of the matrix
  uint8_t flags[3] = {0, 0, 0};
  auto fetch_flags = [&](int win) __attribute__((always_inline)) {
    const uint8_t* seq = a.bmask + ((int64_t)b * a.bm_heads + (a.bm_heads > 1 ? h : 0)) * a.bm_qblocks * (int64_t)a.bm_kblocks;
#pragma unroll
    for (int r = 0; r < 3; ++r) flags[r] = seq[(int64_t)min(rq0 + r, a.bm_qblocks - 1) * a.bm_kblocks + min(win + l, a.bm_kblocks - 1)];
  };
  if constexpr (BS) fetch_flags(0);

  // ---- visited key blocks: [0, n_a) and [win0, win0 + n_b)
  const int last_blk = i_tile_max / BN;
  int n_a, win0, n_b;
  if (!sa) {
    n_a = last_blk + 1; win0 = 0; n_b = 0;
  } else {
    const int sink_end = min(a.sink_lim, i_tile_max + 1);    // keys [0, sink_end) are sinks in reach
    n_a = (sink_end + BN - 1) / BN;
    const int wfirst = window_start(i_tile_min, a.blk_shift, a.win_blocks);   // first key any row's window reaches
    win0 = max(wfirst / BN, n_a);
    n_b = last_blk + 1 - win0;
    if (n_b < 0) n_b = 0;
  }
  const int n_blocks = n_a + n_b;
  // a split tile: this unit takes part ci of the list
  int it0 = 0, n_iter = n_blocks, n_parts = 1;             // (n_iter: one past its last)
  if (SPLIT && chunk < n_blocks) {
    n_parts = (n_blocks + chunk - 1) / chunk;
    it0 = (int)((int64_t)ci * n_blocks / n_parts);
    n_iter = (int)((int64_t)(ci + 1) * n_blocks / n_parts);
  }
  if (SPLIT && tid == 0 && ci < n_parts) {
    fin = {rows, rem0, grp, a.hq, n_parts > 1 ? slot0 + ci * slot_step : -1, a.out_fp32, tile_off, (FLUX_GLOBAL void*)a.out, (FLUX_GLOBAL float*)a.part_o, (FLUX_GLOBAL float*)a.part_ml};
    if (a.split_units > 0 && ci == 0) a.tile_info[((int64_t)b * a.hkv + kvh) * a.n_qtiles + qt] = i32x4{slot0, slot_step, n_parts, 0};
  }
  if constexpr (SPLIT) {
    // (said to be uniform behind the branch of one thread: the loop over the blocks is compiled for lanes that leave it at
    // different times otherwise)
    it0 = __builtin_amdgcn_readfirstlane(it0);
    n_iter = __builtin_amdgcn_readfirstlane(n_iter);
    if (__builtin_amdgcn_readfirstlane(ci) >= __builtin_amdgcn_readfirstlane(n_parts)) return;
  }

  const char* kbase = (const char*)(a.k + (int64_t)b * a.stride_b + (int64_t)kvh * a.stride_h);
  const char* vbase = (const char*)(a.v + (int64_t)b * a.stride_b + (int64_t)kvh * a.stride_h);
  const int pitch_g = (int)a.stride_t * 2;                   // bytes between rows in the cache

  // ---- direct global -> LDS transfers.  One transfer moves 64 x 16 bytes to 1 KB of consecutive LDS;
  // which (row, chunk) a lane fetches decides where that chunk lands.  Per lane, the row and chunk of
  // each of this wave's transfers are fixed for the whole kernel.
  // Transfer I covers rows I*RPI .. +RPI-1 of a tile; lane l sits at (row l/CPR, physical chunk l%CPR) and
  // fetches the logical chunk that the swizzle maps there.  Wave w issues the transfers w, w + NW, ...  For K the
  // swizzle of row (w + NW*t)*RPI + l/CPR is (4w + l/16) & (CPR-1) for both head sizes, a per-lane constant.
  const int v_lrow = l / CPR;
  const int k_chunk = (l % CPR) ^ ((4 * w + (l >> 4)) & (CPR - 1));
  auto k_slot = [&](int t, int rmax) __attribute__((always_inline)) { return min((w + NW * t) * RPI + v_lrow, rmax) * pitch_g + k_chunk * 16; };
  // the 32-byte units of a V row are XOR-swizzled by the row (D = 128: row & 7; D = 64, two rows per 64
  // banks: (row >> 1) & 3), which makes the transposing reads below conflict-free; the row of transfer
  // w + NW*t, lane l is (w + NW*t) * RPI + l / CPR, so the swizzle is a per-lane constant
  const int v_swz = D == 128 ? ((4 * (w & 1) + v_lrow) << 1) : (((v_lrow >> 1) & 3) << 1);
  const int v_chunk = (l % CPR) ^ v_swz;
  auto v_slot = [&](int t, int rmax) __attribute__((always_inline)) { return min((w + NW * t) * RPI + v_lrow, rmax) * pitch_g + v_chunk * 16; };
  int k_off[KPW], v_off[VPW];                                // byte offsets inside a tile that is fully cached
#pragma unroll
  for (int t = 0; t < KPW; ++t) k_off[t] = k_slot(t, BN);
#pragma unroll
  for (int t = 0; t < VPW; ++t) v_off[t] = v_slot(t, BN);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(FLUX_LDS char*)smem;

  const uint32_t lds_w = lds0 + 1024 * w;                    // this wave's 1 KB slot inside every NW KB of a stage

  // tile index (in units of BN keys) of iteration `it`: the blocks [0, n_a) first, then [win0, win0 + n_b)
  auto tile_of = [&](int it) __attribute__((always_inline)) { return it < n_a ? it : win0 + (it - n_a); };

  // All transfers of one tile with rows clamped to the cached length: the first tile, and a last tile that
  // is only partly inside the cache.
  auto issue_tile_clamped = [&](int tile, int stage) __attribute__((always_inline)) {
    const int j0 = tile * BN;
    const int rmax = len - 1 - j0;                           // rows past the cached length are clamped
    const char* kt = kbase + (int64_t)j0 * pitch_g;
    const char* vt = vbase + (int64_t)j0 * pitch_g;
    const uint32_t lk = lds_w + stage * STAGE;
#pragma unroll
    for (int t = 0; t < KPW; ++t)
      lds_copy16(kt, k_slot(t, rmax), lk + 1024 * NW * t);
#pragma unroll
    for (int t = 0; t < VPW; ++t)
      lds_copy16(vt, v_slot(t, rmax), lk + KTILE + 1024 * NW * t);
  };

  // The first tile is asked for as soon as it is known which one that is, in front of the query rows and of all that the loop needs to
  // know besides (block-sparse form: it is not known yet).  The memory latencies of a workgroup's start show in its time: only
  // the other workgroup of the CU works meanwhile.  They come one after the other: the arguments (once for all, see above), the
  // lengths and the mode (together, see above), this.  Workgroups took 3.3 us from their start to the first tile (us before / now, 32/8
  // heads of 128: 129 to 3001 tokens in 5 sequences 122.6 / 120.9, 1000 tokens 21.2 / 20.8, 32 x 100 24.6 / 23.7, 32768 tokens
  // sparse 1684 / 1678, 7000 and 13000 tokens block-sparse 217.0 / 212.5).
  if constexpr (!BS) {
    if (n_iter > it0) issue_tile_clamped(tile_of(it0), 0);
  }

  // ---- Q operand: lane (n, g) holds d = 32*kc + 8*g .. +7 of its two query rows
  bf16x8 qf[QB][KC];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const __bf16* qrow = a.q + row_off(min(r_w0 + 16 * qb + n, rows - 1));
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) qf[qb][kc] = *(const bf16x8*)(qrow + 32 * kc + 8 * g);
  }

  // this lane's two query rows (column n of column block qb; rows past the last one repeat it): position, and first key
  // of the row's SA window
  int i_mine[QB], w_lo_mine[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    i_mine[qb] = i_tile_min + tok_of(min(r_w0 + 16 * qb + n, rows - 1));
    w_lo_mine[qb] = window_start(i_mine[qb], a.blk_shift, a.win_blocks);
  }
  // first key of the SA window of the wave's first row and of its last row
  const int w_lo_first = window_start(i_w_min, a.blk_shift, a.win_blocks);
  const int w_lo_last = window_start(max(i_w_max, i_w_min), a.blk_shift, a.win_blocks);

  // ---- per-lane LDS read offsets (bytes, relative to stage 0; the stage is added as an immediate)
  // K fragment (kb, kc): row 16*kb + n, logical chunk 4*kc + g (d = 32*kc + 8*g ..), swizzled by the row
  const int k_xr = D == 128 ? n : (n >> 1);
  int k_rd[KC];
#pragma unroll
  for (int kc = 0; kc < KC; ++kc) k_rd[kc] = n * KPITCH + (((4 * kc + g) ^ k_xr) * 16);
  // V^T fragment for output block db: the transposing read of lane (n, g) addresses row 4*g + n/4, columns
  // 16*db + 4*(n%4) .. +3, and returns V^T[16*db + n][keys 4g .. 4g+3] of the 16-row group
  const int v_row = 4 * g + (n >> 2);
  const int v_xr = D == 128 ? (v_row & 7) : ((v_row >> 1) & 3);
  int v_rd[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) v_rd[db] = KTILE + v_row * ROWB + ((db ^ v_xr) * 32) + (n & 3) * 8;

  float m_ref[QB];                                           // the score the exponents of a row refer to
  float mneg[QB];                                            // -m_ref * scale_log2 (0 while a row has no reference yet)
  float l_run[QB];                                           // this lane's part of the row sums
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m_ref[qb] = -INFINITY;
    mneg[qb] = l_run[qb] = 0.f;
  }
  bool all_ref = false;                                      // wave-uniform: every row of the wave has a reference
  f32x4 o[DB][QB];
#pragma unroll
  for (int i = 0; i < DB; ++i)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) o[i][qb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- which iterations are PLAIN for this wave: the wave is active, every key of the block is visible to
  // every row of the wave (no element mask, nothing to skip).  In tile indices: the block ends at or before the
  // wave's first row (tile < c_end), and for SA it lies wholly inside the sinks (tile < s_full) or starts at
  // or after the window start of the wave's LAST row (tile >= w_first_full).  As iteration ranges:
  // [0, pa_end) and [pb_begin, pb_end).  A wave issues its instructions in order and two waves share a SIMD, so
  // every instruction of the loop shows in its time: the plain iterations (all but a few per workgroup) skip the
  // mask flags and the block's first key altogether.
  int pa_end = 0, pb_begin = 0, pb_end = 0;
  if (wave_active) {
    const int c_end = (i_w_min + 1) / BN;
    if (!sa) {
      pa_end = min(n_a, c_end);
    } else {
      pa_end = min(min(n_a, c_end), a.sink_lim / BN);
      const int w_first_full = (w_lo_last + BN - 1) / BN;
      pb_begin = n_a + max(w_first_full - win0, 0);
      pb_end = min(n_a + max(c_end - win0, 0), n_blocks);
    }
  }
  // the last tile may be only partly inside the cache; every other tile is whole
  const bool last_whole = n_iter > it0 && len - 1 - tile_of(n_iter - 1) * BN >= BN - 1;
  const int lim_whole = last_whole ? n_iter : n_iter - 1;    // iterations it + 1 < lim_whole transfer a whole tile
  const unsigned pb_len = pb_end > pb_begin ? pb_end - pb_begin : 0;
  const int64_t step_b = (int64_t)BN * pitch_g;              // bytes from one key block to the next
  const int64_t jump_b = (int64_t)(win0 - n_a + 1) * step_b; // from the last sink block to the first window block
  const char* kt_n = kbase + (int64_t)(n_iter > it0 + 1 ? tile_of(it0 + 1) : 0) * step_b;   // the tile the next transfer brings in
  const char* vt_n = vbase + (int64_t)(n_iter > it0 + 1 ? tile_of(it0 + 1) : 0) * step_b;

  auto next_kept_block = [&](int& rows) __attribute__((always_inline)) -> int {
    for (;;) {
      const unsigned long long any = scan_bits[0] | scan_bits[1] | scan_bits[2];
      if (__builtin_expect(any != 0, 1)) {
        const int bit = __builtin_ctzll(any);
        rows = (int)((scan_bits[0] >> bit) & 1) | (int)(((scan_bits[1] >> bit) & 1) << 1) | (int)(((scan_bits[2] >> bit) & 1) << 2);
        const unsigned long long clr = ~(1ull << bit);
        scan_bits[0] &= clr;
        scan_bits[1] &= clr;
        scan_bits[2] &= clr;
        return scan_win + bit;
      }
      scan_win += 64;
      if (scan_win > last_blk) return -1;
      const int kbk = scan_win + l;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const int rb = rb0 + r;                              // absolute query block
        const bool own = r < n_rb && kbk <= rb, asked = own && kbk < rb && sa;   // never a later block (causal), nothing for absent rows;
        // the diagonal block is kept whatever the flag says.  A matrix too small for the lengths found on the device hides what
        // it does not cover, and says so
        const bool inside = rq0 + r < a.bm_qblocks && kbk < a.bm_kblocks;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(asked && !inside) != 0 && w == 0 && h == 0, 0)) atomicOr(a.status, (uint32_t)FLUX_DEV_BAD_LENGTH);
        scan_bits[r] = __builtin_amdgcn_ballot_w64(own && (!asked || (inside && flags[r] != 0)));
      }
      if (scan_win + 64 <= last_blk) fetch_flags(scan_win + 64);
    }
  };
  int nxt_kb = -1, nxt_rows = 0;

  // One iteration.  STG (the LDS stage of this tile) is a compile-time constant: the loop is unrolled by two so
  // that every LDS address is a loop-invariant register plus an immediate.
  auto iteration = [&](int it, auto stg_c) __attribute__((always_inline)) {
    constexpr int STG = decltype(stg_c)::value;
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0): this wave's transfers have landed
    __syncthreads();                                         // ... and everyone's; the other stage is free
    if constexpr (BS) {
      nxt_kb = next_kept_block(nxt_rows);
      if (__builtin_expect(nxt_kb >= 0, 1)) {                // the next kept block, in flight during the math below
        if (__builtin_expect((nxt_kb + 1) * BN <= len, 1)) {
          const int64_t off = (int64_t)nxt_kb * step_b;
          if constexpr (KPW == 4) dma_tile4<(STG ^ 1) * STAGE, KTILE>(kbase + off, vbase + off, k_off, v_off, lds_w);
          else dma_tile2<(STG ^ 1) * STAGE, KTILE>(kbase + off, vbase + off, k_off, v_off, lds_w);
        } else {
          issue_tile_clamped(nxt_kb, STG ^ 1);
        }
      }
    } else if (__builtin_expect(it + 1 < lim_whole, 1)) {    // the next tile, in flight during the math below
      if constexpr (KPW == 4) dma_tile4<(STG ^ 1) * STAGE, KTILE>(kt_n, vt_n, k_off, v_off, lds_w);
      else dma_tile2<(STG ^ 1) * STAGE, KTILE>(kt_n, vt_n, k_off, v_off, lds_w);
      const int64_t adv = it + 2 == n_a ? jump_b : step_b;   // on to the tile after it (the window part starts at win0)
      kt_n += adv;
      vt_n += adv;
    } else if (it + 1 < n_iter) {
      issue_tile_clamped(tile_of(it + 1), STG ^ 1);          // a last tile that is only partly inside the cache
    }
    bool plain = it < pa_end || (unsigned)(it - pb_begin) < pb_len;
    // block-sparse form: this block (cur_kb) as the wave's rows see it.  The wave's 32 rows lie in one or two of
    // the tile's query blocks; the block is plain when both keep it and it ends at or before the wave's first row.
    const int bs_j0 = cur_kb * BN, bs_rows = cur_rows;
    if constexpr (BS) {
      const int r_lo = (i_w_min >> 6) - rb0, r_hi = (max(i_w_max, i_w_min) >> 6) - rb0;
      const bool k_lo = (bs_rows >> r_lo) & 1, k_hi = (bs_rows >> r_hi) & 1;
      plain = wave_active && k_lo && k_hi && bs_j0 + BN - 1 <= i_w_min;
      cur_kb = nxt_kb;                                       // the state moves on; this iteration keeps bs_j0 / bs_rows
      cur_rows = nxt_rows;
      if (__builtin_expect(!plain && (!wave_active || bs_j0 > i_w_max || !(k_lo || k_hi)), 0)) return;   // nothing for this wave here
    }

    FLUX_LDS char* st = (FLUX_LDS char*)smem + STG * STAGE;
    // Order of the block, written out so that every LDS read is issued well before its use (the fences keep
    // the compiler from moving the reads):
    //   K fragments of half 0 | S^T half 0, the K fragments of half 1 read between its MFMAs |
    //   S^T half 1, the V fragments of half 0 read between its MFMAs | weights |
    //   O^T += half 0, the V fragments of half 1 read between its MFMAs | O^T += half 1
    f32x4 s[KB][QB];             // s[kb][qb][i]: key j0 + 16*kb + 4*g + i against query row (qb, n)
    bf16x8 pf[QB][KS];           // pf[qb][ks]: weights of keys 32*ks + {4g..4g+3, 16+4g..16+4g+3}, as a B operand
    bf16x8 kf[KB][KC];
    bf16x8 vf[KS][DB];
    auto read_k = [&](int kb, int kc) __attribute__((always_inline)) { kf[kb][kc] = *(FLUX_LDS bf16x8*)(st + k_rd[kc] + 16 * kb * KPITCH); };
    auto read_v = [&](int ks, int db) __attribute__((always_inline)) {
      FLUX_LDS char* vp = st + v_rd[db] + 32 * ks * ROWB;
      const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((FLUX_LDS bf16x4*)vp);
      const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((FLUX_LDS bf16x4*)(vp + 16 * ROWB));
      vf[ks][db] = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    // Softmax weights against the reference m_ref the accumulators already refer to, WITHOUT looking for the
    // block's maximum first: any reference gives the same quotient, and fp32 / bf16 keep their relative
    // precision over the whole exponent range.  A row without a reference yet uses 0.
    float l_blk[QB];
    auto weights = [&]() __attribute__((always_inline)) {
      const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        l_blk[qb] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          uint32_t pk[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const f32x4& sv = s[2 * ks + (t >> 1)][qb];
            const float p0 = fast_exp2(__builtin_fmaf(sv[2 * (t & 1)], a.scale_log2, mneg[qb]));
            const float p1 = fast_exp2(__builtin_fmaf(sv[2 * (t & 1) + 1], a.scale_log2, mneg[qb]));
            pk[t] = pack_bf16(p0, p1);
            // the denominator sums the same rounded weights the numerator uses
            l_blk[qb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk[t]), ones, l_blk[qb], false);
          }
          pf[qb][ks] = __builtin_bit_cast(bf16x8, u32x4{pk[0], pk[1], pk[2], pk[3]});
        }
      }
    };
    auto accumulate = [&](int ks) __attribute__((always_inline)) {        // o[db][qb][i] is d = 16*db + 4*g + i of query row (qb, n)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
          o[db][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[ks][db], pf[qb][ks], o[db][qb], 0, 0, 0);
    };
    // Only when a row has no reference yet, or some weight of the block left the guarded range (or
    // overflowed), does the wave take the block's maximum, move the reference of THAT row there (rescaling l and O) and
    // redo the weights.  In the steady state the maximum, its cross-lane steps and the rescale are not executed.  Rows
    // that need no move keep their reference, so that a row's result does not depend on the rows that share its wave
    // (launch shapes group rows differently, and give the same bits).
    auto weights_guarded = [&]() __attribute__((always_inline)) {
      weights();
      // (one ballot per comparison: each is then the comparison's own lane mask, with no vector instruction between)
      if (__builtin_expect(!all_ref || (__builtin_amdgcn_ballot_w64(!(l_blk[0] < kWeightGuard)) | __builtin_amdgcn_ballot_w64(!(l_blk[QB - 1] < kWeightGuard))) != 0, 0)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          float mloc = s[0][qb][0];
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) mloc = fmaxf(mloc, s[kb][qb][i]);
          mloc = fmaxf(mloc, __shfl_xor(mloc, 16));                              // over the 4 lanes of the row
          mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
          // the row's own reason: no reference yet, or a weight of 2^31 and more (which trips the guard by itself, so that
          // the row moves whatever the others do)
          const bool move = m_ref[qb] == -INFINITY || __builtin_fmaf(mloc, a.scale_log2, mneg[qb]) >= 31.f;
          const float m_new = fmaxf(m_ref[qb], mloc);
          // (selects and no branch: a branch that differs between lanes makes the compiler structurise the whole loop, which
          // leaves taken branches behind in every block)
          const bool moves = move && m_new > m_ref[qb];                          // false while both are -inf
          const float al = moves ? fast_exp2((m_ref[qb] - m_new) * a.scale_log2) : 1.f;   // 0 for a row's first reference
          l_run[qb] *= al;
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db][qb] *= al;
          m_ref[qb] = moves ? m_new : m_ref[qb];
          mneg[qb] = moves ? -m_new * a.scale_log2 : mneg[qb];
        }
        weights();
        all_ref = __builtin_amdgcn_ballot_w64((m_ref[0] == -INFINITY) | (m_ref[QB - 1] == -INFINITY)) == 0;
      }
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) l_run[qb] += l_blk[qb];
    };

    // a block that an edge of the visible set crosses, or that this wave does not see at all, needs the
    // block's first key and the mask flags; a plain block needs none of that scalar work
    int j0 = 0;
    bool mask_causal = false, mask_edge = false;
    if constexpr (BS) {
      j0 = bs_j0;
      mask_causal = !plain;
    } else if (__builtin_expect(!plain, 0)) {
      j0 = tile_of(it) * BN;
      bool skip = !wave_active || j0 > i_w_max;
      mask_causal = j0 + BN - 1 > i_w_min;                   // the diagonal crosses the block
      if (sa) {
        const bool all_sink = j0 + BN <= a.sink_lim;
        if (!all_sink) {
          if (j0 >= a.sink_lim && j0 + BN - 1 < w_lo_first) skip = true;          // before every window
          mask_edge = j0 < w_lo_last;                        // a window or sink edge falls inside the block
        }
      }
      if (skip) return;
    }
    // Wave priorities: the second product above the scores, and those above the softmax and the transfers.  Of the two waves of
    // a SIMD one then gets through its MFMAs while the other does its vector work, instead of both taking turns at either (us with
    // the softmax raised, nothing raised, and so, 32/8 heads of 128: 8192 tokens 458 / 465 / 438, 4000 126 / 133 / 118, 4 x 512
    // behind 16000 491 / 469 / 435, 32768 tokens 6899 / 6760 / 6655; other orders of the four parts lie between).
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) read_k(kb, kc);
    __builtin_amdgcn_sched_barrier(0);
    // S^T of keys 0..31 with the K fragments of keys 32..63 read between the MFMAs, then S^T of keys 32..63 with the V
    // fragments of keys 0..31 read between them: a read between two MFMAs costs the wave a few cycles, in a run of
    // reads sixteen, and every fragment is asked for at least sixteen MFMAs before its use.  The accumulators start
    // from what the caller put into s.
    auto scores = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < 2 * KC; ++t) {
        const int kc = t >> 1, kb = t & 1;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][kc], qf[qb][kc], s[kb][qb], 0, 0, 0);
        read_k(2 + kb, kc);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int t = 0; t < 2 * KC; ++t) {
        const int kc = t >> 1, kb = 2 + (t & 1);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][kc], qf[qb][kc], s[kb][qb], 0, 0, 0);
#pragma unroll
        for (int db = t * DB / (2 * KC); db < (t + 1) * DB / (2 * KC); ++db) read_v(0, db);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // Element masks are put into the accumulators the scores start from: 0 for a visible pair, -inf for a hidden one
    // (the sum of the products then stays -inf), so a plain block starts from the constant 0 and the scores of either
    // kind of block come out of the MFMAs in the same registers.  (With the masks applied to the finished scores the
    // compiler keeps masked and unmasked scores in different registers and copies all 32 of them in every plain
    // block.)  Key j = j0 + 4*g + c with the constant c = 16*kb + i, so each bound is moved into the lane once
    // (bound - j0 - 4*g) and compared with constants.
    if (__builtin_expect(mask_edge, 0)) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const int hi = i_mine[qb] - j0 - 4 * g, lo = w_lo_mine[qb] - j0 - 4 * g, sl = a.sink_lim - j0 - 4 * g;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int c = 16 * kb + i;
            const bool vis = (c <= hi) & ((c < sl) | (c >= lo));
            s[kb][qb][i] = vis ? 0.f : -INFINITY;
          }
      }
      scores();
    } else if (__builtin_expect(mask_causal, 0)) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        int hi = i_mine[qb] - j0 - 4 * g;
        // block-sparse form: a row whose query block does not keep this key block sees none of it
        if constexpr (BS) hi = ((bs_rows >> ((i_mine[qb] >> 6) - rb0)) & 1) ? hi : -1;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[kb][qb][i] = 16 * kb + i <= hi ? 0.f : -INFINITY;
      }
      scores();
    } else {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) s[kb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
      scores();
    }
    __builtin_amdgcn_s_setprio(0);
    weights_guarded();
    __builtin_amdgcn_s_setprio(2);
    __builtin_amdgcn_sched_barrier(0);
    // O^T += keys 0..31 with the V fragments of keys 32..63 read between the MFMAs
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) o[db][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[0][db], pf[qb][0], o[db][qb], 0, 0, 0);
      read_v(1, db);
      __builtin_amdgcn_sched_barrier(0);
    }
    accumulate(1);
    __builtin_amdgcn_s_setprio(0);
  };

  if constexpr (!BS) {
    for (int it = it0; it < n_iter; it += 2) {
      iteration(it, std::integral_constant<int, 0>());
      if (__builtin_expect(it + 1 < n_iter, 1)) iteration(it + 1, std::integral_constant<int, 1>());
    }
  } else {
    cur_kb = next_kept_block(cur_rows);
    if (cur_kb >= 0) issue_tile_clamped(cur_kb, 0);
    while (cur_kb >= 0) {
      iteration(0, std::integral_constant<int, 0>());
      if (__builtin_expect(cur_kb < 0, 0)) break;
      iteration(0, std::integral_constant<int, 1>());
    }
  }

  // ---- lane (n, g) holds d = 16*db + 4*g .. +3 of its two query rows
  const int f_rows = SPLIT ? __builtin_amdgcn_readfirstlane(fin.rows) : rows, f_slot = SPLIT ? __builtin_amdgcn_readfirstlane(fin.slot) : -1;
  const int f_rem0 = SPLIT ? fin.rem0 : rem0, f_grp = SPLIT ? fin.grp : grp, f_hq = SPLIT ? fin.hq : a.hq;
  const int64_t f_off = SPLIT ? fin.tile_off : tile_off;
  const int f_fp32 = SPLIT ? fin.out_fp32 : a.out_fp32;
  FLUX_GLOBAL void* f_out = SPLIT ? fin.out : (FLUX_GLOBAL void*)a.out;
  const float f_inv = __builtin_amdgcn_rcpf((float)f_grp);
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    float l_tot = l_run[qb];
    l_tot += __shfl_xor(l_tot, 16);
    l_tot += __shfl_xor(l_tot, 32);
    const float inv = 1.0f / l_tot;
    // bf16 rows: of two output blocks side by side, the lanes of odd g hand their part of the first to the lane of g - 1 and
    // get its part of the second, so that a lane stores eight columns in a row, and a store covers 64 bytes of each of its 16 rows
    // instead of 32: the address unit takes as long per row for either.  (All lanes take part, whatever they store.)  A workgroup
    // stored its tile in 1.4 us, of the 6 to 7 us between the last block of one workgroup and the first of the next (us with stores
    // of 8 bytes / now, 32/8 heads of 128: 129 to 3001 tokens in 5 sequences 123.2 / 121.3, 4 x 8192 1565 / 1554, 7000 and 13000
    // tokens block-sparse 222.6 / 217.1, 16384 226.4 / 222.6).
    u32x4 pk[DB / 2];
#pragma unroll
    for (int db = 0; db < DB; db += 2) {
      const f32x4 lo = o[db][qb] * inv, hi = o[db + 1][qb] * inv;
      const auto x0 = __builtin_amdgcn_permlane16_swap(pack_bf16(lo[0], lo[1]), pack_bf16(hi[0], hi[1]), false, false);
      const auto x1 = __builtin_amdgcn_permlane16_swap(pack_bf16(lo[2], lo[3]), pack_bf16(hi[2], hi[3]), false, false);
      pk[db / 2] = u32x4{x0[0], x1[0], x0[1], x1[1]};
    }
    const int x = r_w0 + 16 * qb + n;
    if (x >= f_rows) continue;
    if (SPLIT && f_slot >= 0) {
      // part of a tile: the unnormalised rows, their references and weight sums go to the workspace
      const int64_t row = (int64_t)f_slot * BM + x;
      if (g == 0) {
        fin.part_ml[2 * row] = m_ref[qb];
        fin.part_ml[2 * row + 1] = l_tot;
      }
      FLUX_GLOBAL float* dst = fin.part_o + row * D + 4 * g;
#pragma unroll
      for (int db = 0; db < DB; ++db) *(FLUX_GLOBAL f32x4*)(dst + 16 * db) = o[db][qb];
    } else {
      const int t = !PACK ? x : (int)(((float)(f_rem0 + x) + 0.5f) * f_inv);
      const int64_t off = f_off + (t * f_hq + (PACK ? f_rem0 + x - t * f_grp : 0)) * D;
      if (f_fp32) {
#pragma unroll
        for (int db = 0; db < DB; ++db) *(FLUX_GLOBAL f32x4*)((FLUX_GLOBAL float*)f_out + off + 16 * db + 4 * g) = o[db][qb] * inv;
      } else {
        FLUX_GLOBAL __bf16* dst = (FLUX_GLOBAL __bf16*)f_out + off + 16 * (g & 1) + 8 * (g >> 1);
#pragma unroll
        for (int db = 0; db < DB; db += 2) *(FLUX_GLOBAL u32x4*)(dst + 16 * db) = pk[db / 2];
      }
    }
  }
}

// The tiles whose key blocks were shared out over several units: out = sum_c w_c O_c / sum_c w_c l_c with
// w_c = exp(m_c - max m), parts in order.  D / 4 threads per row, a tile's rows over the gridDim.x workgroups of a tile (merge_rows
// each), the tiles of a sequence over gridDim.y = merge_wgs (as many as there are by the host's bounds, or fewer that take several each: a sequence
// that is not split costs its workgroups one load).
template <int D, int BM>
__global__ __launch_bounds__(256) void prefill_merge_kernel(PrefillArgs a) {
  constexpr int RPP = 1024 / D;           // rows per pass
  const int b = blockIdx.z;
  // What says whether there is anything to do is asked for together: the sequence's flag and lengths and, where a workgroup has one tile
  // by the host's bounds, that tile's entry (whatever it holds if the sequence has no such tile), and the other arguments.  A merge
  // is latencies one behind the other (us of the whole call with these in a row / together, 32/8 heads of 128: 16 tokens behind 30000
  // 36.6 / 35.4, 128 behind 16256 48.6 / 47.9, 100 behind 5000 34.4 / 33.5; 8/2 heads of 64, 34 and 112 behind 38574 and 608 30.9 / 29.8;
  // with many workgroups, most of which have nothing to do or all the same, half a us goes the other way: 512, 40 and 30 tokens behind 5000 to
  // 5800 65.3 / 65.7, 4 x 256 behind 2300 51.8 / 52.3).  The entry comes by a vector load, which a workgroup that leaves does not
  // wait for (by a scalar load 512, 40 and 30 tokens 66.4), and what the grid is comes with the arguments.
  const bool single = a.merge_wgs == a.hkv * a.n_qtiles;
  const i32x4* infos = a.tile_info + (int64_t)b * a.hkv * a.n_qtiles;
  int most = a.tile_info[a.batch * a.hkv * a.n_qtiles + b][0], q_end = a.cu_q[b + 1], len = a.kv_len[b];
  const int q_begin = a.cu_q[b];
  int at = blockIdx.y;                                       // (the workgroups are not more than the entries)
  asm volatile("" : "+v"(at));
  const i32x4 mine = infos[at];
  asm volatile("" : "+s"(most) : "s"(q_end), "s"(len), "s"(q_begin), "s"(a.capacity), "s"(a.group), "s"(a.hq), "s"(a.by_qtiles), "s"(a.part_o), "s"(a.part_ml),
      "s"(a.out), "s"(a.out_fp32), "s"(a.scale_log2), "s"(a.merge_rows));
  if (most < 2) return;                                      // none of its tiles was split
  int n_q = q_end - q_begin;
  len = len < 0 ? 0 : (len > a.capacity ? a.capacity : len);
  n_q = min(n_q, len);
  const int64_t n_rows = (int64_t)n_q * a.group;
  const int d = 4 * (threadIdx.x % (D / 4));
  const int per = a.merge_rows;
  // tiles of a KV head: all that the bounds count, or those that there are, which then take turns
  const int n_t = single ? a.n_qtiles : (int)min((n_rows + BM - 1) / BM, (int64_t)a.n_qtiles);
  for (int tile = blockIdx.y; tile < a.hkv * n_t; tile += a.merge_wgs) {
    const int kvh = single ? quotient(tile, a.by_qtiles) : tile / n_t, qt = tile - kvh * n_t;
    const int64_t row0 = (int64_t)qt * BM;
    if (row0 >= n_rows) continue;
    i32x4 info;
    if (single) {
#pragma unroll
      for (int i = 0; i < 3; ++i) info[i] = __builtin_amdgcn_readfirstlane(mine[i]);
    } else {
      info = infos[(int64_t)kvh * a.n_qtiles + qt];
    }
    const int parts = info[2];
    if (parts < 2) continue;
    for (int x = (int)blockIdx.x * per + threadIdx.x / (D / 4); x < ((int)blockIdx.x + 1) * per; x += RPP) {
      const int64_t row = row0 + x;
      if (row >= n_rows) break;
      const int64_t r0 = (int64_t)info[0] * BM + x, step = (int64_t)info[1] * BM;
      // four parts at a time, so that their loads are in flight together (the last part again where there are fewer)
      float m = -INFINITY, den = 0.f;
      f32x4 num = {0.f, 0.f, 0.f, 0.f};
      for (int c0 = 0; c0 < parts; c0 += 4) {
        float mc[4], lc[4];
        f32x4 oc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int64_t r = r0 + min(c0 + u, parts - 1) * step;
          mc[u] = c0 + u < parts ? a.part_ml[2 * r] : -INFINITY;
          lc[u] = a.part_ml[2 * r + 1];
          oc[u] = *(const f32x4*)(a.part_o + r * D + d);
        }
        const float m_new = fmaxf(fmaxf(fmaxf(mc[0], mc[1]), fmaxf(mc[2], mc[3])), m);
        if (m_new == -INFINITY) continue;                      // none of these parts sees a key of the row
        const float al = fast_exp2((m - m_new) * a.scale_log2);
        den *= al;
        num *= al;
        m = m_new;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float w = fast_exp2((mc[u] - m) * a.scale_log2);
          den += w * lc[u];
          num += w * oc[u];
        }
      }
      const float inv = 1.0f / den;
      const int64_t off = ((int64_t)(q_begin + row / a.group) * a.hq + (int64_t)kvh * a.group + row % a.group) * D + d;
      if (a.out_fp32) *(f32x4*)((float*)a.out + off) = num * inv;
      else *(u32x2*)((__bf16*)a.out + off) = u32x2{pack_bf16(num[0] * inv, num[1] * inv), pack_bf16(num[2] * inv, num[3] * inv)};
    }
  }
}

hipError_t launch_prefill(const Ctx& c, const flux_attn_cfg& cfg, const void* q, const int32_t* cu_q,
                          int max_q_len, int max_kv_len, const flux_kv_cache& cache, const uint8_t* mode,
                          const BlockMask* bm, void* out, hipStream_t s) {
  const float scale = cfg.softmax_scale != 0.f ? cfg.softmax_scale : 1.0f / sqrtf((float)cfg.head_dim);
  PrefillArgs a;
  a.q = (const __bf16*)q;
  a.cu_q = cu_q;
  a.k = (const __bf16*)cache.k;
  a.v = (const __bf16*)cache.v;
  a.stride_b = cache.stride_b;
  a.stride_h = cache.stride_h;
  a.stride_t = cache.stride_t;
  a.kv_len = cache.kv_len;
  a.mode = mode;
  a.capacity = cache.capacity;
  a.hq = cfg.n_q_heads;
  a.hkv = cfg.n_kv_heads;
  a.group = cfg.n_q_heads / cfg.n_kv_heads;
  a.batch = cache.batch;
  const SaGeom geom = sa_geom(cfg);
  a.sink_lim = geom.sink_lim;
  a.win_blocks = geom.win_blocks;
  a.blk_shift = geom.shift;
  constexpr int BM = 128;
  a.scale_log2 = scale * kLog2e;
  a.out_fp32 = cfg.out_dtype;
  a.out = out;
  a.status = c.status;
  a.bmask = bm ? bm->flags : nullptr;
  a.bm_heads = bm ? bm->heads : 0;
  a.bm_qblocks = bm ? bm->n_qblocks : 0;
  a.bm_kblocks = bm ? bm->n_kblocks : 0;
  if (max_q_len == 0) return hipSuccess;
  const long long n_pairs = (long long)cache.batch * cfg.n_kv_heads;
  // Batches are planned on the device (longest first, no empty workgroups).  us without a plan -> with it: 45 to 4876
  // tokens in 6 sequences, 28/4 heads, 317 -> 182; 17 and 2856 tokens 115 -> 66; 32/8 heads, 2782, 35, 64 and 802 tokens 78
  // -> 74; 300 and 400 tokens under a bound of 8192 18.6 -> 12.7; 8 x 2048 equal ones 278 -> 280.  Their tiles are packed
  // where that leaves a quarter fewer (64 prompts of 16 tokens 18.5 -> 9.1), or behind a cached context any fewer (64 x 16
  // tokens behind 900 81 -> 41).
  // Queries behind a cached context may have their tiles split (us before -> now, 32/8 heads of 128): 16 new tokens
  // behind 4000 cached 70 -> 27, behind 32000 528 -> 35; 128 behind 32000 546 -> 76; 512 behind 32000 549 -> 229; 1000
  // behind 32000 562 -> 435; 200, 333, 150 and 512 behind 16200, 9001, 24000 and 12345 297 -> 230; 100 and 4000 behind
  // 60000 and 3000 1258 -> 406.  Whether they are is decided on the device (split_pays); a launch that may split but does
  // not (a layer with a short sparse window, say) pays for the plan and the second launch all the same, 0.5 to 3 us.  So
  // the host lets only those that its bounds say may gain: few tiles for the length of the lists, or a batch (whose bounds
  // count tiles that short sequences do not have) with contexts long enough that one uneven sequence costs more than that:
  // 512, 40 and 30 tokens behind 5000 to 5800 123 -> 66, 4 x 256 equal ones behind 2300 50 -> 53.  The more tiles the bounds count,
  // the longer the lists have to be: 900, 3000, 200, 100 and 60 tokens behind 500, 700, 30000, 4000 and 60000 (28/4 heads, 3300 tiles,
  // 939 blocks) 951 -> 270, 238 to 2004 tokens behind 583 to 35383 (2520, 558) 585 -> 305, 504, 61 and 1573 tokens behind 1044,
  // 5599 and 761 (16/8 heads, 600, 89) 102 -> 54; of those that gain nothing 6 x 700 behind 5000 (28/4 heads, 936, 90) 262.1 -> 262.7,
  // 28 to 2368 tokens behind 767 to 28243 in six sequences (3552, 257) 366.5 -> 369.7.  Only sequences whose tiles are split take part in
  // the partial results, and they have the first units of the launch, so that the workspace need not hold one per tile.
  const long long packed = ((long long)max_q_len * a.group + BM - 1) / BM;    // tiles of a pair whose rows come from all heads
  const long long tiles = n_pairs * packed, blocks = ((long long)max_kv_len + 63) / 64;
  const long long unit_bytes = (long long)BM * (cfg.head_dim + 2) * 4, info_bytes = ((tiles + cache.batch) * 16 + 255) / 256 * 256;
  const long long fit = ((long long)c.partials_bytes - info_bytes) / unit_bytes;   // units whose partial results the workspace holds
  const long long grown = 64 + tiles / 24, least = tiles <= kSplitFewTiles ? 40 : (tiles <= 2048 && grown > 128 ? 128 : grown);
  const bool split = !bm && cache.batch <= 64 && max_kv_len > max_q_len && blocks > kMinSplitBlocks &&
                     ((tiles <= 768 && split_pays((int)tiles, (int)blocks, cfg.head_dim == 64 ? kResident64 : kResident128)) ||
                      (cache.batch > 1 && tiles <= kSplitMaxTiles && blocks >= least)) &&
                     fit >= 64 + 8 * cache.batch && (tiles + 8) * blocks < 0x7FFFFFFFll;
  const long long whole = n_pairs * a.group * ((max_q_len + 127ll) / 128);    // tiles of one head each
  const bool plan = split || (!bm && cache.batch > 1 && cache.batch <= 64 && whole >= kPlanTiles);
  const long long unpacked = whole / n_pairs;
  const bool pack = split || (plan && (max_kv_len > max_q_len ? packed < unpacked : 4 * packed <= 3 * unpacked));
  // Few tiles take 64 rows each, 16 per wave: twice the workgroups, and half the work of a block in each of them, where a
  // workgroup (or two) per CU walks its blocks one after the other and the chip waits for the longest.  us with 128 rows /
  // with 64, 32/8 heads of 128 unless said, append included: 512 tokens 23.3 / 19.9, 1000 33.3 / 28.2, 1500 46.1 / 41.2; 8/2
  // heads of 64, 1000 tokens 22.6 / 18.2; 16/8 heads, 3000 tokens 75.8 / 67.2; 700 tokens behind 900 42.1 / 35.0.  64-row
  // tiles read K and V twice as often, so it ends where all of them are not resident at once: above half as many 128-row
  // tiles as the chip holds if they walk lists of one length (1500 tokens behind 1500 78 / 87, a sparse layer of 128 + 512
  // keys at 1500 tokens 36.1 / 38.8, 600, 580 and 500 tokens 32.0 / 34.5), later for one whole prompt that no window cuts,
  // whose lists are half as long in the mean (1700 tokens 49.5 / 47.3, 2000 57.8 / 58.9).
  const int resident = cfg.head_dim == 64 ? kResident64 : kResident128;
  const bool triangular = cache.batch == 1 && max_kv_len == max_q_len && a.sink_lim + ((long long)a.win_blocks << a.blk_shift) >= max_q_len;
  const bool half = !bm && !plan && whole <= (triangular ? resident / 8 * 7 : resident / 2);
  const long long n_qtiles = half ? (max_q_len + 63ll) / 64 : ((long long)max_q_len * (pack ? a.group : 1) + BM - 1) / BM;
  a.n_qtiles = (int)n_qtiles;
  a.by_group = divisor(a.group);
  a.by_hkv = divisor(a.hkv);
  a.by_qtiles = divisor(a.n_qtiles);
  // The pairs of a block-sparse launch change XCD every 16 tiles, those of shorter prompts 16 times over the prompt: XA on
  // structured input, us for append, selection and launch with 16 tiles and as here: 4096 tokens 124 / 119.5, 16384 tokens
  // 478 / 470, 7000 and 13000 tokens 472 / 452, 16/8 heads 12000 tokens 192 / 187; not sooner for long ones, whose workgroups
  // share what the L2 holds (32768 tokens, everything kept, every 16, 8, 4 and 1 tiles: 7480, 7540, 7610 and 7980).
  a.turn = n_qtiles < 32 ? 2 : n_qtiles < 256 ? (int)n_qtiles / 16 : 16;
  a.split_units = a.part_units = 0;
  a.part_o = a.part_ml = nullptr;
  a.tile_info = nullptr;
  long long n_wg;
  if (plan) {
    a.xcd_map = 3;
    if (split) a.split_units = kSplitUnits;
    n_wg = (pack ? tiles : whole) + 8 * cache.batch + a.split_units;         // (the units of a sequence are padded to whole rounds of the XCDs)
    if (split) {
      a.tile_info = (i32x4*)c.partials;
      a.part_units = (int)(fit < n_wg ? fit : n_wg);
      a.part_o = (float*)((char*)c.partials + info_bytes);
      a.part_ml = a.part_o + (long long)a.part_units * BM * cfg.head_dim;
    }
  } else if (n_pairs % 8 == 0) {
    a.xcd_map = 1;
    n_wg = n_qtiles * cfg.n_q_heads * cache.batch;
  } else if (8 % n_pairs == 0) {
    a.xcd_map = 2;
    const long long share = 8 / n_pairs;
    n_wg = 8 * a.group * ((n_qtiles + share - 1) / share);
  } else {
    a.xcd_map = 0;
    n_wg = n_qtiles * cfg.n_q_heads * cache.batch;
  }
  if (n_wg > 0x7FFFFFFFll) return hipErrorInvalidValue;
  a.n_wg = (int)n_wg;
  const dim3 grid((unsigned)n_wg);
  const bool d128 = cfg.head_dim == 128;
  if (bm) {
    if (d128) hipLaunchKernelGGL((prefill_kernel<128, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((prefill_kernel<64, true>), grid, dim3(256), 0, s, a);
  } else if (plan) {
    if (pack && d128) hipLaunchKernelGGL((prefill_kernel<128, false, true, true>), grid, dim3(256), 0, s, a);
    else if (pack) hipLaunchKernelGGL((prefill_kernel<64, false, true, true>), grid, dim3(256), 0, s, a);
    else if (d128) hipLaunchKernelGGL((prefill_kernel<128, false, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((prefill_kernel<64, false, true>), grid, dim3(256), 0, s, a);
  } else {
    if (half && d128) hipLaunchKernelGGL((prefill_kernel<128, false, false, false, 1>), grid, dim3(256), 0, s, a);
    else if (half) hipLaunchKernelGGL((prefill_kernel<64, false, false, false, 1>), grid, dim3(256), 0, s, a);
    else if (d128) hipLaunchKernelGGL((prefill_kernel<128, false>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((prefill_kernel<64, false>), grid, dim3(256), 0, s, a);
  }
  if (a.split_units > 0) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // (few tiles have many parts each: a row per thread; otherwise two, since most workgroups find nothing to do)
    const unsigned per_tile = 128 * cfg.head_dim / 1024 / (tiles <= kSplitFewTiles ? 1 : 2);
    const long long per_seq = (long long)cfg.n_kv_heads * a.n_qtiles, most = 8192 / (per_tile * cache.batch);
    a.merge_rows = BM / (int)per_tile;
    a.merge_wgs = (int)(per_seq < most ? per_seq : most);
    const dim3 mgrid(per_tile, (unsigned)a.merge_wgs, cache.batch);
    if (cfg.head_dim == 128) hipLaunchKernelGGL((prefill_merge_kernel<128, 128>), mgrid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((prefill_merge_kernel<64, 128>), mgrid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace flux
