// flux_attn_decode: split-K streaming attention for one query row per sequence (Eq. 1 / Eq. 2 with
// one query; the decode step of Sec. 3.3 / App. B.3).
//
// Decode is bound by reading the K and V rows of the cache once from HBM.  The work of one
// (sequence, KV head) pair is the VISIBLE key list (FA: all positions; SA: the sinks followed by the
// window tail, so the hidden middle of the cache is never addressed) in blocks of 32 keys.  The lists of all pairs
// are laid end to end, and every workgroup takes the same share of that one long list, wherever it begins
// and ends: a run of blocks of one pair is a PART, and a workgroup whose range crosses from one pair into the next works
// off its parts one after the other.  (Calls of few keys, and of some hundred short lists, give a workgroup blocks of one
// list only.)  One workgroup of 256 threads, or 512 in calls of few keys, serves all query heads of the GQA
// group at once, so every K/V row is fetched exactly once per step.
//
// The range is found ON THE DEVICE from the lengths and mode bytes the call finds there (a prefix sum over the batch), so
// the mix of lengths and modes in the batch does not show in how evenly the chip is loaded (see DecodePlan for why the
// ranges are equal).
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
// The waves keep private (m, l, O) and are merged through LDS at the end of a part.  A pair that lies in one workgroup's
// range is done then; otherwise the part's unnormalised rows go to the workspace, and the part that arrives last at its
// pair (an arrival counter) merges the pair's parts in a fixed order (deterministic, no float atomics).  Without arrival
// counters (the static scratch) a second small kernel does, with the same sums in the same order.
#include <type_traits>
#include <utility>

#include "flux_internal.h"

namespace flux {

// What the cut is taken from.
struct SplitArgs {
  const int32_t* kv_len;
  const uint8_t* mode;
  int batch, capacity;
  int ring;               // != 0: the cache is a sink + ring store of a sparse layer, kv_len is logical, no mode bytes
  int sink_lim, win_blocks, blk_shift;   // SA geometry (see sa_geom)
  int max_keys;           // the host's bound on the keys any sequence attends to
  int pps;                // (KV head, query block) pairs per sequence = hkv * qblocks
  int bump;               // 1: the call also appends one row per sequence, so every list is one key longer than kv_len says
  int block_shift;        // lists are cut into blocks of 2^block_shift keys
  int most_by_four;       // calls of eight waves: workgroups up to which they take four blocks of a list where lists are merged
  int aligned_shift;      // few blocks: one workgroup per 4, 8 or 16 of a list while that takes at most 2^aligned_shift (see Cut); < 0: not
};

struct DecodeArgs {
  const __bf16* q;        // [B, Hq, D]
  const __bf16* k;
  const __bf16* v;
  int64_t stride_b, stride_h, stride_t;   // elements
  SplitArgs sp;
  int hq, hkv, group;     // group = hq / hkv
  int qblocks;            // ceil(group / 16)
  int rpu;                // rows per part = min(group, 16)
  float scale_log2;       // softmax scale * log2(e)
  float* part_o;          // unnormalised rows of the parts of unfinished pairs, [place][rpu][D] (see part_place)
  float* part_ml;         // their reference (score units) and weight sum, [place][rpu][2]
  int* table;             // two launches: [batch][2]: first block and blocks per pair of every sequence, and the cut, for the merge kernel
  uint32_t* status;       // sticky device status word
  // the fused decode step only: the row each sequence appends at position kv_len[b], [B, Hkv, D]
  const __bf16* k_new;
  const __bf16* v_new;
  uint32_t* arrived;      // calls merged in place: the counters (see kDecodeCounters); all zero between calls
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

// ---- the cut.  Blocks of all pairs, sequence by sequence and pair by pair, numbered from 0.  While they are few (one per
// wave of two workgroups per CU) every list is rounded up to a multiple of 4 and a workgroup takes 4, so that none
// crosses from one pair into the next; 8 where every list has no more than that (nothing to merge) or more than 64 (half
// the rows to merge).  (Calls of eight waves: see kDecodeFewWgs.)  Of 256 to 512 short lists it takes one each.  Otherwise the
// lists lie end to end, and workgroup u of 256 or 512 takes [range_begin(u), range_begin(u + 1)): equal shares not of the
// blocks but of what they take, for which a list is counted as a multiple of the waves and some blocks more (see find_cut).
struct Cut {
  int total;        // blocks
  int shift;        // equal shares: log2 of the workgroups
  int align;        // log2 of the blocks that a workgroup takes of a list; 0: an equal share of all lists
  int round, pad;   // a list of nb blocks is counted as nb rounded up to a multiple of round + 1, and pad more
};
__device__ __forceinline__ int cut_wgs(Cut c) { return c.align > 0 ? c.total >> c.align : 1 << c.shift; }
__device__ __forceinline__ int range_begin(Cut c, int u) {
  return c.align > 0 ? u << c.align : (int)(((unsigned long long)(unsigned)u * (unsigned)c.total) >> c.shift);
}
// the workgroup whose range holds block x
__device__ __forceinline__ int range_of(Cut c, int x) {
  if (c.align > 0) return x >> c.align;
  int u = min((int)((float)x * ((float)(1 << c.shift) / (float)c.total)), (1 << c.shift) - 1);
  while (range_begin(c, u) > x) --u;
  while (range_begin(c, u + 1) <= x) ++u;
  return u;
}
// Where the rows of part `i` of a pair go whose first part lies in the range of workgroup `first`: a range holds at most one
// part that its pair goes on behind and one that its pair began before.
__device__ __forceinline__ int part_place(int first, int i) { return i == 0 ? 2 * first + 1 : 2 * (first + i); }

__device__ __forceinline__ int blocks_of(const SplitArgs& s, int nv) { return (nv >> s.block_shift) + ((nv & ((1 << s.block_shift) - 1)) != 0 ? 1 : 0); }

// ---- the sequences of a call.  Lane i of every wave looks after `run` of them from i * run on: one each in a batch of up to
// 64, which stays in registers; larger batches of up to kDecodeTable are read once, by all waves together, into a table in LDS.
// (Read in groups of 64, each behind the one before it, for both passes of the cut and for every list that a range goes on to:
// us before / now, 1000 lists of 20 to 200 keys at 28/4 heads 119.1 / 107.2, 512 of 50 to 300 at 32/8 130.9 / 127.0.)
constexpr int kDecodeTable = 2048;
struct Seq {
  int len, md, nb;  // rows, mode bits (see load_seq), blocks
};
typedef FLUX_LDS u32x2 SeqTable;   // [run][64]: sequence i * run + j is entry j * 64 + i; its rows, and 4 * blocks + mode bits

__device__ __forceinline__ Seq load_counted(const SplitArgs& s, int b, bool& bad) {
  Seq q;
  bool sparse;
  int s_end, tail_start;
  load_seq(s, b, q.len, q.md, bad);
  q.nb = blocks_of(s, seq_visible(s, q.len, q.md, bad, sparse, s_end, tail_start));
  return q;
}
__device__ __forceinline__ Seq seq_at(const SplitArgs& s, const SeqTable* table, int run, int i, int j) {
  if (run * 64 <= kDecodeTable) {
    const u32x2 e = table[j * 64 + i];
    return Seq{(int)e[0], (int)(e[1] & 3), (int)(e[1] >> 2)};
  }
  bool bad;
  return load_counted(s, i * run + j, bad);
}

struct Lanes {
  Seq q;            // batches of up to 64: this lane's sequence
  int run;          // sequences of a lane
  int incl;         // blocks up to and including this lane's
  bool bad;         // this lane saw a clamp trip
  bool merged;      // calls of eight waves: some list takes more than one workgroup
};
__device__ __forceinline__ int counted(Cut c, int nb) { return nb > 0 ? ((nb + c.round) & ~c.round) + c.pad : 0; }

// (called by all waves of a workgroup, w: this one, of W)
template <int D, int W>
__device__ __forceinline__ Cut find_cut(const SplitArgs& s, int lane, int w, SeqTable* table, Lanes& r) {
  // Going on from one list to the next, a workgroup stands still for a memory latency and the merge of its waves, about as long
  // as four blocks of head dimension 128 take, and for up to three waves without a block.  Ranges of equally many blocks that
  // held whole lists, such as the eight sparse ones of a sequence among long ones, were the last ones of their call: us
  // before / now per layer, 32/8 heads of 128: 13 lists of 1223 to 15370 keys, half of them cut at 144, 42.5 / 32.0, 32 ragged ones at
  // 28/4 heads 40.1 / 36.9, 16 ring lists of 2112 at 28/4 25.0 / 23.7, 13 of 144 to 13696 37.1 / 33.7, 29 of 139 to 2305 26.8
  // / 26.3, 21 of 296 to 4373 at head dimension 64 23.4 / 18.7.  (3 to 6 blocks, and 5 to 12 at head dimension 64, differ by 2 %.)
  // With two workgroups per CU (see kLists) the other one streams meanwhile, and a block takes twice as long: a list of head
  // dimension 128 is a multiple of two and two blocks more then.  us with four and four / so: 104 lists of 1 to 4 keys among 24 of 2000
  // 53.0 / 48.7, 128 of 50 to 299 31.2 / 30.4, 1000 of 20 to 199 at 28/4 heads 73.4 / 72.1, 53 of 36 to 1044 at 16/8 36.3 / 35.5.
  // At head dimension 64 there is nothing in it: 136 of 6 to 200 18.9 / 20.4, 122 of 39 to 1278 45.9 / 44.9.
  constexpr int kSeam = 512 / D;
  // Two workgroups per CU where there are as many lists as CUs, since at most seams the other one goes on (us with one / two,
  // 32/8 heads of 128: 128 lists of 300 keys 39.9 / 34.5, 128 of 100 to 3000 61.8 / 52.6, 1000 of 20 to 200 at 28/4 heads 107 /
  // 82; but 16 lists of 2112, 128 in all, 29.4 / 31.0, 8 x 131072 629 / 665).  At head dimension 64 from a quarter of that on:
  // one workgroup has half the bytes in flight there (21 sequences of 296 to 4373 keys 22.8 / 20.5).
  constexpr int kLists = D == 64 ? 64 : 256;
  r.run = (s.batch + 63) >> 6;
  r.bad = false;
  r.q = Seq{0, 1, 0};
  if (__builtin_expect(r.run == 1, 1)) {
    if (lane < s.batch) r.q = load_counted(s, lane, r.bad);
  } else if (r.run * 64 <= kDecodeTable) {
    for (int j = w; j < r.run; j += W) {
      Seq q = {0, 1, 0};
      bool bad = false;
      if (lane * r.run + j < s.batch) q = load_counted(s, lane * r.run + j, bad);
      table[j * 64 + lane] = u32x2{(uint32_t)q.len, (uint32_t)(4 * q.nb + q.md)};
      r.bad |= bad;
    }
    __syncthreads();
  }
  // each(f): f(blocks) for every sequence of this lane
  auto take = [&](auto each) __attribute__((always_inline)) {
    Cut c = {0, kDecodeWgsShift, 0, 0, 0};
    if constexpr (W == 8) {
      bool merged = false;                                  // some list takes more than one workgroup
      int mine = 0, by_four = 0;
      each([&](int nb) __attribute__((always_inline)) {
        merged |= nb > 8;
        mine += (nb + 7) & ~7;
        by_four += (nb + 3) & ~3;
      });
      int incl = wave_inclusive_sum(s.pps * by_four);
      r.merged = __builtin_amdgcn_ballot_w64(merged) != 0;
      c.align = r.merged && __builtin_amdgcn_readlane(incl, 63) <= 4 * s.most_by_four ? 2 : 3;
      if (c.align == 3) incl = wave_inclusive_sum(s.pps * mine);
      c.round = (1 << c.align) - 1;
      r.incl = incl;
      c.total = __builtin_amdgcn_readlane(incl, 63);
      return c;
    }
    if (s.aligned_shift >= 0) {
      bool between = false;
      each([&](int nb) __attribute__((always_inline)) { between |= nb > 8 && nb <= 64; });
      c.align = __builtin_amdgcn_ballot_w64(between) == 0 ? 3 : 2;
      c.round = (1 << c.align) - 1;
    }
    // too many workgroups for that: one for each list where that pays, or an equal share of all lists: over how many ranges, and
    // what a list counts (calls of very many lists do not round)
    auto share = [&]() __attribute__((always_inline)) {
      int lists = 0, blocks = 0;
      each([&](int nb) __attribute__((always_inline)) {
        lists += nb != 0 ? s.pps : 0;
        blocks += s.pps * nb;
      });
      lists = __builtin_amdgcn_readlane(wave_inclusive_sum(lists), 63);
      const bool two = gridDim.x >= 2 << kDecodeWgsShift && lists >= kLists;   // workgroups per CU
      // 256 to 512 lists of up to 16 blocks take a workgroup each, none of which has a seam or anything to merge; up to 24 blocks
      // where there are hardly fewer lists than workgroups, and 24 (32 at head dimension 64) where every CU has one.  us in equal
      // ranges / so, 32/8 heads of 128 unless said: 64 lists of 200 to 328 keys 24.3 / 19.1, 64 of 50 to 296 21.1 / 16.4, 48 of
      // 300 to 508 25.7 / 23.2, 33 of 300 to 508 21.1 / 19.8, 40 of 50 to 439 at head dimension 64 13.8 / 11.2; 64 of 500 to 760
      // 39.6 / 35.1, 120 of 50 to 630 at 28/4 heads 28.8 / 24.8; 32 of 500 to 760 24.6 / 21.3, 32 of 50 to 760 20.9 / 19.7, 32 of
      // 50 to 630 at head dimension 64 13.4 / 11.1, 32 of 700 to 1010 there 17.0 / 15.2.
      // With fewer or longer lists the CU with two of the longest is the last (70 of 50 to 630 at 28/4 21.4 / 26.4, 48 of 700
      // to 1010 39.7 / 41.2, 33 of 500 to 760 26.7 / 27.9, 32 of 50 to 1010 22.4 / 23.8).
      if (s.aligned_shift >= 0 && two && lists >= 1 << kDecodeWgsShift && lists <= 1 << s.aligned_shift) {
        const int most = lists == 1 << kDecodeWgsShift ? (D == 64 ? 32 : 24) : lists > (7 << s.aligned_shift) / 8 ? 24 : 16;
        bool longer = false;
        each([&](int nb) __attribute__((always_inline)) { longer |= nb > most; });
        if (__builtin_amdgcn_ballot_w64(longer) == 0) {
          c.align = 5;
          c.round = 31;
          return;
        }
      }
      c.align = 0;
      c.shift = kDecodeWgsShift + (two ? 1 : 0);
      if (s.aligned_shift < 0) return;
      // Lists of one length that take a whole number of ranges each: no range has a seam, so they are cut evenly, and one
      // workgroup per CU is enough (8 lists of 4224 keys 29.6 / 29.4, 32 of 2048 50.9 / 47.3, 64 of 1000 at 28/4 heads 30.6 / 27.1)
      if ((lists & (lists - 1)) == 0 && lists <= 1 << c.shift) {
        blocks = __builtin_amdgcn_readlane(wave_inclusive_sum(blocks), 63);
        bool other = false;
        each([&](int nb) __attribute__((always_inline)) { other |= nb != 0 && (unsigned)nb * (unsigned)lists != (unsigned)blocks; });
        if (__builtin_amdgcn_ballot_w64(other) == 0) {
          if (lists <= 1 << kDecodeWgsShift) c.shift = kDecodeWgsShift;
          c.round = c.pad = 0;
          return;
        }
      }
      const bool beside = D == 128 && two;
      c.round = beside ? 1 : W - 1;
      c.pad = beside ? kSeam / 2 : kSeam;
    };
    if (s.aligned_shift < 0) share();
    for (;;) {
      int mine = 0;
      each([&](int nb) __attribute__((always_inline)) { mine += counted(c, nb); });
      r.incl = wave_inclusive_sum(s.pps * mine);
      c.total = __builtin_amdgcn_readlane(r.incl, 63);
      if (c.align == 0 || c.total <= 1 << (s.aligned_shift + c.align)) break;
      share();
    }
    if (c.align > 0) return c;
    // (lists that are not rounded up may have fewer blocks than there are workgroups: no range is empty, or it would be
    // counted among the parts of a list)
    while (c.shift > 0 && c.total >> c.shift == 0) --c.shift;
    return c;
  };
  if (__builtin_expect(r.run == 1, 1)) return take([&](auto f) __attribute__((always_inline)) { f(r.q.nb); });
  return take([&](auto f) __attribute__((always_inline)) {
    if (r.run * 64 <= kDecodeTable) {
      for (int j = 0; j < r.run; ++j) f(seq_at(s, table, r.run, lane, j).nb);
    } else {
      for (int j = 0; j < r.run && lane * r.run + j < s.batch; ++j) {
        bool bad = false;
        f(load_counted(s, lane * r.run + j, bad).nb);
        r.bad |= bad;
      }
    }
  });
}

// The sequence whose lists hold block x (x < total).
struct Place {
  int b, len, md;
  int begin;        // first block of its first pair
  int nb;           // blocks of a pair, as counted
  int real;         // ... that there are
};
__device__ __forceinline__ Place find_place(const SplitArgs& s, Cut c, const Lanes& r, int lane, const SeqTable* table, int x) {
  const int i = __builtin_amdgcn_readfirstlane(__builtin_popcountll(__builtin_amdgcn_ballot_w64(r.incl <= x)));   // whose lane
  if (__builtin_expect(r.run == 1, 1)) {
    const int real = __builtin_amdgcn_readlane(r.q.nb, i), nb = counted(c, real);
    return Place{i, __builtin_amdgcn_readlane(r.q.len, i), __builtin_amdgcn_readlane(r.q.md, i), __builtin_amdgcn_readlane(r.incl, i) - s.pps * nb, nb, real};
  }
  Place p = {0, 0, 1, 0, 1, 1};
  int base = i > 0 ? __builtin_amdgcn_readlane(r.incl, i - 1) : 0;
  for (int j0 = 0; j0 < r.run; j0 += 64) {
    Seq q = {0, 1, 0};
    if (j0 + lane < r.run && i * r.run + j0 + lane < s.batch) q = seq_at(s, table, r.run, i, j0 + lane);
    const int nb = counted(c, q.nb), incl = base + wave_inclusive_sum(s.pps * nb);
    const int end = __builtin_amdgcn_readlane(incl, 63);
    if (x < end) {                                          // wave-uniform
      const int j = __builtin_amdgcn_readfirstlane(__builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= x)));
      p.nb = __builtin_amdgcn_readlane(nb, j);
      p = Place{i * r.run + j0 + j, __builtin_amdgcn_readlane(q.len, j), __builtin_amdgcn_readlane(q.md, j), __builtin_amdgcn_readlane(incl, j) - s.pps * p.nb, p.nb, __builtin_amdgcn_readlane(q.nb, j)};
      break;
    }
    base = end;
  }
  return p;
}

// The cut as a table, for the merge kernel: entry b = (first block, blocks per pair) of sequence b; behind them, the cut.
__device__ __forceinline__ void write_cut_table(const SplitArgs& s, Cut c, int lane, int* table) {
  for (int b0 = 0, base = 0; b0 < s.batch; b0 += 64) {
    int nb = 0;
    if (b0 + lane < s.batch) {
      bool bad, sparse;
      int len, md, s_end, tail_start;
      load_seq(s, b0 + lane, len, md, bad);
      nb = blocks_of(s, seq_visible(s, len, md, bad, sparse, s_end, tail_start));
    }
    const int incl = wave_inclusive_sum(s.pps * counted(c, nb));
    if (b0 + lane < s.batch) {
      table[2 * (b0 + lane)] = base + incl - s.pps * counted(c, nb);
      table[2 * (b0 + lane) + 1] = nb;
    }
    base += __builtin_amdgcn_readlane(incl, 63);
  }
  if (lane == 0) {
    int* const t = table + 2 * s.batch;
    t[0] = c.total;
    t[1] = c.shift;
    t[2] = c.align;
    t[3] = c.round;
    t[4] = c.pad;
  }
}

// ---- rows that pass between workgroups of one launch, which may sit on different XCDs: written and read at device
// scope (past the L2s, which are not coherent with each other).  `base` is wave-uniform, `at` a byte offset.
__device__ __forceinline__ void store16_dev(float* base, int at, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00027000), at, 0, 16 /*sc1*/);
}
__device__ __forceinline__ f32x4 load16_dev(const float* base, int at) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00027000), at, 0, 16));
}
template <bool DEV>
__device__ __forceinline__ f32x2 load_ml(const float* p) {
  if (!DEV) return *(const f32x2*)p;
  return __builtin_bit_cast(f32x2, __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// ---- the merge of a pair's parts: out = sum_c w_c O_c / sum_c w_c l_c, w_c = exp(m_c - max m).  A wave takes 64 / (D / 4)
// heads at a time, D / 4 lanes each with four columns, and the parts in runs of 16: lane i of every 16 works out the weight
// of part i, which the sum over the parts then takes from it.  The rows of a run are all asked for at once.
template <int CTRL>
__device__ __forceinline__ float row16(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float sum16(float x) {           // over the 16 lanes of a row, the same in all of them
  x += row16<0x128>(x);                                     // row_ror:8, 4, 2, 1
  x += row16<0x124>(x);
  x += row16<0x122>(x);
  return x + row16<0x121>(x);
}
__device__ __forceinline__ float max16(float x) {
  x = fmaxf(x, row16<0x128>(x));
  x = fmaxf(x, row16<0x124>(x));
  x = fmaxf(x, row16<0x122>(x));
  return fmaxf(x, row16<0x121>(x));
}
template <int... I>
__device__ __forceinline__ void add_weighted(f32x4& num, float w, const f32x4 (&o)[16], std::integer_sequence<int, I...>) {
  ((num += row16<0x150 + I>(w) * o[I]), ...);               // row_newbcast:I, the weight of part I
}
struct Merged {
  float m, den;
  f32x4 num;
};
// Lane l's columns of head `head0` + l / (D / 4), over the runs first_run, first_run + step, ...
template <int D, bool DEV>
__device__ __forceinline__ Merged merge_runs(const float* part_o, const float* part_ml, int rpu, int first, int parts, int nq, float scale_log2, int head0, int first_run, int step, int l) {
  constexpr int TPR = D / 4;
  const int row = min(head0 + l / TPR, nq - 1), d = 4 * (l % TPR), j = l & 15;
  Merged r = {-INFINITY, 0.f, f32x4{0.f, 0.f, 0.f, 0.f}};
  for (int c0 = 16 * first_run; c0 < parts; c0 += 16 * step) {
    const f32x2 ml = load_ml<DEV>(part_ml + 2 * (part_place(first, min(c0 + j, parts - 1)) * rpu + row));
    f32x4 o[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int at = (part_place(first, min(c0 + i, parts - 1)) * rpu + row) * D + d;   // (the last part again where there are fewer)
      if (DEV) o[i] = load16_dev(part_o, at * 4);
      else o[i] = *(const f32x4*)(part_o + at);
    }
    const float mj = c0 + j < parts ? ml[0] : -INFINITY;
    const float m_new = fmaxf(r.m, max16(mj));
    const float al = fast_exp2((r.m - m_new) * scale_log2); // 0 for the first run (every part holds a key)
    const float w = fast_exp2((mj - m_new) * scale_log2);
    r.num *= al;
    r.den = r.den * al + sum16(w * ml[1]);
    r.m = m_new;
    add_weighted(r.num, w, o, std::make_integer_sequence<int, 16>());
  }
  return r;
}
// All heads of one pair by a workgroup of four waves; `store` is given (head, column, four values).  Where the heads take one
// or two waves and there are several runs, the other waves take every other run and all meet in LDS (Merged[4][64]).
template <int D, bool DEV, int W, class Store>
__device__ __forceinline__ void merge_pair(const float* part_o, const float* part_ml, int rpu, int first, int parts, int nq, float scale_log2, char* lds, int w, int l, Store store) {
  constexpr int TPR = D / 4, HPW = 64 / TPR;
  auto finish = [&](int head0, const Merged& r) __attribute__((always_inline)) {
    const int qi = head0 + l / TPR;
    if (qi < nq) store(qi, 4 * (l % TPR), f32x4{r.num[0] / r.den, r.num[1] / r.den, r.num[2] / r.den, r.num[3] / r.den});
  };
  const int groups = (nq + HPW - 1) / HPW;                  // of heads that a wave takes at a time
  const int split = groups > 2 || parts <= 16 ? 1 : 4 / groups;
  for (int i = w; i < groups * split; i += W) {
    const int head0 = (split == 1 ? i : i % groups) * HPW;
    const Merged r = merge_runs<D, DEV>(part_o, part_ml, rpu, first, parts, nq, scale_log2, head0, split == 1 ? 0 : i / groups, split, l);
    if (split == 1) finish(head0, r);
    else ((Merged*)lds)[64 * i + l] = r;
  }
  if (split == 1) return;                                   // uniform for the workgroup
  __syncthreads();
  if (w >= groups) return;
  float m = -INFINITY;
  for (int i = 0; i < split; ++i) m = fmaxf(m, ((Merged*)lds)[64 * (w + i * groups) + l].m);
  Merged t = {m, 0.f, f32x4{0.f, 0.f, 0.f, 0.f}};
  for (int i = 0; i < split; ++i) {
    const Merged r = ((Merged*)lds)[64 * (w + i * groups) + l];
    const float wgt = fast_exp2((r.m - m) * scale_log2);    // exp2(-inf) = 0 for a wave without runs
    t.num += wgt * r.num;
    t.den += wgt * r.den;
  }
  finish(w * HPW, t);
}

// FUSED: the call is a whole decode step of the layer (Sec. 3.3): it also appends the row k_new / v_new of every
// sequence at position kv_len[b].  The workgroup with the first block of a list stores the row in the cache; the
// workgroups that attend to it take it from k_new / v_new, so no read waits for that store.  The lengths are moved on by the
// last workgroup to have read them.
//
// IN_PLACE: the part that arrives last at its pair merges the pair.  Its rows pass between workgroups that may sit on
// different XCDs: they are written and read with device-scope accesses, and a part counts itself only after its own
// stores have been acknowledged.
//
// W: waves per workgroup, 4, or 8 in calls of few short lists (see DecodePlan): eight blocks of one list per workgroup, so that
// a wave has one block and no second wait for memory.
template <int D, bool NT, bool FUSED, bool IN_PLACE, int W = 4>
__global__ __launch_bounds__(64 * W, 2) void decode_splitk_kernel(DecodeArgs a) {
  constexpr int KC = D / 32;          // MFMA k-steps over the head dimension
  constexpr int DB = D / 16;          // 16-wide output blocks over the head dimension
  constexpr int VL = D / 16;          // 16-byte V loads per lane per 32-key block
  constexpr int CPR = D / 8;          // 16-byte chunks per row
  constexpr int VROW = D + 8;         // padded LDS row (elements)
  constexpr int RED = D + 4;          // floats from one row of the merge buffer to the next

  // V staging of the waves; at the end of a part the merge of the waves ([W][16][RED] floats and [W][16][2])
  constexpr int STAGING = W * 32 * VROW * 2, RED_BYTES = W * 16 * (RED + 2) * 4;
  __shared__ __attribute__((aligned(16))) char smem[STAGING > RED_BYTES ? STAGING : RED_BYTES];
  __shared__ int last_of_pair;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int g = l >> 4, n = l & 15;
  const int wg = blockIdx.x;

  // ---- the range of this workgroup
  __shared__ u32x2 s_seq[W == 8 ? kDecodeFewWgs : kDecodeTable];   // (a call of eight waves has no more sequences than workgroups)
  SeqTable* const seqs = (SeqTable*)s_seq;
  Lanes lanes;
  const Cut cut = find_cut<D, W>(a.sp, l, w, seqs, lanes);
  if constexpr (W == 8) __builtin_assume(cut.align > 0);
  if (wg == 0 && lanes.bad) atomicOr(a.status, (uint32_t)FLUX_DEV_BAD_LENGTH);
  // FUSED: the workgroups count themselves, first on one of kDecodeGather words (a word takes some 10 ns per count), when
  // all their waves hold the lengths; the one that completes the count moves the lengths on.  Called by one wave, in two
  // steps: the answer to the first count is not waited for until there is nothing else to do.  Few workgroups of eight waves
  // count themselves on one word, where their answers have the time (see below).
  const bool one_word = W == 8 && !lanes.merged && (int)gridDim.x <= kDecodeOneWord;   // (and no words to count)
  uint32_t counted = 0;
  auto count_in = [&]() __attribute__((always_inline)) {
    if (l == 0) counted = __hip_atomic_fetch_add(a.arrived + (one_word ? 0 : kCounterStride * (1 + (wg & (kDecodeGather - 1)))), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  bool counts_words = one_word;
  auto count_word = [&]() __attribute__((always_inline)) {  // whoever completes a word counts it
    if (one_word) return;
    const int x = wg & (kDecodeGather - 1), expected = ((int)gridDim.x - 1 - x) / kDecodeGather + 1;
    counts_words = __builtin_amdgcn_readfirstlane(counted) + 1 == (uint32_t)expected;
    if (counts_words && l == 0) {
      a.arrived[kCounterStride * (1 + x)] = 0;              // ready for the next call on this stream
      counted = __hip_atomic_fetch_add(a.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  auto move_lengths = [&]() __attribute__((always_inline)) {
    if (!counts_words || __builtin_amdgcn_readfirstlane(counted) + 1 != (uint32_t)(one_word ? (int)gridDim.x : min((int)gridDim.x, kDecodeGather))) return;
    for (int i = l; i < a.sp.batch; i += 64) {
      int len = a.kv_len_rw[i];
      len = len < 0 ? 0 : (len > a.sp.capacity ? a.sp.capacity : len);
      a.kv_len_rw[i] = len < a.sp.capacity ? len + 1 : len;
    }
    if (l == 0) a.arrived[0] = 0;
  };
  auto count_out = [&]() __attribute__((always_inline)) {
    count_word();
    move_lengths();
  };
  if (wg == (int)gridDim.x - 1) {
    if constexpr (!IN_PLACE) {
      // leaves the cut behind for the merge kernel, which then needs neither the lengths nor the scan
      if (w == 0) write_cut_table(a.sp, cut, l, a.table);
    }
  }
  // IN_PLACE: sequences without keys have no blocks, and their rows are zero: workgroup u writes those of sequences u, u +
  // gridDim.x, ... when it has nothing else to do (all of them written by one workgroup, in front of its range: 24 lists of 2000
  // keys among 104 empty ones 113 us, now 41; 8 of 4000 among 24 40 / 29).  FUSED: every list holds the appended row.
  auto zero_rows = [&]() __attribute__((always_inline)) {
    if constexpr (IN_PLACE && !FUSED) {
      if (__builtin_amdgcn_ballot_w64(lanes.run > 1 || (l < a.sp.batch && lanes.q.nb == 0)) == 0) return;
      for (int b = wg; b < a.sp.batch; b += (int)gridDim.x) {
        const int i = b / lanes.run, j = b - i * lanes.run;
        if ((lanes.run == 1 ? __builtin_amdgcn_readlane(lanes.q.nb, i) : seq_at(a.sp, seqs, lanes.run, i, j).nb) != 0) continue;
        const int64_t off = (int64_t)b * a.hq * D;
        for (int x = 8 * tid; x < a.hq * D; x += 8 * 64 * W) {
          const u32x4 zero = {0, 0, 0, 0};
          if (a.out_fp32) {
            *(u32x4*)((float*)a.out + off + x) = zero;
            *(u32x4*)((float*)a.out + off + x + 4) = zero;
          } else {
            *(u32x4*)((__bf16*)a.out + off + x) = zero;
          }
        }
      }
    }
  };
  if (wg >= cut_wgs(cut) || cut.total == 0) {         // nothing to do: uniform for the whole workgroup
    if constexpr (FUSED) {
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __syncthreads();                                      // every wave holds the lengths
      if (w == 0) {
        count_in();
        count_out();
      }
    }
    zero_rows();
    return;
  }
  int at = range_begin(cut, wg);
  const int range_end = range_begin(cut, wg + 1);
  Place place = find_place(a.sp, cut, lanes, l, seqs, at);
  const int rows_at = (at - place.begin);
  int pair = __builtin_amdgcn_readfirstlane((int)((float)rows_at / (float)place.nb));   // (put right below: the quotient may be off by one)
  pair -= pair * place.nb > rows_at ? 1 : 0;
  pair += (pair + 1) * place.nb <= rows_at ? 1 : 0;

  // ---- the part in work: blocks [x0, x1) of the list of (sequence place.b, pair)
  int x0, x1, c1, seam, seam_add, wrap_at, new_key;
  const __bf16 *kbase, *vbase, *knew, *vnew;
  const int ring_window = a.sp.win_blocks << a.sp.blk_shift;
  auto set_part = [&]() __attribute__((always_inline)) {
    const int kvh = a.qblocks == 1 ? pair : pair / a.qblocks;
    const int begin = place.begin + pair * place.nb;
    x0 = at - begin;
    x1 = min(place.real, range_end - begin);
    bool bad = false, sparse;
    int s_end, tail_start;
    c1 = seq_visible(a.sp, place.len, place.md, bad, sparse, s_end, tail_start);
    // list index p >= seam = s_end maps to key p + tail_start - s_end.  Ring store (s_end = sink_lim when sparse): that key sits
    // in row sink_lim + (key - sink_lim) % ring_window = p + ring0, less ring_window from p = wrap_at on
    seam = sparse ? s_end : 0x7FFFFFFF;
    seam_add = tail_start - s_end;
    wrap_at = 0x7FFFFFFF;
    if (a.sp.ring && sparse) {
      seam_add %= ring_window;
      wrap_at = s_end + ring_window - seam_add;
    }
    kbase = a.k + (int64_t)place.b * a.stride_b + (int64_t)kvh * a.stride_h;
    vbase = a.v + (int64_t)place.b * a.stride_b + (int64_t)kvh * a.stride_h;
    // FUSED: the appended row is position place.len - 1, the last key of every list (none when the cache was full).
    new_key = -1;
    if constexpr (FUSED) {
      knew = a.k_new + ((int64_t)place.b * a.hkv + kvh) * D;
      vnew = a.v_new + ((int64_t)place.b * a.hkv + kvh) * D;
      if (place.md & 2) new_key = place.len - 1;            // the sequence takes its row
      else if (x0 == 0 && pair == 0 && tid == 0) atomicOr(a.status, (uint32_t)FLUX_DEV_KV_OVERFLOW);
    }
  };
  set_part();

  auto key_of = [&](int p) __attribute__((always_inline)) -> int {
    p = min(p, c1 - 1);                                     // keep every address inside the list
    return p + (p >= seam ? seam_add : 0) - (p >= wrap_at ? ring_window : 0);
  };

  // A 32-key block whose keys are 32 consecutive cache rows (every block of an FA list, and all but the
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
  auto load_block = [&](int p0) __attribute__((always_inline)) {                           // p0 is wave-uniform
    const int r0 = key_of(p0);
    // (FUSED: the block that holds the appended row takes the per-lane path, where that row comes from k_new / v_new)
    const bool linear = c1 - p0 >= 32 && key_of(p0 + 31) - r0 == 31 && !(FUSED && new_key >= 0 && r0 + 31 >= new_key);
    if (linear) {
      const __bf16* kb0 = kbase + (int64_t)r0 * a.stride_t;
      const __bf16* vb0 = vbase + (int64_t)r0 * a.stride_t;
#pragma unroll
      for (int sb = 0; sb < 2; ++sb)
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) kreg[sb][kc] = ld((const u32x4*)(kb0 + 16 * sb * a.stride_t + k_lane + 32 * kc));
#pragma unroll
      for (int i = 0; i < VL; ++i) vreg[i] = ld((const u32x4*)(vb0 + i * RPL * a.stride_t + v_lane));
    } else {
      // all rows first, then all loads: a row worked out between two loads makes the second wait for the first
      const __bf16 *krow[2], *vrow[VL];
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        const int key = key_of(p0 + 16 * sb + n);
        krow[sb] = (FUSED && key == new_key ? knew : kbase + (int64_t)key * a.stride_t) + 8 * g;
      }
#pragma unroll
      for (int i = 0; i < VL; ++i) {
        const int key = key_of(p0 + (i * 64 + l) / CPR);
        vrow[i] = (FUSED && key == new_key ? vnew : vbase + (int64_t)key * a.stride_t) + (l % CPR) * 8;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int sb = 0; sb < 2; ++sb)
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) kreg[sb][kc] = ld((const u32x4*)(krow[sb] + 32 * kc));
#pragma unroll
      for (int i = 0; i < VL; ++i) vreg[i] = ld((const u32x4*)vrow[i]);
    }
  };

  FLUX_LDS __bf16* vs = (FLUX_LDS __bf16*)smem + w * 32 * VROW;

  // The first block of a part is asked for before anything else of it: the query rows (which the first scores wait
  // for as well) and the appended row (stored once the part has been streamed) follow behind it.  Asked for in front of
  // it they hold it up by a memory latency, and by far more in the workgroups that find the memory pipes full of the other
  // workgroups' blocks: the last ones of an 8 x 4224 key call began to stream 17 us into a launch of 25.
  int p0, p_end;
  bf16x8 qf[KC];
  u32x4 new_row = {0, 0, 0, 0};
  FLUX_GLOBAL __bf16* new_row_at = nullptr;                 // where this thread's piece of the appended row goes
  auto begin_part = [&]() __attribute__((always_inline)) {
    // the part's keys, 32 at a time round the waves: p_end is where they end or the list does
    p0 = (int)min((int64_t)x0 << a.sp.block_shift, (int64_t)c1) + 32 * w;
    p_end = (int)min((int64_t)x1 << a.sp.block_shift, (int64_t)c1);
    if (W == 4 && p0 < p_end) load_block(p0);               // (eight waves have so little in flight that the order is free:
    __builtin_amdgcn_sched_barrier(0);                      // 1 x 144 keys 6.7 us so, 6.6 with the queries first)
    // ---- Q operand: lane (n, g) holds d = 32*kc + 8*g .. +7 of query head kvh*group + 16*qb + n (columns past the group's
    // last head repeat its first one; what they give is left out at the end)
    const int kvh = a.qblocks == 1 ? pair : pair / a.qblocks, qb = a.qblocks == 1 ? 0 : pair % a.qblocks;
    const int qh = 16 * qb + n;
    const __bf16* qrow = a.q + ((int64_t)place.b * a.hq + (int64_t)kvh * a.group + (qh < a.group ? qh : 0)) * D;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) qf[kc] = *(const bf16x8*)(qrow + 32 * kc + 8 * g);
    if constexpr (W == 8) {
      __builtin_amdgcn_sched_barrier(0);
      if (p0 < p_end) load_block(p0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (FUSED) {
      new_row_at = nullptr;
      if (x0 == 0 && qb == 0 && new_key >= 0 && tid < 2 * CPR) {
        new_row = *(const u32x4*)((tid < CPR ? knew : vnew) + 8 * (tid % CPR));
        new_row_at = (FLUX_GLOBAL __bf16*)const_cast<__bf16*>(tid < CPR ? kbase : vbase) + (int64_t)new_key * a.stride_t + 8 * (tid % CPR);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  begin_part();
  // Eight waves: nothing reads the lengths behind here, so workgroups with a whole list count themselves while its keys are on
  // their way (3 x 144 keys 7.4 us counted at the end, 7.0 so).  The others do it at the end, where they wait for their rows anyway
  // (1 x 2001 9.8 counted there, 10.1 here).
  if constexpr (FUSED && W == 8) {
    if (x0 == 0 && x1 == place.real) {
      __builtin_amdgcn_s_barrier();                         // every wave holds the lengths
      if (w == W - 1) count_in();
    }
  }

  for (;;) {
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 o[DB];
#pragma unroll
    for (int i = 0; i < DB; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    while (p0 < p_end) {
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
      const int pnext = W == 4 && p_end - p0 > 32 * W ? p0 + 32 * W : p_end;   // (of eight waves, each has one block at most)
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
      if (W == 4 && pnext < p_end) load_block(pnext);
      __builtin_amdgcn_sched_barrier(0);
      if (c1 - p0 < 32) {
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
      const float m_new = fmaxf(m_run, mloc);               // finite: the block holds a valid key
      const float alpha = fast_exp2((m_run - m_new) * a.scale_log2);
      const float mneg = -m_new * a.scale_log2;
      m_run = m_new;
      // Each weight goes to the matrix cores as the sum of two bf16 values, its upper bits and what they leave of it (to
      // 2^-16 of the weight).  Rounded to one bf16 value the result would depend on how a list is cut: the weight of the key
      // that sets a wave's reference is exactly 1, so every wave more has another of the heaviest keys exact.  The matrix
      // cores are idle for most of the time that a block takes to arrive (no call takes longer for it; relative error at 8 x 4224
      // keys and fp32 output 1.35e-3 with one bf16 value, 4.0e-6 with two).  (The second term is never 0, nor so small
      // that its bf16 value is: an infinite V row stays infinite where the first term is not 0.)
      uint32_t pk[4], rest[4];
      float psum = 0.f;
#pragma unroll
      for (int sb = 0; sb < 2; ++sb)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float pa = fast_exp2(__builtin_fmaf(s[sb][2 * i], a.scale_log2, mneg));
          const float pb = fast_exp2(__builtin_fmaf(s[sb][2 * i + 1], a.scale_log2, mneg));
          const uint32_t hi = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, pb), __builtin_bit_cast(uint32_t, pa), 0x07060302u);
          pk[2 * sb + i] = hi;
          rest[2 * sb + i] = pack_bf16(fmaxf(pa - bf16_lo(hi), 0x1p-126f), fmaxf(pb - bf16_hi(hi), 0x1p-126f));
          psum += pa + pb;
        }
      l_run = l_run * alpha + psum;
      const bf16x8 pf = __builtin_bit_cast(bf16x8, u32x4{pk[0], pk[1], pk[2], pk[3]});
      const bf16x8 pr = __builtin_bit_cast(bf16x8, u32x4{rest[0], rest[1], rest[2], rest[3]});
      // ---- O^T += V^T P^T
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        o[db] *= alpha;
        FLUX_LDS __bf16* src = vs + (4 * g + (n >> 2)) * VROW + 16 * db + 4 * (n & 3);
        const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((FLUX_LDS bf16x4*)src);
        const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((FLUX_LDS bf16x4*)(src + 16 * VROW));
        const bf16x8 vf = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
        o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o[db], 0, 0, 0);
        o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pr, o[db], 0, 0, 0);
      }
      p0 = pnext;
    }
    if (FUSED && new_row_at) *(FLUX_GLOBAL u32x4*)new_row_at = new_row;

    // Nothing is in flight any more, which the compiler does not see for a wave without blocks: it would wait for the next
    // part's keys in front of the next part's query rows.
    __builtin_amdgcn_s_waitcnt(0x0F70);                     // vmcnt(0)
    // (the arguments that only the end of a part needs are read again here: kept in scalar registers they push the loop's
    // values out of them)
    const FLUX_CONSTANT DecodeArgs* e = (const FLUX_CONSTANT DecodeArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    if constexpr (W == 4) asm volatile("" : "+s"(e));
    // ---- what the end of this part needs, and on to the next one: its first block is in flight meanwhile
    const int nq = min(16, e->group - (e->qblocks == 1 ? 0 : 16 * (pair % e->qblocks)));
    const int64_t out0 = ((int64_t)place.b * e->hq + (int64_t)(e->qblocks == 1 ? pair : pair / e->qblocks) * e->group + (e->qblocks == 1 ? 0 : 16 * (pair % e->qblocks))) * D;
    const int list0 = place.begin + pair * place.nb;
    const bool empty = x0 >= x1;                            // (the range begins in what is only counted behind a list)
    const bool whole = empty || (x0 == 0 && x1 == place.real);   // the pair lies in this range
    const int first = whole ? wg : range_of(cut, list0);
    const int parts = whole ? 1 : range_of(cut, list0 + place.real - 1) - first + 1;
    at = x1 < place.real ? range_end : list0 + place.nb;
    const bool more = W == 4 && at < range_end;
    if (more) {
      if (++pair == a.sp.pps) {
        place = find_place(a.sp, cut, lanes, l, seqs, place.begin + a.sp.pps * place.nb);   // (the next one that has keys)
        pair = 0;
      }
      set_part();
      begin_part();
    }

    // ---- merge the waves through LDS: red[w][n][0..D-1] = O, ml[w][n] = (m, l); only the columns of heads that exist
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    __syncthreads();                                        // every wave is done with its V staging
    FLUX_LDS float* red = (FLUX_LDS float*)smem;
    FLUX_LDS f32x2* ml = (FLUX_LDS f32x2*)(red + W * 16 * RED);
    if (n < nq) {
      FLUX_LDS float* mine = red + (w * 16 + n) * RED + 4 * g;
#pragma unroll
      for (int db = 0; db < DB; ++db) *(FLUX_LDS f32x4*)(mine + 16 * db) = o[db];
      if (g == 0) ml[w * 16 + n] = f32x2{m_run, l_run};
    }
    __syncthreads();
    auto store_out = [&](int qi, int d, f32x4 r) __attribute__((always_inline)) {
      const int64_t off = out0 + qi * D + d;
      if (e->out_fp32) *(f32x4*)((float*)e->out + off) = r;
      else *(u32x2*)((__bf16*)e->out + off) = u32x2{pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3])};
    };
    const int row0 = part_place(first, wg - first) * e->rpu;
    for (int idx = tid; !empty && idx < nq * (D / 4); idx += 64 * W) {
      const int qi = idx / (D / 4), d = 4 * (idx % (D / 4));
      f32x2 x[W];
      float m = -INFINITY;
#pragma unroll
      for (int ww = 0; ww < W; ++ww) {
        x[ww] = ml[ww * 16 + qi];
        m = fmaxf(m, x[ww][0]);
      }
      f32x4 val = {0.f, 0.f, 0.f, 0.f};
      float den = 0.f;
#pragma unroll
      for (int ww = 0; ww < W; ++ww) {
        const float wgt = fast_exp2((x[ww][0] - m) * e->scale_log2);        // exp2(-inf) = 0 for idle waves
        val += wgt * *(FLUX_LDS f32x4*)(red + (ww * 16 + qi) * RED + d);
        den += wgt * x[ww][1];
      }
      if (whole) {                                          // nothing to merge with
        store_out(qi, d, f32x4{val[0] / den, val[1] / den, val[2] / den, val[3] / den});
      } else if constexpr (IN_PLACE) {
        store16_dev(e->part_o, ((row0 + qi) * D + d) * 4, val);
        if (d == 0) __hip_atomic_store((unsigned long long*)(e->part_ml + 2 * (row0 + qi)), __builtin_bit_cast(unsigned long long, f32x2{m, den}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        *(f32x4*)(e->part_o + (row0 + qi) * D + d) = val;
        if (d == 0) *(f32x2*)(e->part_ml + 2 * (row0 + qi)) = f32x2{m, den};
      }
    }
    const bool counts = FUSED && !more && w == W - 1;
    if (counts && (W == 4 || !whole)) count_in();                       // (every wave of the workgroup has read the lengths)
    if (IN_PLACE && !whole) {
      // ---- the part that arrives last merges the pair
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's rows have reached the point all XCDs see
      __syncthreads();
      if (tid == 0) {
        uint32_t* count = e->arrived + kCounterStride * (1 + kDecodeGather + first);   // (a range holds the beginning of one unfinished pair at most)
        const bool done = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(parts - 1);
        if (done) *count = 0;                               // ready for the next call on this stream
        last_of_pair = done;
      }
      __syncthreads();
      if (counts) count_out();
      if (last_of_pair) merge_pair<D, true, W>(e->part_o, e->part_ml, e->rpu, first, parts, nq, e->scale_log2, smem, w, l, store_out);
    }
    if (counts && whole) count_out();
    if (!more) break;
    __syncthreads();                                        // the merge buffer becomes V staging again
  }
  zero_rows();
}

// The merge of a pair's parts as a launch of its own, one workgroup per (KV head, query block) and sequence.
struct CombineArgs {
  SplitArgs sp;
  const float* part_o;
  const float* part_ml;
  const int* table;       // the cut the first kernel took (see write_cut_table)
  int hq, group, qblocks, rpu, out_fp32;
  float scale_log2;
  void* out;
};

template <int D>
__global__ __launch_bounds__(256) void decode_combine_kernel(CombineArgs a) {
  __shared__ __attribute__((aligned(16))) char smem[4 * 64 * sizeof(Merged)];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, pair = blockIdx.x, b = blockIdx.y;
  const int kvh = pair / a.qblocks, qb = pair - kvh * a.qblocks;
  const int nq = min(16, a.group - 16 * qb);
  const int nb = a.table[2 * b + 1];
  const int64_t out0 = ((int64_t)b * a.hq + (int64_t)kvh * a.group + 16 * qb) * D;
  auto store_out = [&](int qi, int d, f32x4 r) __attribute__((always_inline)) {
    const int64_t off = out0 + qi * D + d;
    if (a.out_fp32) *(f32x4*)((float*)a.out + off) = r;
    else *(u32x2*)((__bf16*)a.out + off) = u32x2{pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3])};
  };
  if (nb == 0) {                                            // an empty cache yields zeros
    for (int it = tid; it < nq * (D / 4); it += 256) store_out(it / (D / 4), 4 * (it % (D / 4)), f32x4{0.f, 0.f, 0.f, 0.f});
    return;
  }
  const int* const t = a.table + 2 * a.sp.batch;
  const Cut cut = {t[0], t[1], t[2], t[3], t[4]};
  const int begin = a.table[2 * b] + pair * counted(cut, nb);
  const int first = range_of(cut, begin), parts = range_of(cut, begin + nb - 1) - first + 1;
  if (parts < 2) return;                                    // done by the first kernel
  merge_pair<D, false, 4>(a.part_o, a.part_ml, a.rpu, first, parts, nq, a.scale_log2, smem, w, l, store_out);
}

// c.decode_counters may be null: the call then takes two launches.
hipError_t launch_decode(const Ctx& c, const flux_attn_cfg& cfg, const void* q, int max_kv_len,
                         const flux_kv_cache& cache, const uint8_t* mode, int ring, const void* k_new,
                         const void* v_new, void* out, hipStream_t s) {
  const bool fused = k_new != nullptr;                       // append + attend + merge in one launch (needs the counters)
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
  a.sp.block_shift = plan.block_shift;
  a.sp.aligned_shift = plan.aligned_shift;
  a.sp.most_by_four = plan.most_by_four;
  a.k_new = (const __bf16*)k_new;
  a.v_new = (const __bf16*)v_new;
  a.hq = cfg.n_q_heads;
  a.hkv = cfg.n_kv_heads;
  a.group = cfg.n_q_heads / cfg.n_kv_heads;
  a.qblocks = (a.group + 15) / 16;
  a.rpu = plan.rpu;
  a.scale_log2 = scale * kLog2e;
  a.table = (int*)c.partials;                                // (calls of two launches only)
  const bool two_launches = !c.decode_counters;
  a.part_o = two_launches || plan.in_partials ? c.partials + decode_rows_at(plan, two_launches) : c.small;
  a.part_ml = a.part_o + (size_t)2 * plan.wgs * plan.rpu * cfg.head_dim;
  a.status = c.status;
  a.arrived = c.decode_counters;
  a.kv_len_rw = cache.kv_len;
  a.out = out;
  a.out_fp32 = cfg.out_dtype;
  const dim3 grid(plan.wgs);
  // K and V bytes one call may read.  A call of a model whose layers together stream more than the 256 MB last-level
  // cache finds none of its rows there, whatever its own size (an SA layer reads 138 MB of a 4 GB cache): from 64 MB
  // on the rows are fetched with nontemporal loads (SA layer 34.5 -> 33.4 us, FA layers as before); smaller calls are
  // bound by their launches either way.
  const bool nt = 4.0 * cache.batch * cfg.n_kv_heads * cfg.head_dim * (double)max_kv_len > 64.0 * 1024 * 1024;
  auto launch = [&](auto d) {
    constexpr int D = decltype(d)::value;
    if (plan.waves == 8) {                                   // (64 MB at most)
      if (fused) hipLaunchKernelGGL((decode_splitk_kernel<D, false, true, true, 8>), grid, dim3(512), 0, s, a);
      else if (c.decode_counters) hipLaunchKernelGGL((decode_splitk_kernel<D, false, false, true, 8>), grid, dim3(512), 0, s, a);
      else hipLaunchKernelGGL((decode_splitk_kernel<D, false, false, false, 8>), grid, dim3(512), 0, s, a);
    } else if (fused) {
      if (nt) hipLaunchKernelGGL((decode_splitk_kernel<D, true, true, true>), grid, dim3(256), 0, s, a);
      else hipLaunchKernelGGL((decode_splitk_kernel<D, false, true, true>), grid, dim3(256), 0, s, a);
    } else if (c.decode_counters) {
      if (nt) hipLaunchKernelGGL((decode_splitk_kernel<D, true, false, true>), grid, dim3(256), 0, s, a);
      else hipLaunchKernelGGL((decode_splitk_kernel<D, false, false, true>), grid, dim3(256), 0, s, a);
    } else {
      if (nt) hipLaunchKernelGGL((decode_splitk_kernel<D, true, false, false>), grid, dim3(256), 0, s, a);
      else hipLaunchKernelGGL((decode_splitk_kernel<D, false, false, false>), grid, dim3(256), 0, s, a);
    }
  };
  if (cfg.head_dim == 128) launch(std::integral_constant<int, 128>());
  else launch(std::integral_constant<int, 64>());
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || c.decode_counters) return e;

  CombineArgs ca;
  ca.sp = a.sp;
  ca.part_o = a.part_o;
  ca.part_ml = a.part_ml;
  ca.table = a.table;
  ca.hq = cfg.n_q_heads;
  ca.group = a.group;
  ca.qblocks = a.qblocks;
  ca.rpu = plan.rpu;
  ca.out_fp32 = cfg.out_dtype;
  ca.scale_log2 = a.scale_log2;
  ca.out = out;
  const dim3 cgrid(plan.pps, cache.batch);
  if (cfg.head_dim == 128) hipLaunchKernelGGL(decode_combine_kernel<128>, cgrid, dim3(256), 0, s, ca);
  else hipLaunchKernelGGL(decode_combine_kernel<64>, cgrid, dim3(256), 0, s, ca);
  return hipGetLastError();
}

}  // namespace flux
