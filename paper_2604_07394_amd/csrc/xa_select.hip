// flux_xa_select: the key blocks each query block of a prompt keeps under the XA sparse mode (Sec. 4.1; Table 3:
// stride 16, threshold 0.9, selection mode "Inverse", block 64), written as the keep matrix that
// flux_attn_prefill_blocksparse consumes.  The paper names the method ("Block Sparse Attention with
// Antidiagonal Scoring") and its parameters only; what is computed is this reading of them:
//
//   1. The scaled score matrix of one head is cut into squares of 16 x 16 positions.  Of square (a, b) only the
//      antidiagonal is looked at (query row offset r against key column offset 15 - r: the rows taken in inverse
//      order against the columns), and of it only the causal samples inside the prompt; e[a][b] is their mean.
//   2. Every row a of e becomes probabilities over its squares b <= a by a softmax.
//   3. The mass of block pair (I, J) is the sum of those probabilities over its 4 x 4 squares divided by the rows
//      of e the query block has; the masses of a query block sum to one.
//   4. Query block I keeps every key block whose mass is at least that of the block at which the masses, taken
//      in descending order, first reach the threshold; and always its own block.
//
// Step 1 is a matrix product over 16 * D numbers per square: the 16 query rows of square row a laid end to end
// against the 16 key rows of square column b laid end to end in inverse order.  Short prompts (and contexts with a tiny
// workspace) take the walk described here, all others the tiled form further down.  One workgroup owns 32 square
// rows (512 queries, 8 query blocks) of one head and walks the square columns 16 at a time (256 keys):
//   - the contraction is split over the four waves by the row offset r (wave w takes r = 4w .. 4w+3), so each
//     wave keeps its share of the query operand in registers for the whole kernel and loads only its share of
//     every key tile, straight from global memory in MFMA operand layout (16x16x32 bf16, S^T = K Q^T); a key
//     fragment is used for both halves of the 32 square rows (the kernel is bound by the rate at which key rows
//     reach the CUs, so every use of a fragment counts), and the next tile is asked for once the MFMAs have
//     taken this tile's registers;
//   - the four partial 32 x 16 tiles meet in LDS, where thread (a, b) adds them in wave order.  On the diagonal
//     the samples r < 8 are not causal: exactly the partial tiles of waves 0 and 1, which are left out there;
//     positions past the prompt are zeroed in the operands, and the number of samples of a square is a closed form;
//   - the softmax over a row of squares needs the row's maximum and sum, which are known only at the end of the
//     row.  Prompts of up to 65536 positions are walked once: of every (square row, key block) the logarithm of
//     the summed exponentials of its 4 squares is kept in LDS (it needs no reference), and when the row's
//     log-sum-exp is known the masses are the exponentials of the differences, summed over the 4 rows of a query
//     block.  Longer prompts (the table would not fit) are walked twice: once for (max, sum), once for the
//     probabilities, which are summed 4 x 4 into the masses (a wave of the reduction phase holds the 4 square rows
//     of one query block);
//   - the threshold is found without sorting: the largest mass value t with sum(mass >= t) >= threshold * total,
//     by bisection over the bit patterns of the positive floats (32 steps, one row reduction each).
#include <type_traits>

#include "flux_internal.h"

namespace flux {

struct XaArgs {
  const __bf16* q;        // [T, Hq, D]
  const int32_t* cu_q;    // [B + 1]
  const __bf16* k;
  int64_t stride_b, stride_h, stride_t;   // elements
  const int32_t* kv_len;
  int capacity;
  int hq, group, batch;
  int n_groups;           // workgroups per (sequence, head): groups of 8 query blocks
  float scale;            // softmax scale (not in log2 units)
  float threshold;
  uint8_t* mask;          // [B, Hq, n_qblocks, n_kblocks]
  int n_qblocks, n_kblocks;
  int tab_cols;           // key blocks the host's bound on the prompt length allows (<= n_kblocks): the width of the LDS tables
  int single_walk;        // the (square row, key block) table fits LDS: one walk over the keys
  uint32_t* status;
};

constexpr int kXaRows = 32;        // square rows per workgroup (512 queries): two halves of 16, the N of one MFMA
constexpr int kXaStride = 16;      // positions per square side (Table 3: stride 16)

template <int D>
__global__ __launch_bounds__(256, 2) void xa_select_kernel(XaArgs a) {
  constexpr int ST = D / 8;        // k-steps of 32 numbers per wave: 4 row offsets x D / 32
  constexpr int SPR = D / 32;      // k-steps per row offset
  extern __shared__ __attribute__((aligned(16))) char xa_smem[];
  float* part = (float*)xa_smem;                       // [2 buffers][4 waves][32 a][16 b]
  float* mass = part + 2 * 4 * 512;                    // [8 query blocks][tab_cols]; one walk: [32 square rows][tab_cols]
  float* lse = part;                                   // one walk: log-sum-exp of every square row, kept where the partial
                                                       // tiles were once the walk is over (two workgroups of a 32768-token
                                                       // prompt then fit the LDS of a CU exactly)
  const bool single = a.single_walk != 0;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int g = l >> 4, nn = l & 15;
  // ---- which (sequence, head, group of 8 query blocks) this workgroup owns.  Workgroups go to the 8 XCDs round-robin
  // by linear id and every XCD has its own L2: all heads and groups that read one (sequence, KV head) pair get ids of
  // one residue mod 8, longest walks first and the heads of a GQA group next to each other, so that the workgroups
  // resident on an XCD walk the same key rows at about the same time and the rows reach that L2 once.
  int grp, h, b;
  {
    const int i = blockIdx.x;
    const int hkv = a.hq / a.group, n_pairs = a.batch * hkv;
    if ((n_pairs & 7) == 0) {
      const int x = i & 7, j = i >> 3;
      // (the XCD's pairs one after the other, not interleaved group by group: the groups past a short sequence's end
      // are empty workgroups, and at fixed places of a short period they would keep falling to the same CUs)
      const int r = j / (a.group * a.n_groups), gd = (j / a.group) % a.n_groups, gh = j % a.group;
      const int pair = x + 8 * r;
      b = pair / hkv;
      h = (pair % hkv) * a.group + gh;
      grp = a.n_groups - 1 - gd;
    } else {
      grp = a.n_groups - 1 - i % a.n_groups;
      h = (i / a.n_groups) % a.hq;
      b = i / (a.n_groups * a.hq);
    }
  }
  const int kvh = h / a.group;

  const int q_begin = a.cu_q[b];
  const int n_q = a.cu_q[b + 1] - q_begin;
  int len = a.kv_len[b];
  // the selection is defined for a whole prompt: as many queries as cached positions
  if (grp == 0 && h == 0 && tid == 0 && (len < 0 || len > a.capacity || n_q != len)) atomicOr(a.status, (uint32_t)FLUX_DEV_BAD_LENGTH);
  len = len < 0 ? 0 : (len > a.capacity ? a.capacity : len);
  int n = n_q < len ? (n_q < 0 ? 0 : n_q) : len;         // positions 0 .. n-1 are scored
  if (n > 64 * a.tab_cols) {                             // a prompt longer than the host's bound: cut there, and say so
    if (grp == 0 && h == 0 && tid == 0) atomicOr(a.status, (uint32_t)FLUX_DEV_BAD_LENGTH);
    n = 64 * a.tab_cols;
  }
  const int a0 = grp * kXaRows;                          // first square row of the workgroup
  uint8_t* mrow0 = a.mask + (((int64_t)b * a.hq + h) * a.n_qblocks + 8 * grp) * (int64_t)a.n_kblocks;
  const int n_sq = (n + kXaStride - 1) / kXaStride;      // square rows / columns of the prompt
  if (a0 >= n_sq) {                                      // nothing to score: the rows of the matrix are cleared
    for (int qb = 0; qb < 8; ++qb)
      if (8 * grp + qb < a.n_qblocks)
        for (int j = tid; j < a.n_kblocks; j += 256) mrow0[(int64_t)qb * a.n_kblocks + j] = 0;
    return;
  }
  const int a_last = min(a0 + kXaRows, n_sq) - 1;        // last existing square row of the workgroup
  const int n_ct = a_last / 16 + 1;                      // column tiles (16 square columns each) to walk

  // ---- query operand of this wave: lane (nn, g) holds, for half ah and k-step st, 8 numbers of query row
  // 16*(a0 + 16*ah + nn) + r, r = 4w + st / SPR, d = 32 * (st % SPR) + 8g; rows past the prompt are zero
  bf16x8 qf[2][ST];
  {
    const u32x4 zero = {0, 0, 0, 0};
#pragma unroll
    for (int ah = 0; ah < 2; ++ah)
#pragma unroll
      for (int st = 0; st < ST; ++st) {
        const int r = 4 * w + st / SPR, d = 32 * (st % SPR) + 8 * g;
        const int pos = kXaStride * (a0 + 16 * ah + nn) + r;
        const int pc = pos < n ? pos : (n > 0 ? n - 1 : 0);
        const u32x4 t = *(const u32x4*)(a.q + ((int64_t)(q_begin + pc) * a.hq + h) * D + d);
        qf[ah][st] = __builtin_bit_cast(bf16x8, pos < n ? t : zero);
      }
  }
  const __bf16* kbase = a.k + (int64_t)b * a.stride_b + (int64_t)kvh * a.stride_h;

  // One column tile: the key operand of this wave is fetched one tile ahead (the fetch of tile ct + 1 is issued
  // right behind the products of tile ct, into the registers they have just read, so the rest of a tile's work
  // covers its latency); partial sums go to part[buf][w].
  // Keys past the prompt (only the last tile can hold any) are fetched from a clamped address and zeroed when
  // they are used, not when they are fetched: a select behind the load would wait for it at once.
  u32x4 kreg[ST];
  auto key_of = [&](int ct, int st) __attribute__((always_inline)) { return kXaStride * (16 * ct + nn) + (kXaStride - 1) - (4 * w + st / SPR); };
  auto fetch_tile = [&](int ct) __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < ST; ++st) {
      const int key = key_of(ct, st);                        // key row of square column 16*ct + nn, inverse order
      const int kc = key < n ? key : (n > 0 ? n - 1 : 0);
      kreg[st] = *(const u32x4*)(kbase + (int64_t)kc * a.stride_t + 32 * (st % SPR) + 8 * g);
    }
  };
  auto partial_tile = [&](int ct, int buf) __attribute__((always_inline)) {
    if (256 * (ct + 1) > n) {                                // uniform: this tile reaches past the prompt
      const u32x4 zero = {0, 0, 0, 0};
#pragma unroll
      for (int st = 0; st < ST; ++st) kreg[st] = key_of(ct, st) < n ? kreg[st] : zero;
    }
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int st = 0; st < ST; ++st)
#pragma unroll
      for (int ah = 0; ah < 2; ++ah)
        acc[ah] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kreg[st]), qf[ah][st], acc[ah], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (ct + 1 < n_ct) fetch_tile(ct + 1);
    __builtin_amdgcn_sched_barrier(0);
    // acc[ah][i] = square (a0 + 16*ah + nn, 16*ct + 4g + i): stored as part[a][b]
#pragma unroll
    for (int ah = 0; ah < 2; ++ah) *(f32x4*)(part + ((buf * 4 + w) * 32 + 16 * ah + nn) * 16 + 4 * g) = acc[ah];
  };
  // the reduction phase: thread (ra, rb) of the workgroup owns the squares (a0 + 16*ah + ra, 16*ct + rb), ah = 0, 1
  const int ra = tid >> 4, rb = tid & 15;
  auto square_value = [&](int ct, int buf, int ah) __attribute__((always_inline)) -> float {
    const int a_abs = a0 + 16 * ah + ra;
    const int b_abs = 16 * ct + rb;
    if (a_abs > a_last || b_abs > a_abs) return -INFINITY;               // no such square
    const int r_min = max(max(b_abs == a_abs ? 8 : 0, kXaStride * b_abs + kXaStride - n), 0);
    const int r_max = min(kXaStride - 1, n - 1 - kXaStride * a_abs);
    const int cnt = r_max - r_min + 1;
    if (cnt <= 0) return -INFINITY;
    const float* p = part + (buf * 4 * 32 + 16 * ah + ra) * 16 + rb;
    // on the diagonal the samples r < 8 (waves 0 and 1) are not causal
    const float lo = b_abs == a_abs ? 0.f : p[0] + p[512];
    const float sum = lo + (p[1024] + p[1536]);
    return a.scale * sum / (float)cnt;
  };

  // ---- first walk: maximum and sum of every row of squares (the 16 lanes rb = 0..15 of a row agree on both)
  float m_row[2] = {-INFINITY, -INFINITY}, l_row[2] = {0.f, 0.f};
  auto first_walk = [&](int ct) __attribute__((always_inline)) {
    const int buf = ct & 1;
    partial_tile(ct, buf);
    __syncthreads();
#pragma unroll
    for (int ah = 0; ah < 2; ++ah) {
      const float e = square_value(ct, buf, ah);
      float mt = e;
      mt = fmaxf(mt, __shfl_xor(mt, 1));
      mt = fmaxf(mt, __shfl_xor(mt, 2));
      mt = fmaxf(mt, __shfl_xor(mt, 4));
      mt = fmaxf(mt, __shfl_xor(mt, 8));
      const float m_new = fmaxf(m_row[ah], mt);
      float pe = e == -INFINITY ? 0.f : __expf(e - m_new);
      pe += __shfl_xor(pe, 1);
      pe += __shfl_xor(pe, 2);
      if (single && (rb & 3) == 0) {                                    // the 4 squares of one key block, reference-free
        const int kbk = 4 * ct + (rb >> 2);
        if (kbk < a.tab_cols) mass[(16 * ah + ra) * a.tab_cols + kbk] = pe > 0.f ? m_new + __logf(pe) : -INFINITY;
      }
      pe += __shfl_xor(pe, 4);
      pe += __shfl_xor(pe, 8);
      l_row[ah] = (m_row[ah] == -INFINITY ? 0.f : l_row[ah] * __expf(m_row[ah] - m_new)) + pe;
      m_row[ah] = m_new;
    }
  };
  fetch_tile(0);
  for (int ct = 0; ct < n_ct; ++ct) first_walk(ct);
  // ---- second walk: probabilities, summed 4 x 4 into block masses.  Wave wv of this phase holds the square rows
  // 16*ah + 4wv .. + 3 (query block 8*grp + 4*ah + wv); a key block is 4 adjacent square columns.
  int rows_in_block[2];                                               // rows of e this wave's query blocks have
#pragma unroll
  for (int ah = 0; ah < 2; ++ah) rows_in_block[ah] = min(4, n_sq - (a0 + 16 * ah + 4 * w));
  auto second_walk = [&](int ct) __attribute__((always_inline)) {
    const int buf = ct & 1;
    partial_tile(ct, buf);
    __syncthreads();
#pragma unroll
    for (int ah = 0; ah < 2; ++ah) {
      const float e = square_value(ct, buf, ah);
      float p = (e == -INFINITY || l_row[ah] == 0.f) ? 0.f : __expf(e - m_row[ah]) / l_row[ah];
      p += __shfl_xor(p, 1);                                          // over the 4 square columns of a key block
      p += __shfl_xor(p, 2);
      p += __shfl_xor(p, 16);                                         // over the 4 square rows of the query block
      p += __shfl_xor(p, 32);
      if ((l & 0x33) == 0 && rows_in_block[ah] > 0) {
        const int kbk = 4 * ct + (rb >> 2);
        if (kbk < a.tab_cols) mass[(4 * ah + w) * a.tab_cols + kbk] = p / (float)rows_in_block[ah];
      }
    }
  };
  __syncthreads();                                                    // the first walk's last readers are done
  if (!single) {
    fetch_tile(0);
    for (int ct = 0; ct < n_ct; ++ct) second_walk(ct);
  } else if (rb == 0) {
#pragma unroll
    for (int ah = 0; ah < 2; ++ah) lse[16 * ah + ra] = m_row[ah] + __logf(l_row[ah]);
  }
  __syncthreads();

  // ---- selection: wave w owns the query blocks 8*grp + w and 8*grp + 4 + w and their masses of key blocks 0 .. own
  const int n_blk = (n + 63) / 64;
  auto wave_sum = [&](float x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    return x;
  };
  for (int ah = 0; ah < 2; ++ah) {
    const int qi = 4 * ah + w;
    const int qb_abs = 8 * grp + qi;
    if (qb_abs >= a.n_qblocks) continue;
    uint8_t* mrow = mrow0 + (int64_t)qi * a.n_kblocks;
    if (qb_abs >= n_blk) {                                            // a row of the matrix beyond the prompt
      for (int j = l; j < a.n_kblocks; j += 64) mrow[j] = 0;
      continue;
    }
    const int nj = min(qb_abs + 1, a.tab_cols);
    float* mq = mass + (single ? 4 * qi : qi) * a.tab_cols;
    if (single) {
      // masses of this query block from the table, written over its first row (this wave alone touches these rows)
      const int rows = min(4, n_sq - (a0 + 4 * qi));
      for (int j = l; j < nj; j += 64) {
        float acc = 0.f;
        for (int r = 0; r < rows; ++r) acc += __expf(mq[r * a.tab_cols + j] - lse[4 * qi + r]);
        mq[j] = acc / (float)rows;
      }
    }
    float tot = 0.f, mx = 0.f;
    for (int j = l; j < nj; j += 64) {
      tot += mq[j];
      mx = fmaxf(mx, mq[j]);
    }
    tot = wave_sum(tot);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    const float need = a.threshold * tot;
    // largest t (as a bit pattern; positive floats order like their bits) with sum(mass >= t) >= need
    uint32_t lo = 0, hi = __builtin_bit_cast(uint32_t, mx) + 1;       // feasible at lo, not at hi (or hi is past the maximum)
    while (hi - lo > 1) {
      const uint32_t mid = lo + (hi - lo) / 2;
      const float t = __builtin_bit_cast(float, mid);
      float sm = 0.f;
      for (int j = l; j < nj; j += 64) sm += mq[j] >= t ? mq[j] : 0.f;
      sm = wave_sum(sm);
      if (sm >= need) lo = mid; else hi = mid;
    }
    const float cut = __builtin_bit_cast(float, lo);
    for (int j = l; j < a.n_kblocks; j += 64) mrow[j] = (j < nj && (mq[j] >= cut || j == qb_abs)) ? 1 : 0;
  }
}

// ---- the same selection as a tiled matrix product followed by a small row kernel
//
// xa_scores_kernel computes the antidiagonal sums as the matrix product they are: a workgroup owns a tile of 128 square
// rows x 128 square columns of one head (four waves of 64 x 64, MFMA 16x16x32 bf16 on S^T = K Q^T) and walks the 16 * D
// numbers of a square in stages of 64, both operands coming through LDS by direct transfers (double buffered, one
// barrier per stage, two workgroups per CU).  Only tiles on or below the diagonal are launched.  The means e[a][b] go to
// the workspace in pieces of [128 square rows][16 square columns]; xa_keep_kernel (one wave per query block) reads its
// 4 rows piece by piece, does what the reduction phase of the walk does and writes the row of the keep matrix.  The
// sums are taken in the order of the walk (four chains of 4 row offsets, added in pairs), and so is everything after
// them: the two forms keep the same blocks, up to the 65536 positions of the single walk.  (Two walks take the quotient of
// exponentials where the others take the difference of logarithms: there a mass next to the cut may fall on either side.)
// What bounds it: the rate at which the L2s deliver operand rows to the CUs.  The walk above fetches every key row once
// per 32 square rows, this form every operand row once per 128 of the other operand: 16384 positions x 32 heads 1.2 GB
// instead of 2.1 GB (us for the selection, both kernels, back to back in a replayed graph: walk 340, here 139; traced, one
// at a time, this kernel takes 138 to 145, 700 TFLOP/s at its core, a quarter of it for the 75 MB of means, and the row kernel,
// which is bound by its vector instructions, 28 to 30).
constexpr int kXaTile = 128;                 // square rows / columns of a tile
constexpr int kXaPiece = kXaTile * 16;       // floats of a piece: 128 square rows x 16 square columns

struct XaScoreArgs {
  const __bf16* q;
  const int32_t* cu_q;
  const __bf16* k;
  int64_t stride_b, stride_h, stride_t;
  const int32_t* kv_len;
  int capacity;
  int hq, group;
  int bh0, n_bh;          // heads (of the whole batch, numbered b * hq + h) this launch works on
  int rt0, rt1;           // their row tiles
  int share;              // 0: plain order; else XCDs per (sequence, KV head) pair (see the kernel)
  int tab_cols;
  float scale, threshold;
  float* e;               // [n_bh][row tile rt0 <= rt < rt1][8 (rt + 1) pieces]
  uint8_t* mask;
  int n_qblocks, n_kblocks;
  int qb0, qb1;           // query blocks of this launch
  uint32_t* status;
};

// Length of the prompt that is scored; what is inconsistent is reported when `report` is set.
__device__ __forceinline__ int xa_prompt_len(int n_q, int kv_len, int capacity, int tab_cols, bool report, uint32_t* status) {
  bool bad = kv_len < 0 || kv_len > capacity || n_q != kv_len;
  const int len = kv_len < 0 ? 0 : (kv_len > capacity ? capacity : kv_len);
  int n = n_q < len ? (n_q < 0 ? 0 : n_q) : len;
  if (n > 64 * tab_cols) {
    bad = true;
    n = 64 * tab_cols;
  }
  if (report && bad) atomicOr(status, (uint32_t)FLUX_DEV_BAD_LENGTH);
  return n;
}

// Tiles of the row tiles below rt; a tile is 8 pieces.
__device__ __host__ __forceinline__ int64_t xa_tiles_below(int rt) { return (int64_t)rt * (rt + 1) / 2; }
constexpr int64_t kXaTileFloats = 8 * kXaPiece;

template <int D>
__global__ __launch_bounds__(256, 2) void xa_scores_kernel(XaScoreArgs a) {
  constexpr int HPR = D / 64;              // stages per row offset r
  constexpr int SEG = 4 * HPR;             // stages per chain of 4 row offsets
  constexpr int NST = 4 * SEG;             // stages of 64 numbers
  constexpr int OPB = kXaTile * 128;       // bytes of one operand tile of a stage: 128 rows of 128 bytes
  __shared__ __attribute__((aligned(1024))) char smem[2 * 2 * OPB];

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int g = l >> 4, nn = l & 15;
  const int64_t tiles0 = xa_tiles_below(a.rt0);
  const int n_tiles = (int)(xa_tiles_below(a.rt1) - tiles0);
  // which head and tile.  Workgroups go to the 8 XCDs by id mod 8: where the pairs of the launch are a multiple of 8 or
  // divide 8, all tiles of a pair get ids of `share` residues (1: one XCD, one L2), the heads of its group side by side
  int bh, tile;
  {
    const int i = blockIdx.x;
    if (a.share > 0) {
      const int x = i & 7, per = a.group * n_tiles, px = 8 / a.share;   // px: pairs worked on at a time
      const int item = (i >> 3) * a.share + x / px;                     // items of the pair sequence of this residue
      const int pair = x % px + px * (item / per);
      tile = (item % per) / a.group;
      bh = pair * a.group + item % a.group;
      if (bh >= a.n_bh) return;                            // padding of the last round
    } else {
      bh = i / n_tiles;
      tile = i % n_tiles;
    }
  }
  const int64_t t_abs = tiles0 + tile;
  int rt = (int)((__builtin_sqrtf(8.f * (float)t_abs + 1.f) - 1.f) * 0.5f);
  while (xa_tiles_below(rt) > t_abs) --rt;
  while (xa_tiles_below(rt + 1) <= t_abs) ++rt;
  rt = __builtin_amdgcn_readfirstlane(rt);                 // (it came through the vector unit)
  const int ct = (int)(t_abs - xa_tiles_below(rt));
  const int b = (a.bh0 + bh) / a.hq, h = (a.bh0 + bh) % a.hq, kvh = h / a.group;
  const int q_begin = a.cu_q[b];
  const int n = xa_prompt_len(a.cu_q[b + 1] - q_begin, a.kv_len[b], a.capacity, a.tab_cols, false, a.status);
  const int n_sq = (n + kXaStride - 1) / kXaStride;
  const int a0 = rt * kXaTile, b0 = ct * kXaTile;
  if (a0 >= n_sq) return;                                  // uniform: past the prompt

  // ---- direct transfers: every stage brings 128 bytes of each of the 128 rows of both operands, 8 rows per transfer.
  // Transfer t, lane l: row 8t + l/8, 16-byte piece l%8; the piece a lane fetches is swizzled by the row (as the K tile of
  // the prefill kernel with rows of 128 bytes: no bank conflicts on the fragment reads below).
  const int pitch_q = a.hq * D * 2, pitch_k = (int)a.stride_t * 2;      // bytes between positions
  const char* qbase = (const char*)(a.q + ((int64_t)(q_begin + kXaStride * a0) * a.hq + h) * D);
  const char* kbase = (const char*)(a.k + (int64_t)b * a.stride_b + (int64_t)kvh * a.stride_h + (int64_t)kXaStride * b0 * a.stride_t);
  const int piece = ((l & 7) ^ ((4 * (w & 1) + (l >> 4)) & 7)) * 16;
  const int q_lim = n - 1 - kXaStride * a0, k_lim = n - 1 - kXaStride * b0;   // last position of the prompt, from the tile's first
  int pos[4], off_q[4], off_k[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    pos[t] = kXaStride * (8 * (w + 4 * t) + (l >> 3));
    off_q[t] = pos[t] * pitch_q + piece;
    off_k[t] = pos[t] * pitch_k + piece;
  }
  const bool rag_q = kXaStride * kXaTile - 1 > q_lim, rag_k = kXaStride * kXaTile - 1 > k_lim;
  const uint32_t lds_w = (uint32_t)(uintptr_t)(FLUX_LDS char*)smem + 1024 * w;
  auto issue = [&](int s, int buf) __attribute__((always_inline)) {
    const int r = s / HPR, half = s % HPR;
    const uint32_t lk = lds_w + buf * 2 * OPB, lq = lk + OPB;
    // positions past the prompt are fetched from its last one; what they would contribute is left out below
    if (!rag_k) {
      const char* p = kbase + (int64_t)(kXaStride - 1 - r) * pitch_k + half * 128;      // keys in inverse order
#pragma unroll
      for (int t = 0; t < 4; ++t) lds_copy16(p, off_k[t], lk + 4096 * t);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) lds_copy16(kbase + half * 128, min(pos[t] + kXaStride - 1 - r, k_lim) * pitch_k + piece, lk + 4096 * t);
    }
    if (!rag_q) {
      const char* p = qbase + (int64_t)r * pitch_q + half * 128;
#pragma unroll
      for (int t = 0; t < 4; ++t) lds_copy16(p, off_q[t], lq + 4096 * t);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) lds_copy16(qbase + half * 128, min(pos[t] + r, q_lim) * pitch_q + piece, lq + 4096 * t);
    }
  };

  const int wa = w & 1, wb = w >> 1;                       // this wave's 64 square rows and 64 square columns of the tile
  const int aw = a0 + 64 * wa, bw = b0 + 64 * wb;
  const bool idle = bw > aw + 63 || aw >= n_sq;            // above the diagonal or past the prompt: transfers only
  const int last = n_sq - 1;                               // the prompt's last square holds last_cnt positions
  const int last_cnt = n - kXaStride * last;
  const bool part = last_cnt < kXaStride && aw <= last && last < aw + 64;   // this wave's rows hold a partial square
  const bool diag = bw == aw;                              // this wave's tile lies on the diagonal
  // acc[i][j][t]: square (aw + 16j + nn, bw + 16i + 4g + t), the chain of row offsets in progress
  f32x4 acc[4][4];
  int rd[2];                                               // LDS offsets of this lane's fragments (row nn of a 16-row block)
#pragma unroll
  for (int kc = 0; kc < 2; ++kc) rd[kc] = nn * 128 + (((4 * kc + g) ^ ((nn >> 1) & 7)) * 16);

  auto stage = [&](int s, int buf) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0): this wave's transfers have landed
    __syncthreads();                                       // ... and everyone's; the other buffer is free
    if (s + 1 < NST) issue(s + 1, buf ^ 1);
    if (idle) return;
    const int r = s / HPR;
    // the column of the prompt's last square holds the samples from 16 - last_cnt on: what the chain has of that square
    // on the diagonal (the only place where it matters) is cleared before the first of them
    if (diag && part && s % HPR == 0 && r == kXaStride - last_cnt) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (4 * g + t == nn && bw + 16 * i + nn == last) acc[i][i][t] = 0.f;
    }
    FLUX_LDS char* st = (FLUX_LDS char*)smem + buf * 2 * OPB;
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      bf16x8 kf[4], qf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) kf[i] = *(FLUX_LDS bf16x8*)(st + (64 * wb + 16 * i) * 128 + rd[kc]);
#pragma unroll
      for (int j = 0; j < 4; ++j) qf[j] = *(FLUX_LDS bf16x8*)(st + OPB + (64 * wa + 16 * j) * 128 + rd[kc]);
      if (part && r >= last_cnt) {                         // the last square row has no such sample
        const u32x4 zero = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (aw + 16 * j + nn == last) qf[j] = __builtin_bit_cast(bf16x8, zero);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[i], qf[j], acc[i][j], 0, 0, 0);
    }
  };
  // The sums of the chains 0 and 1 wait in this lane's own places of the workspace: with them, chain 2 and the chain in
  // progress in registers the kernel spills (192 accumulators; 256 registers at two waves per SIMD).
  f32x4 hi[4][4];                                          // sums of chain 0, later of chain 2
  float* out = a.e + ((int64_t)bh * n_tiles + (xa_tiles_below(rt) - tiles0)) * kXaTileFloats + (int64_t)(8 * ct + 4 * wb) * kXaPiece +
               (64 * wa + nn) * 16 + 4 * g;
  auto chain = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = SEG * c; s < SEG * (c + 1); s += 2) {
      stage(s, 0);
      stage(s + 1, 1);
    }
  };
  issue(0, 0);
  chain(0);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) hi[i][j] = acc[i][j];
  chain(1);
  if (!idle) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) *(f32x4*)(out + i * kXaPiece + j * 256) = hi[i][j] + acc[i][j];
  }
  chain(2);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) hi[i][j] = acc[i][j];
  chain(3);
  if (idle) return;

#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a_abs = aw + 16 * j + nn;
      const f32x4 lo = *(const f32x4*)(out + i * kXaPiece + j * 256);
      f32x4 v;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int b_abs = bw + 16 * i + 4 * g + t;
        const int r_min = max(max(b_abs == a_abs ? 8 : 0, kXaStride * b_abs + kXaStride - n), 0);
        const int cnt = min(kXaStride - 1, n - 1 - kXaStride * a_abs) - r_min + 1;
        // on the diagonal the samples r < 8 are not causal
        const float l01 = b_abs == a_abs ? 0.f : lo[t];
        const float l2 = r_min >= 12 ? 0.f : hi[i][j][t];
        const float sum = l01 + (l2 + acc[i][j][t]);
        v[t] = (a_abs > last || b_abs > a_abs || cnt <= 0) ? -INFINITY : a.scale * sum / (float)cnt;
      }
      *(f32x4*)(out + i * kXaPiece + j * 256) = v;
    }
}

// Values of other lanes by data-parallel-primitive moves (CTRL: quad_perm 0x00-0xff, row_ror:n 0x120+n,
// row_newbcast:n 0x150+n).
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
// ... and `none` where there is no such lane (row_shr:n 0x110+n).
template <int CTRL>
__device__ __forceinline__ float dpp_or(float x, float none) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, none), __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}
// x f + y, rounded after the product as well
__device__ __forceinline__ float scaled_sum(float x, float f, float y) {
#pragma clang fp contract(off)
  const float p = x * f;
  return p + y;
}
// Lane l ends up with the sum over the wave, added in the order of xor exchanges over 32, 16, 8, 4, 2, 1 (once the lanes
// whose numbers agree mod 2k hold the same value, the lane k further round the row holds that of lane l ^ k).
__device__ __forceinline__ float wave_sum_xor(float x) {
  x = sum_across_halves(x);
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  x = __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
  x += dpp<0x128>(x);
  x += dpp<0x124>(x);
  x += dpp<0x4e>(x);      // quad_perm [2, 3, 0, 1]
  x += dpp<0xb1>(x);      // quad_perm [1, 0, 3, 2]
  return x;
}

// One wave per query block; NR: masses a lane holds (one per 64 key blocks).  The row part does what the reduction phase of
// the walk does, with the same roundings, on four pieces at a time: lane l holds the 4 squares of a key block of square row l / 16.
// Bound by its vector instructions; with a lane per square and one piece after the other they were more than twice as many (select
// at 32/8 heads of 128, 16384 positions 151 -> 139 us, 32768 641 -> 591; 8/2 heads of 64, 16384 positions 45.6 -> 41.0).  The logarithm
// of the summed exponentials of a key block's 4 squares is kept in LDS ([4 rows][tab] per wave).
template <int NR, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void xa_keep_kernel(XaScoreArgs a) {
  extern __shared__ __attribute__((aligned(16))) char xa_smem[];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l = threadIdx.x & 63;
  const int n_qb = a.qb1 - a.qb0;
  const int64_t id = (int64_t)blockIdx.x * WAVES + w;
  if (id >= (int64_t)a.n_bh * n_qb) return;                // uniform for the wave; there is no workgroup barrier below
  const int bh = (int)(id / n_qb), qb = a.qb1 - 1 - (int)(id % n_qb);
  const int b = (a.bh0 + bh) / a.hq, h = (a.bh0 + bh) % a.hq;
  const int n_q = a.cu_q[b + 1] - a.cu_q[b];
  const int n = xa_prompt_len(n_q, a.kv_len[b], a.capacity, a.tab_cols, qb == 0 && h == 0 && l == 0, a.status);
  uint8_t* mrow = a.mask + (((int64_t)b * a.hq + h) * a.n_qblocks + qb) * (int64_t)a.n_kblocks;
  const int n_blk = (n + 63) / 64;
  if (qb >= n_blk) {                                       // a row of the matrix beyond the prompt
    for (int j = l; j < a.n_kblocks; j += 64) mrow[j] = 0;
    return;
  }
  const int tab = 64 * NR;
  float* table = (float*)xa_smem + w * 4 * tab;
  const int rr = l >> 4, rb = l & 15;
  const int n_ct = qb / 4 + 1;                             // pieces up to the diagonal
  const int rt = qb / 32, rows = min(4, (n + kXaStride - 1) / kXaStride - 4 * qb);
  const int64_t tiles0 = xa_tiles_below(a.rt0);
  // four pieces at a time: lane (rr, rb) has the 4 squares of key block rb % 4 of piece c0 + rb / 4, in row rr
  const float* src = a.e + ((int64_t)bh * (xa_tiles_below(a.rt1) - tiles0) + (xa_tiles_below(rt) - tiles0)) * kXaTileFloats +
                     (4 * (qb % 32) + rr) * 16 + 4 * (rb & 3);
  auto ask = [&](int c0) { return *(const f32x4*)(src + (int64_t)min(c0 + (rb >> 2), n_ct - 1) * kXaPiece); };
  // m_row is a row's reference behind the last piece, m the one behind this lane's; what refers to it uses 0 while the row has no
  // finite value (the exponentials of -inf are 0 then as well).
  float m_row = -INFINITY, l_row = 0.f;
  f32x4 e_next = ask(0);
  for (int c0 = 0; c0 < n_ct; c0 += 4) {
    const f32x4 e = e_next;
    const bool there = rr < rows && c0 + (rb >> 2) < n_ct; // (rows past the prompt are not written)
    if (c0 + 4 < n_ct) e_next = ask(c0 + 4);
    float x[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) x[t] = there ? e[t] : -INFINITY;
    float m = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    m = fmaxf(m, dpp<0xb1>(m));                            // of the piece ...
    m = fmaxf(m, dpp<0x4e>(m));
    m = fmaxf(m, dpp_or<0x114>(m, -INFINITY));             // ... and of those in front of it (row_shr:4, row_shr:8)
    m = fmaxf(m, dpp_or<0x118>(m, -INFINITY));
    m = fmaxf(m, m_row);
    const float m_use = m == -INFINITY ? 0.f : m;
    float p[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) p[t] = __expf(x[t] - m_use);
    const float pe = (p[0] + p[1]) + (p[2] + p[3]);
    table[rr * tab + 4 * c0 + rb] = pe > 0.f ? m_use + __logf(pe) : -INFINITY;
    float sum = pe + dpp<0xb1>(pe);                        // of the piece
    sum += dpp<0x4e>(sum);
    // the pieces one after the other; where a row's reference moves, what it has so far moves along (elsewhere the factor is 1)
    if (__builtin_amdgcn_ballot_w64(m > m_row) != 0) {
      const float shifted = dpp<0x114>(m);                  // (by all lanes: a lane that is switched off has nothing to give)
      const float before = rb < 4 ? m_row : shifted;
      const float f = before == -INFINITY ? 0.f : __expf(before - m);
      l_row = scaled_sum(l_row, dpp<0x150>(f), dpp<0x150>(sum));
      l_row = scaled_sum(l_row, dpp<0x154>(f), dpp<0x154>(sum));
      l_row = scaled_sum(l_row, dpp<0x158>(f), dpp<0x158>(sum));
      l_row = scaled_sum(l_row, dpp<0x15c>(f), dpp<0x15c>(sum));
      m_row = dpp<0x15c>(m);
    } else {
      l_row += dpp<0x150>(sum);
      l_row += dpp<0x154>(sum);
      l_row += dpp<0x158>(sum);
      l_row += dpp<0x15c>(sum);
    }
  }
  const float lse = m_row + __logf(l_row);
  float lse_r[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) lse_r[r] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lse), 16 * r));
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the table is this wave's own
  __builtin_amdgcn_wave_barrier();
  // masses of key blocks l, l + 64, ...
  float mass[NR];
  float tot = 0.f, top = 0.f;
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    mass[i] = 0.f;
    const int j = 64 * i + l;
    if (j <= qb) {
      float acc = 0.f;
      for (int r = 0; r < rows; ++r) acc += __expf(table[r * tab + j] - lse_r[r]);
      mass[i] = rows == 4 ? acc * 0.25f : acc / (float)rows;  // (the same)
      tot += mass[i];
      top = fmaxf(top, mass[i]);
    }
  }
  tot = wave_sum_xor(tot);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off));
  // ---- the cut: largest t (as a bit pattern; positive floats order like their bits) with sum(mass >= t) >= need
  const float need = a.threshold * tot;
  // (found as soon as at most one mass lies between the bounds: the blocks kept are the same for any t above the mass before)
  // (What lies below a mass of half of (tot - need) / (qb + 1) is at most half of what may be left out: far from where roundings
  // could matter while that is a thousandth of the total, so the search begins there and not at 0.)
  const float spare = tot - need;
  uint32_t lo = spare > 1e-3f * tot ? __builtin_bit_cast(uint32_t, 0.5f * spare / (float)(qb + 1)) : 0, hi = __builtin_bit_cast(uint32_t, top) + 1;
  lo = lo < hi ? lo : hi - 1;
  int above_lo = 64 * NR, above_hi = 0;                    // masses at or above the bounds
  while (hi - lo > 1 && above_lo - above_hi > 1) {
    const uint32_t mid = lo + (hi - lo) / 2;
    const float t = __builtin_bit_cast(float, mid);
    float sm = 0.f;
    int above = 0;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const bool in = mass[i] >= t;
      sm += in ? mass[i] : 0.f;
      above += __builtin_popcountll(__builtin_amdgcn_ballot_w64(in));
    }
    sm = wave_sum_xor(sm);
    if (sm >= need) {
      lo = mid;
      above_lo = above;
    } else {
      hi = mid;
      above_hi = above;
    }
  }
  const float cut = __builtin_bit_cast(float, lo);
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int j = 64 * i + l;
    if (j < a.n_kblocks) mrow[j] = (j <= qb && (mass[i] >= cut || j == qb)) ? 1 : 0;
  }
  for (int j = 64 * NR + l; j < a.n_kblocks; j += 64) mrow[j] = 0;
}

// Launch both kernels for the heads and row tiles of x; `whole`: the query blocks past the last row tile are cleared too.
template <int D>
static hipError_t launch_xa_tiles(XaScoreArgs& x, int n_rt, hipStream_t s) {
  const long long n_tiles = xa_tiles_below(x.rt1) - xa_tiles_below(x.rt0);
  x.qb0 = 32 * x.rt0;
  x.qb1 = x.rt1 == n_rt ? x.n_qblocks : (32 * x.rt1 < x.n_qblocks ? 32 * x.rt1 : x.n_qblocks);
  long long n_wg = n_tiles * x.n_bh;
  x.share = 0;
  if (x.bh0 % x.group == 0 && x.n_bh % x.group == 0) {
    const int pairs = x.n_bh / x.group;
    x.share = pairs % 8 == 0 ? 1 : (8 % pairs == 0 ? 8 / pairs : 0);
    if (x.share > 1) n_wg = (n_tiles * x.group + x.share - 1) / x.share * 8;
  }
  hipLaunchKernelGGL(xa_scores_kernel<D>, dim3((unsigned)n_wg), dim3(256), 0, s, x);
  const long long waves = (long long)x.n_bh * (x.qb1 - x.qb0);
  // four waves per workgroup while their tables leave room for two workgroups in the LDS of a CU
  if (x.tab_cols <= 256) hipLaunchKernelGGL((xa_keep_kernel<4, 4>), dim3((unsigned)((waves + 3) / 4)), dim3(256), 4 * 4 * 256 * 4, s, x);
  else if (x.tab_cols <= 1024) hipLaunchKernelGGL((xa_keep_kernel<16, 2>), dim3((unsigned)((waves + 1) / 2)), dim3(128), 2 * 4 * 1024 * 4, s, x);
  else hipLaunchKernelGGL((xa_keep_kernel<64, 1>), dim3((unsigned)waves), dim3(64), 4 * 4096 * 4, s, x);
  return hipGetLastError();
}

hipError_t launch_xa_select(const Ctx& c, const flux_attn_cfg& cfg, const void* q, const int32_t* cu_q, int max_q_len,
                            const flux_kv_cache& cache, float threshold, uint8_t* mask, int n_qblocks, int n_kblocks,
                            hipStream_t s) {
  XaArgs a;
  a.q = (const __bf16*)q;
  a.cu_q = cu_q;
  a.k = (const __bf16*)cache.k;
  a.stride_b = cache.stride_b;
  a.stride_h = cache.stride_h;
  a.stride_t = cache.stride_t;
  a.kv_len = cache.kv_len;
  a.capacity = cache.capacity;
  a.hq = cfg.n_q_heads;
  a.group = cfg.n_q_heads / cfg.n_kv_heads;
  a.batch = cache.batch;
  a.scale = cfg.softmax_scale != 0.f ? cfg.softmax_scale : 1.0f / sqrtf((float)cfg.head_dim);
  a.threshold = threshold;
  a.mask = mask;
  a.n_qblocks = n_qblocks;
  a.n_kblocks = n_kblocks;
  const int need = (max_q_len + 63) / 64;                 // the prompt is the whole cache: its length is bounded by max_q_len
  a.tab_cols = need < n_kblocks ? (need > 0 ? need : 1) : n_kblocks;
  a.single_walk = a.tab_cols <= kXaSingleWalkMaxKBlocks;
  a.status = c.status;
  // Tiled form.  Its scratch is one float per square at or below the diagonal (rounded up to tiles); heads, or row tiles of
  // one head, are worked off in as many rounds as the context's workspace makes necessary (it must hold one row tile).
  // 32-bit byte offsets inside a tile bound the strides.
  // Prompts bounded by less than 1024 positions (head dimension 64: 320) stay with the walk above: one launch instead of
  // two, and a tile of 128 square rows would be mostly empty.  One prompt, walk / tiles in us, 32/8 heads of 128: 300
  // positions 29 / 32, 1000 positions 34.8 / 34.2, 4096 positions 65 / 42, 8192 positions 129 / 63, 16384 positions
  // 342 / 170, 33000 positions 1600 / 700, 65536 positions 5500 / 2700; 8/2 heads of 64: 300 positions 26 / 22, 16384
  // positions 130 / 50.
  const int n_rt = (a.tab_cols + 31) / 32;
  const long long tile_bytes = kXaTileFloats * sizeof(float);
  const bool tiled = a.tab_cols >= (cfg.head_dim == 128 ? 16 : 5);
  if (tiled && (long long)c.partials_bytes >= n_rt * tile_bytes && (int64_t)a.hq * cfg.head_dim < (1 << 18) && a.stride_t < (1 << 18)) {
    const int total = cache.batch * cfg.n_q_heads;
    XaScoreArgs x;
    x.q = a.q;
    x.cu_q = a.cu_q;
    x.k = a.k;
    x.stride_b = a.stride_b;
    x.stride_h = a.stride_h;
    x.stride_t = a.stride_t;
    x.kv_len = a.kv_len;
    x.capacity = a.capacity;
    x.hq = a.hq;
    x.group = a.group;
    x.tab_cols = a.tab_cols;
    x.scale = a.scale;
    x.threshold = threshold;
    x.e = c.partials;
    x.mask = mask;
    x.n_qblocks = n_qblocks;
    x.n_kblocks = n_kblocks;
    x.status = c.status;
    const long long room = (long long)c.partials_bytes / tile_bytes;   // tiles the workspace holds
    const long long per_head = xa_tiles_below(n_rt);
    long long fit = room / per_head;                                    // whole heads
    const long long most = 0x3FFFFFFFll / (per_head > n_qblocks ? per_head : n_qblocks);   // grid sizes
    if (fit > most) fit = most;
    if (fit < total) {                                                  // whole rounds of 8, 4, 2 or 1 groups where they fit
      for (int p = 8; p >= 1; p >>= 1)
        if (fit >= p * a.group) {
          fit = (p == 8 ? fit / (8 * a.group) * 8 : p) * a.group;
          break;
        }
    }
    for (int bh0 = 0; bh0 < total; bh0 += x.n_bh) {
      x.bh0 = bh0;
      x.n_bh = fit < 1 ? 1 : (total - bh0 < fit ? total - bh0 : (int)fit);
      for (x.rt0 = 0; x.rt0 < n_rt; x.rt0 = x.rt1) {
        x.rt1 = n_rt;
        while (fit < 1 && xa_tiles_below(x.rt1) - xa_tiles_below(x.rt0) > room) --x.rt1;
        const hipError_t e = cfg.head_dim == 128 ? launch_xa_tiles<128>(x, n_rt, s) : launch_xa_tiles<64>(x, n_rt, s);
        if (e != hipSuccess) return e;
      }
    }
    return hipSuccess;
  }
  const int groups = (n_qblocks + 7) / 8;                 // every row of the matrix is written
  a.n_groups = groups;
  const dim3 grid((unsigned)((long long)groups * cfg.n_q_heads * cache.batch));
  const size_t lds = xa_select_lds_bytes(a.tab_cols);
  if (cfg.head_dim == 128) {
    if (lds > 48 * 1024) {
      const hipError_t e = hipFuncSetAttribute((const void*)xa_select_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(xa_select_kernel<128>, grid, dim3(256), lds, s, a);
  } else {
    if (lds > 48 * 1024) {
      const hipError_t e = hipFuncSetAttribute((const void*)xa_select_kernel<64>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(xa_select_kernel<64>, grid, dim3(256), lds, s, a);
  }
  return hipGetLastError();
}

}  // namespace flux
