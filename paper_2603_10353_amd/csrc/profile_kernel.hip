// Recovery profiles (paper Section 2.4), two dense causal passes that are not on the hot path:
//
//  * mass_kernel: at block granularity, the attention weight every query block puts on every key
//    block of the causal triangle, under full attention,
//      mass[s][h][i][j] = 1/n_i * sum over the valid queries t of block i, keys u of block j, u <= t,
//                         of softmax_t(q_t . k_u * scale)                    (j <= i; rows sum to 1)
//    Sorted per row and accumulated it gives the recovery curves that budget shifting consumes,
//    and summed over a selection it says how much of the attention that selection keeps.
//  * token_recovery_kernel: at the paper's own granularity, for every query token the sum of its
//    k largest attention weights, for up to eight budgets k at once.
//
// Both use the first contraction of the attention kernels (64-key K tiles copied global->LDS
// into swizzled 256-byte rows, S^T = K Q^T with Q in registers, a lane owns one query column) and
// have no second one.  One workgroup = 128 consecutive queries of a (sequence, head), whatever the
// block size, in one or a few sweeps over their keys; the scores are recomputed in every sweep (the
// triangle of scores does not fit anywhere).  The longest are launched first, so that the tail of
// the launch is short.
#include <cfloat>

#include "attn_common.h"

namespace shplb {
namespace {

// 128 consecutive queries of one (sequence, head) swept over their keys in tiles of kTile; a wave owns 32
// queries.  The tiles are software-pipelined: the MFMAs of the next tile are issued before the work on the
// present one's scores, which depends on none of them, and a tile is copied one whole step ahead of its use.
// kSmall: the contraction in 16x16x32 MFMAs, of two groups of 16 queries, instead of 32x32x16: for a pass at the card's
// power limit (the block mass of 32 heads x 32K tokens 4.60 -> 3.99 ms, with the kept sums below).  The token recovery, whose
// state is per query, is near that limit too, but waits for LDS and for VALU issue: with small products 32 heads x 32K tokens
// take 12.2 ms for 11.7 and 28 x 6001, two budgets, 925 us for 833.  With the MFMAs behind the work on the scores the mass takes
// 4.18 ms, and launches of one workgroup per compute unit or fewer, whose SIMDs have one wave, are slower than with 32x32x16: 8/2
// heads x 4000 tokens 51.5 us for 49.7, now 48.8; 8/2 x 1000 18.0 for 17.4, now 17.3.
template <bool kSmall>
struct QueryRun {
  static constexpr int kQueries = 128, kWaves = kQueries / 32;
  static constexpr int kTile = 64, MT = kTile / 32;                  // keys of a tile
  static constexpr int kStageBytes = kTile * kRowBytes;
  static constexpr int kRoundRows = 4 * kWaves;                      // key rows one copy instruction per wave moves
  static constexpr int kRounds = kTile / kRoundRows;
  // A lane's scores: 32 of query n, v[mt][r] of key 32 mt + 8 (r / 4) + 4 hi + r % 4 (n, hi: lane % 32 and lane / 32), or 16 each
  // of queries n and 16 + n, v[qg][mt][r] of key 16 mt + 4 hi + r (lane % 16 and lane / 16).
  static constexpr int QG = 2;
  struct Large { f32x16 v[MT]; };
  struct Small { f32x4 v[QG][kTile / 16]; };
  typedef std::conditional_t<kSmall, Small, Large> Scores;
  static constexpr int kOperands = kSmall ? 4 * (kTile / 16) : 8 * MT;
  static constexpr int kLook = 8;                                    // operand fetches ahead of the MFMA that uses them
  // Steps between sampled keys are multiples of 1/kOne.  (The largest products fit: all keys, kOne apart, are up
  // to 2^19 x 2^12; of those sampled, 2^11 at most, the last is one of these keys; a step is below 2^24.)
  static constexpr uint32_t kOne = 4096;

  int s, h, i, tid, lane, wave, n, hi;
  int seq_begin, seq_end, n_tiles, q_tok;
  int cp_row, k_rd0;
  uint32_t k_stage0;
  int64_t row_bytes;
  uint32_t widest;                                  // largest distance of a sampled tile's keys, see issue_tile()
  const char* k_head;
  const char* k_lds;                                // two stages of kStageBytes
  bf16x8 qf[8];                                     // B operands of S^T = K Q^T: dims 16ks + 8hi.. of the lane's query, or
                                                    // 32ks + 8hi.. of its two, index 4qg + ks

  // index (of the workgroup) = level * (sequences * heads) + place of the (sequence, head); level 0 is the end of the longest
  // sequence.  Workgroups go to the dies in turn: places x, x + 8, .. are given consecutive heads, so that a
  // die works on few K streams (32 heads, 8 KV heads: on one).  False: this sequence is shorter.
  __device__ __forceinline__ bool init(const SeqMeta& meta, const Strides& st, const uint16_t* __restrict__ k,
                                       int levels, const char* lds, uint32_t index) {
    const int per_level = meta.n_seq * meta.n_q_heads;
    const int level = index / per_level, place = index - level * per_level;
    const int die = place % kXcds;
    const int sh = die * (per_level / kXcds) + min(die, per_level % kXcds) + place / kXcds;
    s = sh / meta.n_q_heads;
    h = sh - s * meta.n_q_heads;
    i = levels - 1 - level;
    seq_begin = meta.tok_begin[s];
    seq_end = meta.tok_begin[s + 1];
    if (i * kQueries >= seq_end - seq_begin) return false;
    tid = threadIdx.x;
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    n = kSmall ? lane & 15 : lane & 31;
    hi = kSmall ? lane >> 4 : lane >> 5;
    n_tiles = (i + 1) * (kQueries / kTile);
    row_bytes = st.kv_t * 2;
    widest = uint32_t(fminf(float(1ull << 32) * (0.999f * kOne / kTile) / float(row_bytes), 0x1p23f));
    k_head = reinterpret_cast<const char*>(k + int64_t(kv_head_of(meta, h)) * st.kv_h);
    k_lds = lds;
    cp_row = 4 * wave + (lane >> 4);
    k_rd0 = n * kRowBytes + ((hi ^ swz(n)) << 4);
    k_stage0 = __builtin_amdgcn_readfirstlane(lds_offset_of(lds) + 4 * wave * kRowBytes);
    q_tok = seq_begin + i * kQueries + wave * 32 + (lane & 31);
    return true;
  }
  __device__ __forceinline__ bool live() const { return q_tok < seq_end; }   // not past the end of the sequence

  __device__ __forceinline__ void load_queries(const Strides& st, const uint16_t* __restrict__ q) {
#pragma unroll
    for (int qg = 0; qg < (kSmall ? QG : 1); ++qg) {
      // (a lane's one query: q_tok; worked out again, token recoveries of several budgets spilled more scalar registers, and
      // 8 heads x 1012 tokens with two took 124.6 us instead of 121.9)
      const int tok = kSmall ? seq_begin + i * kQueries + wave * 32 + 16 * qg + n : q_tok;
      const uint16_t* src = q + int64_t(min(tok, seq_end - 1)) * st.q_t + int64_t(h) * st.q_h + 8 * hi;
      constexpr int kSteps = kSmall ? 4 : 8;
#pragma unroll
      for (int ks = 0; ks < kSteps; ++ks) qf[kSteps * qg + ks] = *reinterpret_cast<const bf16x8*>(src + (kSmall ? 32 : 16) * ks);
    }
  }

  // Copy a tile into LDS stage `buf`: keys kTile x .. of the row's, or of those that are left when only every
  // (stride / kOne)-th is taken.  Rows past the end of the sequence re-read its last key; they are masked.
  // Offsets within a tile are 32 bits wide: the sampled keys of a tile move closer together where K's rows are so
  // far apart that the tile would reach over 4 GiB (`widest`; at 128K tokens, rows of more than 130 KB).  Keys
  // next to each other always fit: rows are less than 2^25 bytes apart, and `widest` is at least kOne then.
  __device__ __forceinline__ void issue_tile(int x, uint32_t stride, int buf) const {
    const uint32_t step = stride == kOne ? kOne : min(stride, widest);
    const int first = int(uint32_t(kTile * x) * stride / kOne);
    const int key_base = min(seq_begin + first, seq_end - 1);
    const int last = seq_end - 1 - key_base;
    const char* k_tile = k_head + int64_t(key_base) * row_bytes;
#pragma unroll
    for (int rd = 0; rd < kRounds; ++rd) {
      const int r = rd * kRoundRows + cp_row;
      const int key = int(__umul24(r, step) / kOne);
      const uint32_t off = uint32_t(min(key, last)) * uint32_t(row_bytes) + (((lane & 15) ^ swz(r)) << 4);
      copy_g2l_16(k_tile, off, __builtin_amdgcn_readfirstlane(k_stage0 + buf * kStageBytes + rd * kRoundRows * kRowBytes));
    }
  }

  __device__ __forceinline__ bf16x8 read_k(int buf, int gi) const {
    const char* kt = k_lds + buf * kStageBytes;
    if (kSmall) return *reinterpret_cast<const bf16x8*>(kt + (k_rd0 ^ ((gi >> 2) << 6)) + (gi & 3) * 16 * kRowBytes);
    return *reinterpret_cast<const bf16x8*>(kt + (k_rd0 ^ ((gi / MT) << 5)) + (gi % MT) * 32 * kRowBytes);
  }
  // raw scores (q . k, unscaled) of the tile in stage `buf`
  __device__ __forceinline__ void scores_of(int buf, Scores& sc) const {
    if constexpr (kSmall) {
#pragma unroll
      for (int qg = 0; qg < QG; ++qg)
#pragma unroll
        for (int mt = 0; mt < kTile / 16; ++mt) sc.v[qg][mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    } else {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) sc.v[mt][r] = 0.0f;
    }
    bf16x8 kf[kOperands];
#pragma unroll
    for (int gi = 0; gi < kLook; ++gi) kf[gi] = read_k(buf, gi);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int gi = 0; gi < kOperands; ++gi) {
      if (gi + kLook < kOperands) kf[gi + kLook] = read_k(buf, gi + kLook);
      if constexpr (kSmall) {
#pragma unroll
        for (int qg = 0; qg < QG; ++qg)
          sc.v[qg][gi & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[gi], qf[4 * qg + (gi >> 2)], sc.v[qg][gi & 3], 0, 0, 0);
      } else {
        sc.v[gi % MT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[gi], qf[gi / MT], sc.v[gi % MT], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // keys above the lane's query to -inf (tiles of the diagonal only)
  __device__ __forceinline__ void mask(int it, Scores& sc) const {
#pragma unroll
    for (int qg = 0; qg < (kSmall ? QG : 1); ++qg) {
      int d = kTile * it - kQueries * i + 4 * hi - (wave * 32 + 16 * qg + n);   // key position minus query position, per register below
      asm volatile("" : "+v"(d));                                           // keep the 32 comparisons here, not hoisted as masks
      if constexpr (kSmall) {
#pragma unroll
        for (int mt = 0; mt < kTile / 16; ++mt) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (d + (16 * mt + r) > 0) sc.v[qg][mt][r] = -INFINITY;
          asm volatile("" : "+v"(sc.v[qg][mt]));
        }
      } else {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (d + (32 * mt + 8 * (r >> 2) + (r & 3)) > 0) sc.v[mt][r] = -INFINITY;
      }
    }
  }

  // A sweep over the row's keys, or over `count` tiles' worth of them evenly spread (a stretch of keys alike
  // must not come in or stay out as a whole), in two parts: start() sends the first tiles on their way (the
  // stages are free after its barrier), sweep() calls per_tile(x, sc) with the raw scores of tile after tile,
  // x = first ..; masked (all keys only): keys above the lane's query are -inf.
  __device__ __forceinline__ uint32_t stride_of(int count) const {
    return __builtin_amdgcn_readfirstlane(uint32_t(n_tiles) * kOne / uint32_t(count));
  }
  __device__ __forceinline__ void start(int first, int count, uint32_t stride) const {
    __syncthreads();
    issue_tile(first, stride, 0);
    if (count > 1) issue_tile(first + 1, stride, 1);
  }
  template <class F>
  __device__ __forceinline__ void sweep(int first, int count, uint32_t stride, bool masked, F&& per_tile) const {
    const int end = first + count;
    Scores sa, sb;
    wait_vmem_all();
    __syncthreads();
    scores_of(0, sa);
    auto step = [&](int x, int buf, Scores& cur, Scores& nxt) {
      if (x + 1 < end) {
        wait_vmem_all();                            // own copies of tile x + 1 have landed
        __syncthreads();                            // everyone's have; the stage of tile x is free
        if (x + 2 < end) issue_tile(x + 2, stride, buf);
        scores_of(buf ^ 1, nxt);
      }
      if (masked && x >= n_tiles - kQueries / kTile) mask(x, cur);
      per_tile(x, cur);
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int x = first; x < end; x += 2) {
      step(x, 0, sa, sb);
      if (x + 1 < end) step(x + 1, 1, sb, sa);
    }
  }
};

// Attention weight of every key block, averaged over the queries of a query block; BQ = the block size.
//
// One sweep over the keys: the exponentials of a query against a fixed reference exponent, summed per key block
// and kept, as many as there is room for, and in all; divided by the query's total and summed over the
// queries of a block once it is known.  A query's sums are kept in LDS (a word per block and query); twice, when
// there are kBankBlocks of them and more to come than fit, these move to 32 registers, alternating between the two
// lanes of the query.  (Written to registers one by one, by an index, they had the compiler copy all 64 of them for
// every key block: 4.8 -> 4.5 ms without.)  Only key blocks behind these (of rows beyond 28K tokens with 128-token
// blocks, 14K with 64) are swept a second time, kLdsBlocks at a time, when the totals are known.
//
// The reference is the largest score of the query's first tile.  It is a scale, not a bound: the sums are floats and
// lose nothing by being large, so it is only raised (and what is kept scaled down, at most a few times per row)
// when a tile's sum leaves the range of useful exponents.
//
// Sums run over keys, tiles, queries and waves in a fixed order: results repeat bit for bit.
// 32 heads x 32K tokens: 4.0 ms, from 4.6 on the same card with 32x32x16 MFMAs, which spend more of the power (the launch
// runs at its limit, at 2.1 GHz), and the copies above.  The VALU issues in 76% of the cycles (per key and 64 queries an
// exponential, a multiply-add and an addition, 16 cycles), the matrix pipe is busy in 51%.
constexpr int kLdsBlocks = 92, kBankBlocks = 64;   // 4 x 92 x 32 words beside the tiles and partial sums: two workgroups
                                                   // per compute unit; two banks of 32 registers
constexpr float kSumRange = 0x1p64f;

typedef float f32x32 __attribute__((ext_vector_type(32)));

typedef QueryRun<true> MassRun;

template <int BQ>
__global__ __launch_bounds__(256, 2) void mass_kernel(SeqMeta meta, Strides st, const uint16_t* __restrict__ q,
                                                      const uint16_t* __restrict__ k, float* __restrict__ mass,
                                                      int levels, float scale_log2) {
  constexpr int kTiles = BQ / MassRun::kTile;                // tiles of a key block
  constexpr int kRows = MassRun::kQueries / BQ;              // query blocks of the workgroup
  constexpr int kRowWaves = MassRun::kWaves / kRows;
  __shared__ __attribute__((aligned(1024))) char k_lds[2][MassRun::kStageBytes];
  __shared__ float s_sums[MassRun::kWaves][kLdsBlocks][32];
  __shared__ float s_weight[MassRun::kWaves][32];
  __shared__ float s_part[MassRun::kWaves][kLdsBlocks];

  MassRun row;
  if (!row.init(meta, st, k, levels, &k_lds[0][0], blockIdx.x)) return;
  const int nb = meta.blk_begin[row.s + 1] - meta.blk_begin[row.s];
  const int n_blocks = min((row.i + 1) * kRows, nb);          // key blocks the workgroup's queries see
  const int n_tiles = n_blocks * kTiles;
  row.start(0, n_tiles, MassRun::kOne);
  row.load_queries(st, q);

  // Sums and what is kept of them belong to query `query` of the wave, the same in lanes l and l ^ 32; the scores of a
  // lane to queries n and 16 + n, of which `query` is one.
  constexpr int QG = MassRun::QG;
  const int query = row.lane & 31, half = row.lane >> 5;
  float (*sums)[32] = s_sums[row.wave];
  float ref[QG] = {0.0f, 0.0f}, part[QG] = {0.0f, 0.0f}, total = 0.0f;
  f32x32 held0, held1;
#pragma unroll
  for (int x = 0; x < 32; ++x) held0[x] = held1[x] = 0.0f;
  const int banks = n_blocks <= kLdsBlocks ? 0 : n_blocks <= kLdsBlocks + kBankBlocks ? 1 : 2;
  int filled = 0;                                             // banks that hold their sums

  auto tile_sums = [&](const MassRun::Scores& sc, float (&sum)[QG]) {
    float s[QG][2];
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) s[qg][0] = s[qg][1] = 0.0f;
#pragma unroll
    for (int x = 0; x < 16; ++x)
#pragma unroll
      for (int qg = 0; qg < QG; ++qg)
        s[qg][x & 1] += __builtin_amdgcn_exp2f(__builtin_fmaf(sc.v[qg][x >> 2][x & 3], scale_log2, -ref[qg]));
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) sum[qg] = s[qg][0] + s[qg][1];
  };
  auto largest = [&](const MassRun::Scores& sc, int qg) {
    float m = sc.v[qg][0][0];
#pragma unroll
    for (int x = 1; x < 16; ++x) m = fmaxf(m, sc.v[qg][x >> 2][x & 3]);
    return quad_max(m) * scale_log2;
  };
  // over the four lanes of a query, and to the lanes whose `query` it is
  auto collected = [](const float (&x)[QG]) {
    uint32_t a = __float_as_uint(x[0]), b = __float_as_uint(x[1]);
    swap_rows(a, b);
    return pair_sum(__uint_as_float(a) + __uint_as_float(b));
  };
  row.sweep(0, n_tiles, MassRun::kOne, true, [&](int x, MassRun::Scores& sc) {
    const int j = x / kTiles - kBankBlocks * filled;          // where the block's sums are kept
    // every query sees its sequence's first key; a tile whose scores are all -inf weighs nothing against any reference
    if (x == 0)
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) ref[qg] = fmaxf(largest(sc, qg), -FLT_MAX);
    float sum[QG];
    tile_sums(sc, sum);
    if (__any(!(sum[0] <= kSumRange) || !(sum[1] <= kSumRange))) {
      float alpha[QG];
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) {
        const float raised = fmaxf(ref[qg], largest(sc, qg));
        alpha[qg] = __builtin_amdgcn_exp2f(ref[qg] - raised);
        ref[qg] = raised;
        part[qg] *= alpha[qg];
      }
      const float own = row.lane & 16 ? alpha[1] : alpha[0];
      total *= own;
      // (blocks behind the kept ones keep counting j: they are not in LDS, and are swept again against the final reference)
      for (int y = half; y < min(j, kLdsBlocks); y += 2) sums[y][query] *= own;
#pragma unroll
      for (int y = 0; y < 32; ++y) {
        held0[y] *= own;
        held1[y] *= own;
      }
      tile_sums(sc, sum);
    }
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) part[qg] += sum[qg];
    if (kTiles == 1 || x % kTiles == kTiles - 1) {
      const float block = collected(part);
      total += block;
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) part[qg] = 0.0f;
      if (j < kLdsBlocks) sums[j][query] = block;             // (both lanes of the query, the same)
      if (j == kBankBlocks - 1 && filled < banks) {
        asm volatile("" ::: "memory");                        // the wave's own sums
#pragma unroll
        for (int y = 0; y < 32; ++y) {                        // (selected, not branched: pointers to the banks would put them in memory)
          const float kept = sums[2 * y + half][query];
          held1[y] = filled == 0 ? held1[y] : kept;
          held0[y] = filled == 0 ? kept : held0[y];
        }
        filled += 1;
        asm volatile("" ::: "memory");
      }
    }
  });
  // a query's share of its block's average; none for a query past the end of the sequence
  const int q_block = row.i * kRows + row.wave / kRowWaves;   // the wave's query block
  const int n_valid = min(BQ, row.seq_end - row.seq_begin - q_block * BQ);
  s_weight[row.wave][query] = row.live() ? 1.0f / (total * float(n_valid)) : 0.0f;

  // the key blocks base .. base + count whose sums are in LDS: over the wave's queries (a lane takes a block
  // and goes round them), then over the waves of a query block
  auto flush = [&](int base, int count) {
    asm volatile("" ::: "memory");                            // sums and weights are the wave's own
    for (int y = row.lane; y < count; y += 64) {
      float a = 0.0f;
#pragma unroll 8
      for (int x = 0; x < 32; ++x) {
        const int n = (x + row.lane) & 31;
        a += sums[y][n] * s_weight[row.wave][n];
      }
      s_part[row.wave][y] = a;
    }
    __syncthreads();
    for (int y = row.tid; y < count * kRows; y += 256) {
      const int r = kRows == 1 ? 0 : y / count, j = y - r * count, i = row.i * kRows + r;
      float a = s_part[r * kRowWaves][j];
#pragma unroll
      for (int w = 1; w < kRowWaves; ++w) a += s_part[r * kRowWaves + w][j];
      if (i < nb && base + j <= i) mass[meta.score_off[row.s] + (int64_t(row.h) * nb + i) * nb + base + j] = a;
    }
    __syncthreads();
  };
  flush(kBankBlocks * banks, min(n_blocks - kBankBlocks * banks, kLdsBlocks));
  auto flush_bank = [&](int base, const f32x32& held) {
#pragma unroll
    for (int x = 0; x < 32; ++x) sums[2 * x + half][query] = held[x];
    flush(base, kBankBlocks);
  };
  if (banks > 0) flush_bank(0, held0);
  if (banks > 1) flush_bank(kBankBlocks, held1);
  for (int base = kLdsBlocks + 2 * kBankBlocks; base < n_blocks; base += kLdsBlocks) {
    const int count = min(n_blocks - base, kLdsBlocks);
    row.start(base * kTiles, count * kTiles, MassRun::kOne);
    row.sweep(base * kTiles, count * kTiles, MassRun::kOne, true, [&](int x, MassRun::Scores& sc) {
      float sum[QG];
      tile_sums(sc, sum);
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) part[qg] += sum[qg];
      if (kTiles == 1 || x % kTiles == kTiles - 1) {
        sums[x / kTiles - base][query] = collected(part);
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) part[qg] = 0.0f;
      }
    });
    flush(base, count);
  }
}

typedef QueryRun<false> Run;
struct TokenBudgets {
  int32_t k[SHPLB_MAX_TOKEN_BUDGETS];
};

// The order in which workgroups take the rows, which lie in order of their length.  The counting sweep of the token recovery
// waits for LDS, the last one for the VALU, and the dispatcher puts workgroup b beside workgroup b - (compute units), which has
// a row of the same length: the two went through the same sweeps at the same time.  Now the second lap of compute units starts
// on rows of half the length, after which one of the pair counts while the other sums, for most of the launch (the rows get shorter
// slowly).  12345 tokens x 32 heads, four budgets: 6.92 -> 6.60 ms; 6001 x 28, two: 832 -> 814 us; 16K x 32, one: 3.04 -> 3.01 ms;
// 32K, at the card's power limit, 0.3 to 1%.  A third or two thirds of the length: less, at 6001 tokens slower than none.
// Launches of fewer than five laps, or whose rows of half the length are part of the first, keep their order: with 3.5 laps
// (3576 tokens x 32, three budgets) 568 -> 582 us, with 5.1 (6001 x 28) as above.
// In a batch the laps also count workgroups whose sequence is shorter, which return at once and leave less of the pairing
// above.  19 batches of equal and unequal sequences, one to five budgets: 12000 and 11000 tokens x 28/4 heads, three budgets, 8.32 ->
// 8.10 ms, 20000 and three of 1000 x 4/2 2.31 -> 2.24 ms, eight of 3000 x 8/2 310 -> 301 us; most within 1%, the least
// favourable 2000 and thirty of 10 tokens x 8, 170.9 -> 172.4 us.
struct Laps {
  uint32_t lap, half;                                // workgroups of a lap, the first row of half the longest's length
  __device__ __forceinline__ uint32_t index_of(uint32_t b) const {
    if (b < lap) return b;
    if (b - lap < lap) return half + b - lap;
    return b - lap < half ? b - lap : b;             // those before the second lap's rows, then those behind them
  }
};

// Sum of the k largest attention weights of every query, for M budgets k at once.
//
// The weight of a key grows with its raw score, so the k largest weights belong to the k largest scores.
// The triangle of scores fits nowhere: every question about it is a sweep over the keys that computes them
// again, and the kernel is bound by the number of sweeps.  Per query it needs two, and a little sampling:
//
//   1. a few tiles, evenly spread, give the range of the query's scores, then a histogram of a few more tiles
//      over that range gives an interval that should hold the k-th largest score (a guess only: the sampled
//      keys of the last tiles may be ones the query does not see; scores that are no numbers are left out);
//   2. a sweep counts the scores in kBins bins over the interval, the outermost ones open: the bin that holds
//      the k-th largest is known, and how many scores lie above it.  With more keys in the bin than there
//      is room for, or with the k-th largest in an open bin, the sweep is done again over that bin or over
//      what lies beyond.  A bin no wider than the resolution of a score (ties) needs no more division, nor does
//      the lower open bin once it lies so far below the largest score that its weights are zero (-inf among them);
//   3. the last sweep takes the exponentials: their sum, the sum of those above the bin, and the scores in
//      the bin to a list.  The list gives the few weights that are missing.
//
// Counters are a word per (bin, query) in LDS, private to the query's wave, in the bank of its lane: an
// LDS atomic without a result, and nothing of the search is held in registers but the map from scores to
// bins.  Bins are taken as x = fma(score, a, b) around 2^23, where a float is a whole number and its low bits
// are the bin: rounding keeps the order of the scores, so bins are exact intervals whatever a and b are.
// The list takes the counters' place; the two lanes of a query fill it from its two ends.
// Sums are per tile first, then over tiles, always in the same order: results repeat bit for bit.
//
// 32 heads x 32K tokens, k = 4096: 11.5 to 12.0 ms on several cards, against 131 ms with the threshold found bit by bit in 27
// to 29 sweeps; three budgets at 4000 tokens x 16 heads 520 us.  The two sweeps and the samples would take 6.8 ms without any
// work on the scores, which is what their MFMAs, 2.05 passes of products, take at the card's power limit (1.32 PFLOP/s, at
// 1.5 GHz; the whole kernel runs at 2.1 GHz).  Three waves per SIMD (tiles of 32 keys, 74 bins) were slower, 16.4 ms; so were workgroups of eight waves
// that share a tile, 2.5%, also with half of the waves doing their MFMAs behind the work on the scores, 6%.
constexpr int kBins = 95;                          // and the longest list: 128 queries x 95 words leave room for
                                                   // two workgroups per compute unit beside the tiles
constexpr int kInner = 85, kFirst = 5;             // an interval is spread over bins kFirst .. kFirst + kInner
constexpr float kWhole = 8388608.0f;               // 2^23
constexpr int kRangeTiles = 256 / Run::kTile, kSampleTiles = 2048 / Run::kTile;  // tiles sampled for the range, and at most for the interval
// Tiles of a row that is searched over its whole range at once: sampling costs such rows as much as the sweep it
// would save (384 and 768 keys alike; with 1536, 1391 tokens x 28 heads, three budgets, take 365 instead of 262 us)
constexpr int kSmallRow = 768 / Run::kTile;
constexpr float kFar = 0x1p126f;                   // intervals end here, so that their widths are numbers
constexpr float kNoWeight = 160.0f;                // 2^-160 is zero: so far below the largest, in log2 units of weight
// Sweeps of a search at most.  One that divides the interval leaves 1/42 of it or less, one beyond it reaches 32 times as
// far: some ten at most between the far end of an interval and ties.  Still open then (k-th scores beyond kFar): NaN.
constexpr int kSearchRounds = 64, kUnknown = -1;

template <int M>
__global__ __launch_bounds__(256, 2) void token_recovery_kernel(SeqMeta meta, Strides st,
                                                                const uint16_t* __restrict__ q,
                                                                const uint16_t* __restrict__ k,
                                                                float* __restrict__ recovery, TokenBudgets budgets,
                                                                int n_out, int levels, Laps laps, float scale_log2,
                                                                int total_tokens) {
  typedef __attribute__((address_space(3))) uint32_t LdsWord;
  typedef __attribute__((address_space(3))) float LdsFloat;
  constexpr int MT = Run::MT;
  constexpr uint32_t kBinBytes = 32 * 4;           // a word for each of a wave's queries
  __shared__ __attribute__((aligned(1024))) char k_lds[2][Run::kStageBytes];
  __shared__ __attribute__((aligned(16))) uint32_t s_bins[Run::kWaves][kBins][32];
  __shared__ int s_open[2][Run::kWaves];

  Run row;
  if (!row.init(meta, st, k, levels, &k_lds[0][0], laps.index_of(blockIdx.x))) return;
  const int visible = row.q_tok - row.seq_begin + 1;          // keys the lane's query sees
  int fewest = budgets.k[0];
#pragma unroll
  for (int b = 1; b < M; ++b) fewest = min(fewest, budgets.k[b]);
  auto store = [&](int b, float r) {
    if (b < n_out && row.hi == 0 && row.live())
      recovery[(int64_t(b) * meta.n_q_heads + row.h) * total_tokens + row.q_tok] = r;
  };
  if ((row.i + 1) * Run::kQueries <= fewest) {           // no query sees more keys than any budget
#pragma unroll
    for (int b = 0; b < M; ++b) store(b, 1.0f);
    return;
  }
  const int all = row.n_tiles;
  const int n_range = all <= kSmallRow ? all : kRangeTiles;
  const int n_sample = all <= kSmallRow ? 0 : max(kRangeTiles, min(all / 16, kSampleTiles));
  uint32_t stride = row.stride_of(n_range);
  row.start(0, n_range, stride);
  row.load_queries(st, q);

  const uint32_t column = lds_offset_of(&s_bins[row.wave][0][0]) + 4 * row.n;      // the query's words, kBinBytes apart
  const uint32_t bin_base = column - (__builtin_bit_cast(uint32_t, kWhole) << 7);  // + bits of kWhole + bin << 7
  static_assert(kBinBytes == 1 << 7, "shifts above and below");
  auto word = [&](int x) { return reinterpret_cast<LdsWord*>(column + x * kBinBytes); };
  auto entry = [&](int x) { return reinterpret_cast<LdsFloat*>(column + x * kBinBytes); };
  auto fence = [] { asm volatile("" ::: "memory"); };         // the words of a wave are its own: order in the program is enough
  auto clear = [&] {
    fence();
    for (int x = row.hi; x < kBins; x += 2) *word(x) = 0;
    fence();
  };
  // least useful width of a bin around scores lo .. hi: half the distance of neighbouring floats, or what
  // changes a weight by 2^-26 of itself
  const float unit = 1.0f / scale_log2;                       // scores that a weight halves over
  auto finest = [&](float lo, float hi) {
    const float least = fmaxf(fmaxf(fabsf(lo), fabsf(hi)) * 0x1p-24f, 0x1p-26f * unit);
    return __builtin_amdgcn_fmed3f(least, 0x1p-120f, 0x1p119f);
  };
  auto finite = [](float s) { return __builtin_amdgcn_classf(s, 0x1f8); };   // neither an infinity nor a NaN
  float bin_lo, bin_w, map_a, map_b;                          // interval's begin, width of a bin, x = fma(score, map_a, map_b)
  bool ties;                                                  // bins hold one score each (as far as a weight can tell)
  auto spread = [&](float lo, float hi) {
    lo = __builtin_amdgcn_fmed3f(lo, -kFar, kFar);
    hi = __builtin_amdgcn_fmed3f(hi, -kFar, kFar);
    const float least = finest(lo, hi);
    bin_lo = lo;
    bin_w = fmaxf((hi - lo) * (1.0f / kInner), least);
    ties = bin_w <= least;
    map_a = 1.0f / bin_w;
    map_b = (kWhole + kFirst) - map_a * lo;
  };
  auto bin_begin = [&](int u) { return bin_lo + (float(u - kFirst) - 0.5f) * bin_w; };
  float top_score = -INFINITY;
  auto count_bins = [&](int, Run::Scores& sc) {
    // Addresses of four scores, then their atomics: score after score, every atomic waited for three dependent operations in
    // one register (32K x 32 heads 12.0 -> 11.7 ms; two or eight at a time take as long, within 0.5%, at 32K and up to 3% more
    // at 1500 tokens).
    constexpr int G = 4;
#pragma unroll
    for (int g = 0; g < 16 * MT; g += G) {
      uint32_t at[G];
#pragma unroll
      for (int r = 0; r < G; ++r) {
        const float s = sc.v[(g + r) / 16][(g + r) % 16];
        const float x = __builtin_amdgcn_fmed3f(__builtin_fmaf(s, map_a, map_b), kWhole, kWhole + (kBins - 1));
        at[r] = (__builtin_bit_cast(uint32_t, x) << 7) + bin_base;
        top_score = fmaxf(top_score, s);
      }
#pragma unroll
      for (int r = 0; r < G; ++r) asm volatile("" : "+v"(at[r]));   // all four, before the first atomic
      asm volatile("" : "+v"(top_score));
#pragma unroll
      for (int r = 0; r < G; ++r)
        __hip_atomic_fetch_add(reinterpret_cast<LdsWord*>(at[r]), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  };
  // the bin that holds the rank-th largest score: how many scores lie above it and in it
  auto find = [&](int rank, int& bin, int& above, int& inside) {
    fence();
    int c = 0;
    bin = above = inside = 0;
#pragma unroll 5
    for (int x = kBins - 1; x >= 0; --x) {
      const int here = int(*word(x));
      if (c < rank && c + here >= rank) {
        bin = x;
        above = c;
        inside = here;
      }
      c += here;
    }
  };

  // ---- 1. where to look
  float lo = INFINITY, hi = -INFINITY;
  row.sweep(0, n_range, stride, n_sample == 0, [&](int, Run::Scores& sc) {
    float top = sc.v[0][0], low = top;
#pragma unroll
    for (int r = 1; r < 16 * MT; ++r) {
      top = fmaxf(top, sc.v[r / 16][r % 16]);
      low = fminf(low, sc.v[r / 16][r % 16]);
    }
    if (__any(!finite(top) || !finite(low))) {                // (masked keys among them)
      top = -INFINITY;
      low = INFINITY;
#pragma unroll
      for (int r = 0; r < 16 * MT; ++r) {
        const float s = sc.v[r / 16][r % 16];
        const bool counts = finite(s);
        top = fmaxf(top, counts ? s : -INFINITY);
        low = fminf(low, counts ? s : INFINITY);
      }
    }
    hi = fmaxf(hi, top);
    lo = fminf(lo, low);
  });
  hi = pair_max(hi);
  lo = -pair_max(-lo);
  if (lo > hi) lo = hi = 0.0f;
  float from[M], to[M];
#pragma unroll
  for (int b = 0; b < M; ++b) {
    from[b] = lo;
    to[b] = hi;
  }
  if (n_sample > 0) {
    stride = row.stride_of(n_sample);
    row.start(0, n_sample, stride);
    clear();
    spread(lo, hi);
    row.sweep(0, n_sample, stride, false, count_bins);
    const float n_keys = float(n_sample * Run::kTile), share = n_keys / float(visible);
    top_score = pair_max(top_score);
    const float sample_top = finite(top_score) ? top_score : hi + kInner * bin_w;
#pragma unroll
    for (int b = 0; b < M; ++b) {
      // the rank in the sample is off by its standard deviation; four of them
      const float rank = fminf(float(budgets.k[b]) * share, n_keys);
      const float off = 4.0f * __builtin_sqrtf(fmaxf(rank * (1.0f - rank / n_keys), 0.0f)) + 4.0f;
      int bin, above, inside;
      find(max(1, int(rank - off)), bin, above, inside);
      to[b] = bin < kBins - 1 && rank > off ? bin_begin(bin + 1) : sample_top;
      find(min(n_sample * Run::kTile, int(rank + off)), bin, above, inside);
      from[b] = bin > 0 ? bin_begin(bin) : bin_begin(0) - kInner * bin_w;
    }
  }

  // ---- 2. the bin of the k-th largest score, budget after budget
  float above_from[M], list_from[M];                          // scores from which on: above the bin, in the bin or above
  int rest[M], listed[M], list_at[M];                         // keys wanted from the bin, entries and place of its list
  bool tied[M];                                               // all scores of the bin count as one: the list is that one
  int used = 0, round = 0;
#pragma unroll
  for (int b = 0; b < M; ++b) {
    above_from[b] = list_from[b] = INFINITY;
    rest[b] = listed[b] = list_at[b] = 0;
    tied[b] = false;
  }
  stride = Run::kOne;
  for (int b = 0; b < n_out; ++b) {
    int want = 0;
    float f = 0.0f, t = 0.0f;
#pragma unroll
    for (int x = 0; x < M; ++x)
      if (x == b) {
        want = budgets.k[x];
        f = from[x];
        t = to[x];
      }
    bool open = row.live() && visible > want;
    const bool search = open;
    const int room = (kBins - used) / (n_out - b);
    int bin = 0, above = 0, inside = 0;
    spread(f, t);
    for (int tries = 0;; ++tries, ++round) {
      // does any query of the workgroup still search?  (two flag sets: a wave may write the next
      // round's flag while another still reads this round's; the sweep's barriers separate the rounds)
      if (row.lane == 0) s_open[round & 1][row.wave] = 0;
      if (__any(open) && row.lane == 0) s_open[round & 1][row.wave] = 1;
      __syncthreads();
      int any_open = 0;
#pragma unroll
      for (int w = 0; w < Run::kWaves; ++w) any_open |= s_open[round & 1][w];
      if (!__builtin_amdgcn_readfirstlane(any_open) || tries == kSearchRounds) break;
      row.start(0, all, stride);
      clear();
      top_score = -INFINITY;                                  // (the samples' may be a key the query does not see)
      row.sweep(0, all, stride, true, count_bins);
      top_score = pair_max(top_score);
      if (open) {
        find(want, bin, above, inside);
        // beyond the interval: most often just beyond
        const float reach = (tries == 0 ? 2.0f : 32.0f) * kInner * bin_w;
        const float nothing = fmaxf(top_score - kNoWeight * unit, -kFar);   // no weight from here down
        if (!finite(top_score)) {
          open = false;                                       // the weights are no numbers, nor will the result be one
        } else if (bin == 0) {
          if (bin_begin(1) + bin_w <= nothing) open = false;  // all keys that weigh anything are among the k largest
          else spread(fmaxf(bin_begin(1) - reach, nothing), bin_begin(1) + bin_w);
        } else if (bin == kBins - 1) {
          spread(bin_begin(kBins - 1) - bin_w, tries == 0 ? fminf(bin_begin(kBins - 1) + reach, top_score) : top_score);
        } else if (inside <= room || ties) {
          open = false;
        } else {
          const float low = bin_begin(bin) - 0.5f * bin_w, high = bin_begin(bin + 1) + 0.5f * bin_w;
          spread(low, high);
        }
      }
    }
    ++round;
    // the least scores that fall on bins `bin` and `bin + 1`: the map keeps the order, so by bisection
    auto least_score = [&](float x) {
      int low = int(0x80800000), high = 0x7f7fffff;           // floats as integers of the same order
      while (low < high) {
        const int mid = int((int64_t(low) + high) >> 1);
        const float s = __builtin_bit_cast(float, mid ^ ((mid >> 31) & 0x7fffffff));
        if (__builtin_fmaf(s, map_a, map_b) >= x) high = mid;
        else low = mid + 1;
      }
      return __builtin_bit_cast(float, low ^ ((low >> 31) & 0x7fffffff));
    };
    const bool listing = search && bin > 0;                   // (none of the lower open bin's weigh anything)
    const float least_in = listing ? least_score(kWhole + float(bin)) : INFINITY;
    const float least_above = search ? least_score(kWhole + float(bin + 1)) : INFINITY;
    const bool tie = inside > room;
    const int entries = tie ? 1 : inside;
#pragma unroll
    for (int x = 0; x < M; ++x)
      if (x == b) {
        list_from[x] = least_in;
        above_from[x] = least_above;
        rest[x] = open ? kUnknown : want - above;
        listed[x] = listing ? entries : 0;
        list_at[x] = used;
        tied[x] = tie;
      }
    if (listing) used += entries;
  }

  // ---- 3. weights
  row.start(0, all, stride);
  const float ref = top_score * scale_log2;
  auto weight = [&](float s) { return __builtin_amdgcn_exp2f(__builtin_fmaf(s, scale_log2, -ref)); };
  uint32_t put[M];                                            // where the lane's next entry goes
  float sum = 0.0f, top[M];
#pragma unroll
  for (int b = 0; b < M; ++b) {
    put[b] = column + (list_at[b] + (row.hi == 0 || tied[b] ? 0 : listed[b] - 1)) * kBinBytes;
    top[b] = 0.0f;
  }
  fence();
  // Sums and masks of a group of scores first, without a branch; then the scores of the group that go to a list, which few
  // do: a scalar test and a branch each.  (With the branch behind every score's own comparison a score waited for its
  // exponential, two comparisons and four scalar operations before the next one began; 32K x 32 heads, one budget: 12.4 ->
  // 11.9 ms, 6001 tokens x 28 heads, two: 903 -> 818 us; eight: 3000 tokens x 8/2 heads 1185 -> 957 us, 8000 x 32/8 7.98 -> 6.84
  // ms.  Groups of 8 over all budgets take up to 2% more.  The masks cost scalar registers: 5, 14, 38 and 90 of them are
  // spilled with 1, 2, 4 and 8 budgets; with groups of 32 104 to 586 are, which is as slow as no groups.)
  constexpr int G = 16 / M;
  row.sweep(0, all, stride, true, [&](int, Run::Scores& sc) {
    float sum0 = 0.0f, sum1 = 0.0f, part[M];
#pragma unroll
    for (int b = 0; b < M; ++b) part[b] = 0.0f;
#pragma unroll
    for (int g = 0; g < 16 * MT; g += G) {
      auto score = [&](int r) { return sc.v[(g + r) / 16][(g + r) % 16]; };
      uint64_t in[M][G];                                      // lanes whose score goes to the list
      float p[G];
#pragma unroll
      for (int r = 0; r < G; ++r) p[r] = weight(score(r));
#pragma unroll
      for (int r = 0; r < G; ++r) {
        if (r & 1) sum1 += p[r];
        else sum0 += p[r];
#pragma unroll
        for (int b = 0; b < M; ++b) {
          const bool over = score(r) >= above_from[b];
          part[b] += over ? p[r] : 0.0f;
          in[b][r] = __builtin_amdgcn_ballot_w64(score(r) >= list_from[b]) & ~__builtin_amdgcn_ballot_w64(over);
        }
      }
      asm volatile("" : "+v"(sum0), "+v"(sum1));              // here, not behind the branches
#pragma unroll
      for (int b = 0; b < M; ++b) asm volatile("" : "+v"(part[b]));
#pragma unroll
      for (int r = 0; r < G; ++r)
#pragma unroll
        for (int b = 0; b < M; ++b)
          if (in[b][r] != 0) {
            if (__builtin_amdgcn_inverse_ballot_w64(in[b][r])) {
              // (a place outside the query's words is none of a list's: held inside, without a branch, 11.9 -> 11.6 ms)
              *reinterpret_cast<LdsFloat*>(column + min(put[b] - column, (kBins - 1) * kBinBytes)) = score(r);
              if (!tied[b]) put[b] += row.hi == 0 ? kBinBytes : 0u - kBinBytes;
            }
          }
    }
    sum += sum0 + sum1;
#pragma unroll
    for (int b = 0; b < M; ++b) top[b] += part[b];
  });
  fence();
  const float total = pair_sum(sum);

  // ---- the rest of the budget from the list: its rest-th largest entry, halving the range of floats until the
  // entries from there on are as many as wanted (or all equal there)
  auto both = [](int c) {
    float x, y;
    pair_values(__int_as_float(c), x, y);
    return __float_as_int(x) + __float_as_int(y);
  };
  auto ordered = [](float s) {
    const int v = __float_as_int(s);
    return v ^ ((v >> 31) & 0x7fffffff);
  };
#pragma unroll
  for (int b = 0; b < M; ++b) {
    const bool search = listed[b] > 0;
    const int end = listed[b];
    int low = search ? ordered(list_from[b]) : 0, high = search ? ordered(above_from[b]) : 0;   // [low, high)
    auto from_on = [&](int v) {
      int c = 0;
      for (int x = row.hi; x < end; x += 2) c += ordered(*entry(list_at[b] + x)) >= v ? 1 : 0;
      return both(c);
    };
    bool open = search && !tied[b] && rest[b] < end;
    while (__any(open)) {
      const int mid = low + int((uint32_t(high) - uint32_t(low)) >> 1);
      const int c = from_on(mid);
      if (open) {
        if (c >= rest[b]) low = mid;
        else high = mid;
        if (c == rest[b] || uint32_t(high) - uint32_t(low) <= 1u) open = false;
      }
    }
    float part = 0.0f;
    int more = 0;
    float at = 0.0f;
    for (int x = row.hi; x < end; x += 2) {
      const float s = *entry(list_at[b] + x);
      at = weight(s);
      if (tied[b] || ordered(s) >= low) {
        part += at;
        more += 1;
      }
    }
    // ties at the place of the k-th: as many as wanted of entries that are all alike
    more = both(more);
    float r = pair_sum(top[b]) + pair_sum(part);
    if (search && more != rest[b]) {
      float w = 0.0f;
      // entries equal to the smallest one taken
      w = tied[b] ? weight(*entry(list_at[b])) : weight(__builtin_bit_cast(float, low ^ ((low >> 31) & 0x7fffffff)));
      r += float(rest[b] - more) * w;
    }
    r /= total;
    if (rest[b] == kUnknown) r = __uint_as_float(0x7fc00000u);
    if (visible <= budgets.k[b]) r = 1.0f;
    store(b, r);
  }
}

template <int M>
void launch_token_recovery_as(const Geometry& g, const uint16_t* q, const uint16_t* k, float* recovery,
                              const TokenBudgets& budgets, int n_out, int levels, Laps laps, uint32_t n_wg, hipStream_t stream) {
  hipLaunchKernelGGL((token_recovery_kernel<M>), dim3(n_wg), dim3(2 * Run::kQueries), 0, stream, g.meta, g.st, q, k,
                     recovery, budgets, n_out, levels, laps, g.scale * 1.4426950408889634f, int(g.total_tokens));
}

}  // namespace

int32_t launch_block_mass(const Geometry& g, const void* q, const void* k, float* mass, hipStream_t stream) {
  const SeqMeta& m = g.meta;
  const int levels = (g.max_nb * m.block + MassRun::kQueries - 1) / MassRun::kQueries;
  const int64_t n_wg = int64_t(levels) * m.n_seq * m.n_q_heads;
  if (n_wg > 0x7fffffff) return SHPLB_E_UNSUPPORTED;
  const float scale_log2 = g.scale * 1.4426950408889634f;
  const auto kernel = m.block == 128 ? mass_kernel<128> : mass_kernel<64>;
  hipLaunchKernelGGL(kernel, dim3(uint32_t(n_wg)), dim3(2 * MassRun::kQueries), 0, stream, m, g.st,
                     static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k), mass, levels, scale_log2);
  if (hipGetLastError() != hipSuccess) return SHPLB_E_HIP;
  return SHPLB_OK;
}

int32_t launch_token_recovery(const Geometry& g, const void* q, const void* k, const int32_t* budgets,
                              int32_t n_budgets, float* recovery, hipStream_t stream) {
  const SeqMeta& m = g.meta;
  const int levels = (g.max_nb * m.block + Run::kQueries - 1) / Run::kQueries;
  const int64_t n_wg = int64_t(levels) * m.n_seq * m.n_q_heads;
  if (n_wg > 0x7fffffff) return SHPLB_E_UNSUPPORTED;
  TokenBudgets kb;
  for (int b = 0; b < SHPLB_MAX_TOKEN_BUDGETS; ++b) kb.k[b] = budgets[std::min(b, n_budgets - 1)];
  const uint16_t* qp = static_cast<const uint16_t*>(q);
  const uint16_t* kp = static_cast<const uint16_t*>(k);
  const uint32_t wg = uint32_t(n_wg);
  const int32_t resident = persistent_workgroups();            // two laps
  if (resident < 0) return SHPLB_E_HIP;
  Laps laps{uint32_t(resident / 2), uint32_t(levels / 2) * m.n_seq * m.n_q_heads};
  if (laps.half < laps.lap || int64_t(laps.half) + laps.lap > n_wg || n_wg < 5 * int64_t(laps.lap)) laps.lap = 0x7fffffff;
  if (n_budgets <= 1) launch_token_recovery_as<1>(g, qp, kp, recovery, kb, n_budgets, levels, laps, wg, stream);
  else if (n_budgets <= 2) launch_token_recovery_as<2>(g, qp, kp, recovery, kb, n_budgets, levels, laps, wg, stream);
  else if (n_budgets <= 4) launch_token_recovery_as<4>(g, qp, kp, recovery, kb, n_budgets, levels, laps, wg, stream);
  else launch_token_recovery_as<8>(g, qp, kp, recovery, kb, n_budgets, levels, laps, wg, stream);
  if (hipGetLastError() != hipSuccess) return SHPLB_E_HIP;
  return SHPLB_OK;
}

}  // namespace shplb
