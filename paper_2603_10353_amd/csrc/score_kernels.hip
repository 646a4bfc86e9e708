// Block importance: mean-pool query/key blocks (HBM-bound streaming reduction), then
// pooled logits for the causal lower triangle (a small contraction, fp32 values carried
// as three bf16 planes so that it runs on the bf16 matrix pipe).
#include "attn_common.h"

namespace shplb {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kPoolThreads = 256;
constexpr int kPoolWaves = 4;
constexpr int kPoolElems = 512;   // bf16 elements of a token row covered by one workgroup

__device__ __forceinline__ void add_bf16x8(float (&acc)[8], const u32x4 w) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    acc[2 * c] += __uint_as_float(w[c] << 16);
    acc[2 * c + 1] += __uint_as_float(w[c] & 0xffff0000u);
  }
}

// One workgroup = one block of tokens x 512 consecutive (head, dim) elements.
// The four waves take every fourth token; each lane owns 8 consecutive dims and
// keeps fp32 sums; partial sums meet in LDS in a fixed order (deterministic).  The
// fp32 mean v leaves as three bf16 planes v1 = bf16(v), v2 = bf16(v - v1), v3 = bf16(v - v1 - v2)
// (round to nearest even; the differences are exact in fp32), each plane [heads][blocks][128].
// blockIdx.x enumerates first the Q tiles, then the K tiles.
// Two workgroups per compute unit with 16 loads of 16 bytes in flight per lane: fewer, longer
// streams suit the memory better than full occupancy with 8 in flight (213 against 224 us at
// 128K tokens of a 32/8-head layer).
__global__ __launch_bounds__(kPoolThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void pool_kernel(
    SeqMeta meta, Strides st, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    uint16_t* __restrict__ q_planes, uint16_t* __restrict__ k_planes, int q_chunks, int k_chunks,
    int total_blocks) {
  __shared__ float part[kPoolWaves][kPoolElems];
  // what a single sequence needs of the arguments is loaded together, before the first use
  asm volatile("" ::"s"(q_chunks), "s"(k_chunks), "s"(total_blocks), "s"(meta.n_seq), "s"(meta.n_q_heads), "s"(meta.n_kv_heads), "s"(meta.block),
               "s"(meta.tok_begin[1]), "s"(q), "s"(k), "s"(q_planes), "s"(k_planes), "s"(st.q_t), "s"(st.q_h),
               "s"(st.kv_t), "s"(st.kv_h));
  int bid = blockIdx.x;
  const bool is_q = bid < total_blocks * q_chunks;
  if (!is_q) bid -= total_blocks * q_chunks;
  const int chunks = is_q ? q_chunks : k_chunks;
  const int gblk = bid / chunks;
  const int chunk = bid - gblk * chunks;
  const int n_heads = is_q ? meta.n_q_heads : meta.n_kv_heads;
  const uint16_t* src = is_q ? q : k;
  const int64_t stride_t = is_q ? st.q_t : st.kv_t;
  const int64_t stride_h = is_q ? st.q_h : st.kv_h;
  uint16_t* dst = is_q ? q_planes : k_planes;
  const int64_t plane = int64_t(n_heads) * total_blocks * kHeadDim;

  int t0 = gblk * meta.block, t1 = meta.tok_begin[1];
  if (meta.n_seq > 1) {
    // a lane per sequence: how many end at or before the block, and the rest from the lane of its own
    const int lane = threadIdx.x & 63, blk_end = meta.blk_begin[lane + 1], tok = meta.tok_begin[lane], tok_end = meta.tok_begin[lane + 1];
    const int s = __builtin_popcountll(__ballot(lane < meta.n_seq - 1 && gblk >= blk_end));
    const int first = s > 0 ? __builtin_amdgcn_readlane(blk_end, s - 1) : 0;
    t0 = __builtin_amdgcn_readlane(tok, s) + (gblk - first) * meta.block;
    t1 = __builtin_amdgcn_readlane(tok_end, s);
  }
  t1 = min(t1, t0 + meta.block);
  const int cnt = t1 - t0;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e = chunk * kPoolElems + lane * 8;          // element inside the [heads*128] token row
  const int head = e >> 7, dim = e & 127;
  const bool live = head < n_heads;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (live) {
    const uint16_t* base = src + head * stride_h + dim;
    int t = t0 + wave;
    constexpr int U = 16;             // loads in flight per lane
    for (; t + (U - 1) * kPoolWaves < t1; t += U * kPoolWaves) {
      u32x4 w[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + int64_t(t + u * kPoolWaves) * stride_t));
#pragma unroll
      for (int u = 0; u < U; ++u) add_bf16x8(acc, w[u]);
    }
    // What is left of a ragged block, in flight together likewise (loads past the end repeat the last token;
    // one load after the other, a block of 127 tokens took 15 memory round trips: 48 ragged sequences 22.2 -> 19.5 us,
    // the whole path of an 8231-token prompt 184.5 -> 182.7 us).
    const int left = __builtin_amdgcn_readfirstlane((t1 - t + kPoolWaves - 1) / kPoolWaves);
    if (left > 0) {
      u32x4 w[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + int64_t(min(t + u * kPoolWaves, t1 - 1)) * stride_t));
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (u < left) add_bf16x8(acc, w[u]);
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) part[wave][lane * 8 + c] = acc[c];
  __syncthreads();
  {
    const int x = 2 * threadIdx.x;                  // two neighbouring dims per thread
    const int ee = chunk * kPoolElems + x;
    const int hh = ee >> 7, dd = ee & 127;
    if (hh < n_heads) {
      float v0 = (((part[0][x] + part[1][x]) + part[2][x]) + part[3][x]) / float(cnt);
      float v1 = (((part[0][x + 1] + part[1][x + 1]) + part[2][x + 1]) + part[3][x + 1]) / float(cnt);
      if (is_q) {
        // query means stay fp32: the scoring kernel loads each row into registers anyway and splits it
        // there (two thirds of the bytes of three planes, on a buffer that is written once and read 2.5 times)
        float* qm = reinterpret_cast<float*>(q_planes) + (int64_t(hh) * total_blocks + gblk) * kHeadDim + dd;
        *reinterpret_cast<float2*>(qm) = float2{v0, v1};
        return;
      }
      uint16_t* at = dst + (int64_t(hh) * total_blocks + gblk) * kHeadDim + dd;
#pragma unroll
      for (int pl = 0; pl < 3; ++pl) {
        const __bf16 b0 = (__bf16)v0, b1 = (__bf16)v1;
        *reinterpret_cast<uint32_t*>(at + pl * plane) =
            uint32_t(__builtin_bit_cast(uint16_t, b0)) | uint32_t(__builtin_bit_cast(uint16_t, b1)) << 16;
        v0 -= float(b0);
        v1 -= float(b1);
      }
    }
  }
}

// scores[s][h][i][j] = (qbar[h][i] . kbar[h/G][j]) * scale for j <= i.
//
// fp32 products on the bf16 matrix pipe.  The pooling kernel stores every pooled value v as
// three bf16 planes v = v1 + v2 + v3 (v1 = bf16(v), v2 = bf16(v - v1), v3 = bf16(v - v1 - v2):
// all 24 mantissa bits), and a product is taken as q1k1 + q1k2 + q2k1 + q2k2 + q1k3 + q3k1;
// the dropped cross terms are below 2^-24 of the product, what an fp32 multiply rounds away
// anyway.  Six v_mfma_f32_32x32x16_bf16 do the work of eight v_mfma_f32_32x32x2_f32 in
// 3/8 of the time.
//
// One workgroup = 128 query-block rows (32 per wave; see kWaves) of one (sequence, head) x a chunk of
// key-block rows, streamed in tiles of 32 through a double-buffered LDS stage; three
// workgroups share a compute unit and hide each other's copy latency.  The Q planes of a
// wave's rows stay in registers as MFMA B-operands; a K tile is 3 planes x 32 rows of 256
// bytes, copied global->LDS directly and laid out like the K tiles of the attention kernels
// (chunk c of row r at slot c ^ swz(r)).  Lane (n, hi) ends up with row i = n of the 32x32
// output tile and four runs of four consecutive j: 16-byte stores.  Two accumulators take
// the six products in turn (no MFMA waits for the one before it) and are added at the end;
// the order of additions is fixed.
// Launches of few rows (kWaves = 1, see the rule in launch_pool_scores()) take workgroups of one wave, one K tile and one
// LDS stage: of sequences of up to 32 blocks three of four waves would have no row, and half as many workgroups would fit a
// compute unit.  (Whole path, 48 short sequences x 28 heads 159.0 -> 153.3 us.)
constexpr int kScoreJ = 32;                           // key-block rows per LDS stage
constexpr int kPlanes = 3;
constexpr int kScoreStageBytes = kPlanes * kScoreJ * kRowBytes;   // 24 KB
// chunks (of 2^log_chunk key-block rows) that hold some j <= i for the rows of tile row tr
__host__ __device__ constexpr int score_chunks_of_row(int tr, int log_chunk, int tile) {
  return ((tr * tile + tile - 1) >> log_chunk) + 1;
}

template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(3, 3))) void score_kernel(
    SeqMeta meta, const uint16_t* __restrict__ q_planes, const uint16_t* __restrict__ k_planes,
    float* __restrict__ scores, int total_blocks, int log_chunk, float scale) {
  constexpr int kScoreTile = 32 * kWaves;               // query-block rows per workgroup
  __shared__ __attribute__((aligned(1024))) char k_lds[kWaves == 1 ? 1 : 2][kScoreStageBytes];
  // what needs no sequence is loaded together, before the first use
  asm volatile("" ::"s"(meta.n_q_heads), "s"(meta.n_kv_heads), "s"(meta.kv_map), "s"(q_planes), "s"(k_planes), "s"(scores), "s"(total_blocks),
               "s"(log_chunk), "s"(scale));
  const int sh = blockIdx.z;
  const int s = small_quotient(sh, meta.n_q_heads), h = sh - s * meta.n_q_heads;
  const int nb = meta.blk_begin[s + 1] - meta.blk_begin[s];
  // blockIdx.x enumerates (128-row tile of query blocks, chunk of key blocks) pairs of the
  // lower triangle, tile row by tile row.  Consecutive workgroup ids go to different XCDs,
  // so every die gets the same share of live work (a square grid would hand die x the whole
  // chunk column x, most of which lies above the diagonal for large x).
  int tr = 0, rest = int(blockIdx.x);
  while (rest >= score_chunks_of_row(tr, log_chunk, kScoreTile)) rest -= score_chunks_of_row(tr++, log_chunk, kScoreTile);
  const int ti = tr * kScoreTile, chunk = 1 << log_chunk, tj = rest << log_chunk;
  if (ti >= nb) return;                             // shorter sequence of a varlen batch
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hi = lane >> 5;
  const int g = meta.kv_map ? kv_head_of(meta, h) : small_quotient(h, small_quotient(meta.n_q_heads, meta.n_kv_heads));
  const int i_first = ti + 32 * wave;               // this wave's rows
  const int i_last = min(ti + kScoreTile, nb) - 1;  // last row of the workgroup
  if (tj > i_last) return;                          // chunk entirely right of a short sequence's last row (before any copy is issued)
  const int n_jt = (min(tj + chunk, i_last + 1) - tj + kScoreJ - 1) / kScoreJ;   // 32-row K tiles with some j <= i
  const int64_t k_plane = int64_t(meta.n_kv_heads) * total_blocks * kHeadDim;
  const char* k_rows = reinterpret_cast<const char*>(k_planes + (int64_t(g) * total_blocks + meta.blk_begin[s]) * kHeadDim);

  // copies: a round fills 4 kWaves consecutive tile rows of one plane; a lane's row is its own in each
  constexpr int kRoundRows = 4 * kWaves;
  const int cp_row = 4 * wave + (lane >> 4);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_offset_of(&k_lds[0][0]) + 4 * wave * kRowBytes);
  auto issue_tile = [&](int jt, int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int rd = 0; rd < kScoreJ / kRoundRows; ++rd) {
      const int jl = kRoundRows * rd + cp_row;
      // Rows past the end: repeat the last one, or leave what is there (a column j of the scores depends on
      // row j alone, and these are never stored).
      if (kWaves == 1 && tj + kScoreJ * jt + kRoundRows * rd >= nb) break;
      const int j = min(tj + kScoreJ * jt + jl, nb - 1);
      const uint32_t off = uint32_t(j) * kRowBytes + (((lane & 15) ^ swz(jl)) << 4);
#pragma unroll
      for (int pl = 0; pl < kPlanes; ++pl)
        copy_g2l_16(k_rows + pl * k_plane * 2, off, lds0 + stage * kScoreStageBytes + (pl * kScoreJ + kRoundRows * rd) * kRowBytes);
    }
  };
  issue_tile(0, 0);

  // Q planes of row i_first + n: B operands, lane (n, hi) holds dims 16ks + 8hi .. +7.  The means arrive
  // as fp32 and are split here into the three bf16 planes (v1 = bf16(v), v2 = bf16(v - v1),
  // v3 = bf16(v - v1 - v2); the differences are exact), as the pooling kernel does for the keys.
  bf16x8 qf[kPlanes][8];
  {
    const int i = min(i_first + n, nb - 1);
    const float* src = reinterpret_cast<const float*>(q_planes) +
                       (int64_t(h) * total_blocks + meta.blk_begin[s] + i) * kHeadDim + 8 * hi;
    f32x4 raw[8][2];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      raw[ks][0] = *reinterpret_cast<const f32x4*>(src + 16 * ks);
      raw[ks][1] = *reinterpret_cast<const f32x4*>(src + 16 * ks + 4);
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        float v = raw[ks][c >> 2][c & 3];
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl) {
          const __bf16 b = (__bf16)v;
          qf[pl][ks][c] = b;
          v -= float(b);
        }
      }
  }
  typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
  const uint32_t k_rd0 = lds_offset_of(&k_lds[0][0]) + uint32_t(n * kRowBytes + ((hi ^ swz(n)) << 4));
  auto read_k = [&](int stage, int pl, int ks) __attribute__((always_inline)) {
    return *reinterpret_cast<lds_bf16x8*>((k_rd0 ^ uint32_t(ks << 5)) + uint32_t(stage * kScoreStageBytes + pl * kScoreJ * kRowBytes));
  };
  float* out = scores + meta.score_off[s] + int64_t(h) * nb * nb;

  // Lane (n, hi) holds row i = i_first + n of a finished tile, columns j0 + 8(r/4) + 4hi + (r%4):
  // four runs of four.
  auto store_tile = [&](const f32x16& v16, int j0) __attribute__((always_inline)) {
    const int i = i_first + n;
    if (i >= nb) return;
    float* row = out + int64_t(i) * nb + j0 + 4 * hi;
    const bool aligned = (reinterpret_cast<uintptr_t>(row) & 15) == 0;   // odd block counts shift rows
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      const int j = j0 + 8 * rq + 4 * hi;
      const f32x4 v = {v16[4 * rq], v16[4 * rq + 1], v16[4 * rq + 2], v16[4 * rq + 3]};
      if (j + 3 <= i && aligned) {
        *reinterpret_cast<f32x4*>(row + 8 * rq) = v;
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (j + c <= i) row[8 * rq + c] = v[c];
      }
    }
  };

  // A finished tile is written out one iteration later, behind the barrier: the wait at
  // the top of an iteration covers every memory operation of the wave (how many stores a lane
  // issued depends on its row, so there is no count to wait for), and stores issued just
  // before it would make each iteration pay their full latency.
  f32x16 pend;
  int pend_j0 = -1;
  for (int jt = 0; jt < n_jt; ++jt) {
    const int stage = jt & 1;
    wait_vmem_all();                                // own copies of tile jt have landed
    __syncthreads();                                // everyone's have; the other stage is free
    if (jt + 1 < n_jt) issue_tile(jt + 1, stage ^ 1);
    if (pend_j0 >= 0) {
      store_tile(pend, pend_j0);
      pend_j0 = -1;
    }
    const int j0 = tj + kScoreJ * jt;
    if (j0 > i_first + 31) continue;                // tile entirely above this wave's rows (uniform per wave)
    f32x16 acc_a, acc_b;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_a[r] = acc_b[r] = 0.0f;
    bf16x8 kf[2][kPlanes];
#pragma unroll
    for (int pl = 0; pl < kPlanes; ++pl) kf[0][pl] = read_k(stage, pl, 0);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const int cur = ks & 1;
      if (ks + 1 < 8) {
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl) kf[cur ^ 1][pl] = read_k(stage, pl, ks + 1);
      }
      acc_a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[cur][0], qf[0][ks], acc_a, 0, 0, 0);
      acc_b = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[cur][1], qf[0][ks], acc_b, 0, 0, 0);
      acc_a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[cur][0], qf[1][ks], acc_a, 0, 0, 0);
      acc_b = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[cur][1], qf[1][ks], acc_b, 0, 0, 0);
      acc_a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[cur][2], qf[0][ks], acc_a, 0, 0, 0);
      acc_b = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[cur][0], qf[2][ks], acc_b, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) pend[r] = (acc_a[r] + acc_b[r]) * scale;
    pend_j0 = j0;
  }
  if (pend_j0 >= 0) store_tile(pend, pend_j0);
}

// Both steps in one launch, for few rows of short sequences: a workgroup pools the one query block of its row (sequence, head,
// query block) and, again, all key blocks in front of it, and multiplies them.
//
// Two launches of some 5 us each, of which most is starting, waiting for the first loads and ending, become one.  What that
// costs is key blocks read and added up by every row behind them: some 0.2 us per block of 128 tokens, from the die's L2 (a die
// takes a run of rows; those of a KV head are on one die or, where a run ends inside them, on two and more), see the rule in
// launch_pool_scores().
// A wave pools a block at a time, each of its rows of 16 lanes every fourth token, a lane 8 dims: sums, means, planes and
// products are those of the two kernels above, bit for bit.
// What a wave does per block is mostly VALU work, so full blocks have a loop without a test per token, at addresses from scalar
// registers, and the parts trade dims before their sums meet (each part working out all 8 dims' planes, and tests for all
// tokens, 777 tokens took 26.6 us for 25.8 and 8/2 x 1000 at 64-token blocks 21.3 for 19.3).  All 32 columns of the
// product are the one query block; its 24 dependent MFMAs, on a wave for each accumulator, take 0.4 us.
// Whole path, passes back to back on one card: 32/8 heads x 777 tokens 29.4 -> 25.4 us (24.2 with the arguments
// loaded together and a lane per sequence, 2048 x 8/8 29.9 -> 28.9), x 300 tokens 23.9 -> 19.9, 4/2 x 60
// 23.7 -> 19.8, 28/4 x (513, 129) 26.5 -> 22.0, eight sequences of 250 x 32/8 31.3 -> 26.7.  Workgroups of 16 waves, of which
// one fits a compute unit, are the faster ones only where eight waves take two turns and more at 64-token blocks (16/4 heads
// x 1000: 25.9 for 26.3 us, 8/8 x 2048 29.1 for 29.9).
// 32 loads in flight per lane change nothing.
constexpr int kRowTokens = 2048;                      // of the longest sequence
static_assert(kRowTokens / 64 <= kScoreJ, "one tile of key blocks");

template <int BQ, int kThreads>
__global__ __launch_bounds__(kThreads) void row_score_kernel(SeqMeta meta, Strides st, const uint16_t* __restrict__ q,
                                                             const uint16_t* __restrict__ k, float* __restrict__ scores,
                                                             int rows, float scale) {
  constexpr int kWaves = kThreads / 64;
  __shared__ __attribute__((aligned(1024))) char k_lds[kScoreStageBytes];
  __shared__ __attribute__((aligned(16))) char q_lds[kPlanes][kRowBytes];
  __shared__ float s_sum[2][kScoreJ];
  // what a single sequence needs of the arguments is loaded together, before the first use
  asm volatile("" ::"s"(rows), "s"(meta.n_seq), "s"(meta.blk_begin[1]), "s"(meta.n_kv_heads),
               "s"(meta.kv_map), "s"(q), "s"(k), "s"(scores), "s"(st.q_t), "s"(st.q_h), "s"(st.kv_t), "s"(st.kv_h));
  const int per_die = (rows + kXcds - 1) / kXcds;      // workgroup b is on die b % 8: a run of rows per die
  const int row = int(blockIdx.x) % kXcds * per_die + int(blockIdx.x) / kXcds;
  if (row >= rows) return;
  int s, h, i, nb;
  int64_t score_off;
  decode_row(meta, row, s, h, i, nb, score_off);
  const int g = meta.kv_map ? kv_head_of(meta, h) : small_quotient(h, small_quotient(meta.n_q_heads, meta.n_kv_heads));
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = lane >> 4, chunk = lane & 15;        // tokens part, part + 4, ..; dims 8 chunk ..
  const int seq_begin = meta.tok_begin[s], seq_end = meta.tok_begin[s + 1];

  for (int b = wave; b < i + 2; b += kWaves) {        // the query block, then key blocks 0 .. i
    const bool is_q = b == 0;
    const int j = is_q ? i : b - 1;
    const int t0 = seq_begin + j * BQ, count = min(seq_end - t0, BQ);
    const int64_t stride = is_q ? st.q_t : st.kv_t;
    const char* src = reinterpret_cast<const char*>((is_q ? q + h * st.q_h : k + g * st.kv_h) + t0 * stride);
    const uint32_t step = uint32_t(stride) * 2;          // (strides are below 2^24: 127 tokens fit 32 bits)
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    constexpr int U = 16;                                // loads in flight per lane
    if (count == BQ) {
      const uint32_t off = uint32_t(part) * step + 16 * chunk;
#pragma unroll
      for (int first = 0; first < BQ / 4; first += U) {
        u32x4 w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = *reinterpret_cast<const u32x4*>(src + int64_t(4 * (first + u)) * step + off);
#pragma unroll
        for (int u = 0; u < U; ++u) add_bf16x8(acc, w[u]);
      }
    } else {
      for (int first = 0; first < BQ / 4; first += U) {
        u32x4 w[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          w[u] = *reinterpret_cast<const u32x4*>(src + uint32_t(min(part + 4 * (first + u), count - 1)) * step + 16 * chunk);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool there = part + 4 * (first + u) < count;     // (zero changes no sum: none is -0)
          add_bf16x8(acc, u32x4{there ? w[u][0] : 0u, there ? w[u][1] : 0u, there ? w[u][2] : 0u, there ? w[u][3] : 0u});
        }
      }
    }
    // Parts trade dims until each has two of the eight, 2 part and 2 part + 1, from all four; their sum, in order, is the
    // pool's.  The mean goes to LDS as three planes.
    float of_part[2][4];
    {
      uint32_t a[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) a[c] = __float_as_uint(acc[c]);
#pragma unroll
      for (int c = 0; c < 4; ++c) swap_halves(a[c], a[c + 4]);   // parts 0, 1 now hold dims 0 .. 3, of parts p and p + 2
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        swap_rows(a[c], a[c + 2]);                               // even parts: dims 0, 1 of these, of parts 0 and 1 ..
        swap_rows(a[c + 4], a[c + 6]);                           // .. and of 2 and 3
        of_part[c][0] = __uint_as_float(a[c]);
        of_part[c][1] = __uint_as_float(a[c + 2]);
        of_part[c][2] = __uint_as_float(a[c + 4]);
        of_part[c][3] = __uint_as_float(a[c + 6]);
      }
    }
    float mean[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
      mean[c] = (((of_part[c][0] + of_part[c][1]) + of_part[c][2]) + of_part[c][3]) / float(count);
#pragma unroll
    for (int pl = 0; pl < kPlanes; ++pl) {
      char* at = is_q ? q_lds[pl] + 16 * chunk : k_lds + (pl * kScoreJ + j) * kRowBytes + ((chunk ^ swz(j)) << 4);
      const __bf16 b0 = (__bf16)mean[0], b1 = (__bf16)mean[1];
      *reinterpret_cast<uint32_t*>(at + 4 * part) =
          uint32_t(__builtin_bit_cast(uint16_t, b0)) | uint32_t(__builtin_bit_cast(uint16_t, b1)) << 16;
      mean[0] -= float(b0);
      mean[1] -= float(b1);
    }
  }
  __syncthreads();
  if (wave < 2) {                                        // the two accumulators of score_kernel, a wave each
    const int n = lane & 31, hi = lane >> 5;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    auto q_at = [&](int pl, int ks) { return *reinterpret_cast<const bf16x8*>(q_lds[pl] + 32 * ks + 16 * hi); };
    auto k_at = [&](int pl, int ks) {
      return *reinterpret_cast<const bf16x8*>(k_lds + (pl * kScoreJ + n) * kRowBytes + ((2 * ks + hi ^ swz(n)) << 4));
    };
    // wave 0: q1 k1 + q2 k1 + q1 k3, wave 1: q1 k2 + q2 k2 + q3 k1
    bf16x8 kf[8][2], qf[8][3];
    const int k_first = wave, k_last = wave == 0 ? 2 : 0;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      kf[ks][0] = k_at(k_first, ks);
      kf[ks][1] = k_at(k_last, ks);
      qf[ks][0] = q_at(0, ks);
      qf[ks][1] = q_at(1, ks);
      qf[ks][2] = q_at(wave == 0 ? 0 : 2, ks);
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks][0], qf[ks][0], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks][0], qf[ks][1], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks][1], qf[ks][2], acc, 0, 0, 0);
    }
    if (n == 0)
#pragma unroll
      for (int r = 0; r < 16; ++r) s_sum[wave][8 * (r >> 2) + 4 * hi + (r & 3)] = acc[r];
  }
  __syncthreads();
  if (tid <= i) scores[score_off + (int64_t(h) * nb + i) * nb + tid] = (s_sum[0][tid] + s_sum[1][tid]) * scale;
}

}  // namespace

int32_t launch_pool_scores(const Geometry& g, const void* q, const void* k, float* scores,
                           uint16_t* q_planes, uint16_t* k_planes, int n_compute_units, hipStream_t stream) {
  const SeqMeta& m = g.meta;
  const int64_t longest = int64_t(g.max_nb) * m.block;
  // One launch for both steps up to sequences of 2048 tokens, and as many rows as one of such a sequence per compute unit
  // reads as much as: reading is what it costs.  Whole path in two launches and in one: 8/8 heads x 2048, 64-token blocks 31.0
  // and 29.1 us, 16/4 x 2047 43.7 and 41.2, 40/8 x 1024 39.6 and 37.2, 16 sequences of 250 x 32/8 57.3 and 53.5, 40 of 100 x
  // 28/4 56.1 and 52.3.  Beyond: 4/2 x 4096 61.9 and 64.1, 32/8 x 2000 (two rows a compute unit) 56.0 and 58.2.  Over 100 shapes
  // within the rule, 46 at three quarters of its limit and more, one launch takes 0.83 to 1.01 of the time of two, eagerly and in
  // a graph.
  // That is the path with selection and attention behind the scores.  The scores alone, taken again and again from the same
  // tensors, which the caches then hold, are slower in one launch near the limit (16 sequences of 239 x 28/4 at 64-token
  // blocks, seven rows a compute unit, 15.2 for 10.9 us; the whole path 62.7 for 64.4).
  if (longest <= kRowTokens && g.rows * longest <= int64_t(kRowTokens) * n_compute_units) {
    const int per_die = int((g.rows + kXcds - 1) / kXcds);
    const bool wide = m.block == 64 && longest > 512 && g.rows <= n_compute_units;
    const auto kernel = m.block == 128 ? row_score_kernel<128, 512> : wide ? row_score_kernel<64, 1024> : row_score_kernel<64, 512>;
    hipLaunchKernelGGL(kernel, dim3(per_die * kXcds), dim3(wide ? 1024 : 512), 0, stream, m, g.st, static_cast<const uint16_t*>(q),
                       static_cast<const uint16_t*>(k), scores, int(g.rows), g.scale);
    return hipGetLastError() == hipSuccess ? SHPLB_OK : SHPLB_E_HIP;
  }
  const int q_chunks = (m.n_q_heads * kHeadDim + kPoolElems - 1) / kPoolElems;
  const int k_chunks = (m.n_kv_heads * kHeadDim + kPoolElems - 1) / kPoolElems;
  const int64_t n_wg = g.total_blocks * (q_chunks + k_chunks);
  if (n_wg > 0x7fffffff) return SHPLB_E_UNSUPPORTED;
  hipLaunchKernelGGL(pool_kernel, dim3(uint32_t(n_wg)), dim3(kPoolThreads), 0, stream, m, g.st,
                     static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k), q_planes, k_planes,
                     q_chunks, k_chunks, int(g.total_blocks));
  if (hipGetLastError() != hipSuccess) return SHPLB_E_HIP;
  // Key-block rows per workgroup: the shortest chunk with which the whole launch is resident at
  // once (three workgroups per compute unit); more, shorter workgroups would run in rounds,
  // fewer, longer ones would leave compute units idle.
  const int64_t resident = int64_t(n_compute_units) * 3, n_sh = int64_t(m.n_seq) * m.n_q_heads;
  // Workgroups of one wave, 32 rows and one K tile, while no more than three per compute unit come of it: with four waves such
  // a launch has few workgroups, each of which goes through its tiles in turn.  Scoring call, four waves against one: 32/8 heads x
  // 6000 18.3 -> 16.6 us, x 8231 23.1 -> 21.2, x 16384 37.1 -> 35.9, 8/2 x 20000 18.1 -> 15.5, 28/4 x 8000 with 64-token blocks 20.7 -> 18.7;
  // 32/8 x 24000 (672 workgroups) 49.3 and 49.3, x 32768 (1152) 63.6 and 63.9, with 64-token blocks (4352) 72.1 and 75.4.
  const int tiles32 = (g.max_nb + 31) / 32;
  const bool small = tiles32 == 1 || int64_t(tiles32) * (tiles32 + 1) / 2 * n_sh <= resident;
  const int tile = small ? 32 : 128, tiles = (g.max_nb + tile - 1) / tile;
  int log_chunk = small ? 5 : 6, n_pairs = 0;
  for (;; ++log_chunk) {
    n_pairs = 0;
    for (int tr = 0; tr < tiles; ++tr) n_pairs += score_chunks_of_row(tr, log_chunk, tile);
    if (small || n_pairs * n_sh <= resident || 1 << log_chunk >= tiles * tile) break;
  }
  const dim3 grid(n_pairs, 1, m.n_seq * m.n_q_heads);
  if (small)
    hipLaunchKernelGGL((score_kernel<1>), grid, dim3(64), 0, stream, m, q_planes, k_planes, scores, int(g.total_blocks),
                       log_chunk, g.scale);
  else
    hipLaunchKernelGGL((score_kernel<4>), grid, dim3(256), 0, stream, m, q_planes, k_planes, scores, int(g.total_blocks),
                       log_chunk, g.scale);
  if (hipGetLastError() != hipSuccess) return SHPLB_E_HIP;
  return SHPLB_OK;
}

}  // namespace shplb
