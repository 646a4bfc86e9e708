// Software-pipelined block-sparse causal attention over per-row selected key blocks (gfx950).
//
// Work item = one (sequence, head, query block) row of the selection, or a piece of one.
// Persistent workgroups draw items from cost-descending queues through atomic tickets; a launch of no
// more rows than workgroups has no queues (wq.items is null): every row gets a workgroup.
//
// Tiling (wave64, v_mfma_f32_16x16x32_bf16), for blocks of BQ = 128 or 64 tokens:
//   * a wave owns 32 query rows, in two groups of 16, and keeps Q as MFMA B-operands in registers; a query
//     block is BQ/32 waves.  Block 128: 4 waves, two workgroups per compute unit; block 64: 2 waves, four
//     workgroups per compute unit.  Either way every SIMD holds two waves of different
//     workgroups, each with 256 registers, and one wave's softmax VALU work overlaps the other's
//     MFMAs;
//   * keys are streamed in tiles of KT = BQ/2 keys, two tiles per key block.  K and V rows go
//     from global memory straight into a double-buffered LDS stage (global_load_lds_dwordx4, no
//     staging registers, no LDS store instructions).  Rows are 256 bytes, unpadded; the 16-byte
//     chunk c of row r sits at chunk slot c ^ swz(r), which keeps both the K operand reads and
//     the V transpose reads free of bank conflicts;
//   * the first contraction is S^T = K Q^T (A = K from LDS by 16-byte reads, each operand for both query groups),
//     so a lane holds one query column of each group: the softmax max/sum are in-lane plus two exchanges over the
//     four lanes of a query, and the probabilities feed the second contraction O^T += V^T P^T straight from
//     registers (the key order inside a 32-key MFMA step is permuted identically on both operands, which a sum over
//     keys does not see); V^T operands come from the LDS transpose read (ds_read_b64_tr_b16);
//   * the order of work inside a wave.  A step handles tile t's softmax and second contraction
//     and tile t+1's first contraction:
//
//       step t:  barrier                      K(t+1), V(t) resident; stages of K(t), V(t-1) free
//                the first operands of K(t+1) are fetched, copies K(t+2), V(t+1) start
//                exp / bf16 pack / row sum of the probabilities of tile t (one run of VALU work);
//                if a row sum shows that the reference maximum was too low (rare): true
//                maximum of the tile, rescale O and l, probabilities again
//                the MFMAs of S(t+1), back to back; mask S(t+1) if it is the diagonal block
//                the MFMAs of O += V(t)^T P(t)^T, back to back
//
//     so a wave alternates between a block of MFMAs, at wave priority 1, and a run of VALU work, at priority 0, that
//     depends on none of the MFMAs in flight, and the two waves of a SIMD (of different workgroups,
//     unsynchronised) mostly find the other unit free.
//
// Why 16x16x32: long launches run at the card's power limit, and of MFMAs alone on random operands that limit lets
// through 1.87 PFLOP/s in this shape (the loop of probe_kernels.hip), 1.67 in 32x32x16 (twice the operand reads but half the
// accumulator traffic per product).  By itself the change moved the bound from power (1.64 GHz, matrix pipe 70% busy) to the schedule
// (2.0 GHz, 58%) and gained nothing; then
//   * chunk slots free of conflicts for the new operand reads (see swz()): 128K +2%, 32K +1.3%;
//   * the softmax in front of both contractions, not between them: the latency of the first K operands and the
//     issue of the copies (64 bytes a cycle) pass behind it, and 32 fewer registers live in it: +4%;
//   * the two groups' probabilities in turn, two partial sums each (the dot products form chains): +3%;
//   * priority by phase instead of by turns of 41 us between the workgroups of a compute unit: +0.7%.
// Together: 128K layer 30.7 -> 28.0 ms (1.32 PFLOP/s), 32K 1870 -> 1725 us, with 64-token blocks 2180 -> 1995 us, a
// 64K share of 8 heads 1553 -> 1434 us, an 8K prompt 182 -> 171 us, 48 sequences 148 -> 144 us (whole path).  Now 1.79 GHz
// and 72% at 128K.  Spreading the VALU work between the MFMAs of the same wave, in whatever part, costs 4 to 25%; copies
// issued later in the step or between the exponentials 2 to 5%.
//
// Between items.  An item used to cost about 21 000 cycles beside its tiles (an atomic ticket that waited
// for the output stores in front of it, the record, the first selected blocks, the first tile copies and
// the Q rows, one dependent memory round trip after the other).  Now the ticket is asked for three steps before
// the end (in items of two tiles: at their start), its record is fetched in the last step but one, and the last
// step issues the next item's copies and Q loads as soon as its barrier says that the stages are free; the copies
// are waited for after the output stores, by count, without the stores.  (4.9 tiles an item, 48 sequences x 28
// heads: the launch 135 -> 121 us; 62 tiles, 32K: 1.84 -> 1.80 ms; the 128K layer, 270 tiles, 1.4%.)  With the copies
// started one step later, between the last step and the output, these were 125 us, 1.81 ms and 0.7%.
//
// HALVES: items may be halves of a row's queries (16 a wave), the first 2 H of a queue being those of its H longest rows; see
// queue_place() and in_halves().  A query's sums do not depend on it, as with QS = 2.  (Operands are fetched 6 ahead there: with
// 8, 22 and more registers are spilled in the tile loop, 16%.)
//
// The two score buffers swap roles from step to step (the tile count is even, steps are
// issued in pairs).  LDS operands are fetched kLook ahead of their use.  Fully
// masked sub-tiles are computed like any other (their probabilities are exact zeros).
// With 64-token blocks a tile feeds half as many MFMAs per copy, barrier and item as with 128.
//
// KS = 2: two groups of waves share a 64-token row, each with every other selected block, and combine their
// results in LDS (launches of few 64-token rows, see plan_attention()).
//
// SCORES_FIRST: the MFMAs of S(t+1) in front of the softmax, all at one priority, for 64-token rows shared by two groups and
// dealt without queues: with up to one row per compute unit a SIMD has one wave, and its last MFMAs then run behind its own
// exponentials (2/1 heads x 8000 with a dense one 112.1 -> 108.6 us, 256 dense rows of up to 64 blocks 66.1 -> 64.0, with two
// rows 512 dense ones 73.0 -> 72.1, 512 at 5 to 50% 39.2 -> 38.6).  Pieces from queues, where 512 dense rows take 88.6 us with
// the softmax in front, take 99.9 that way (2/1 x 8000 72.4 -> 71.8, 256 dense rows 65.7 -> 67.2).
//
// COPIERS (KS = 2, up to one 64-token row per compute unit): a wave for each group does nothing but copy its tiles, into four stages, three
// steps ahead.  With one wave per SIMD a step was a chain of its copies (64 bytes a cycle: some 450 of 1600 cycles), products and
// exponentials, and tiles that come from further away than the die's L2 were waited for.  The two waves meet the others at every
// barrier.  Whole path: 2048 x 8/8 heads, 2 to 16 blocks a row, 29.0 -> 26.7 us, 2000 x 8/2 with a dense head 39.3 -> 34.5, 500 x 32/8
// 18.9 -> 17.9, 16000 x 1/1 dense 207 -> 154, two blocks a row 18.0 and 18.0.  With four such waves and two stages 27.1, 35.3,
// 18.1, 209 and 18.8.  Two rows a compute unit have no LDS for it.  For 128-token rows (QS = 2 below), where reading the operands bounds
// a step, it does not pay: 2 to 20% slower.
//
// QS = 2: two groups of four waves share a 128-token row's queries, 16 a wave (launches of no more rows than compute units).
// Both work on the same tiles, group 1 half a step behind, kept there by a second barrier in the middle of a step: one
// group's MFMAs run against the other's softmax.  Group 1 issues the copies, at the start of its step t like above: that is
// the middle of group 0's, when both are done with K(t) and V(t-1).  What it waits for at the start of its next step
// is K(t+2) and V(t+1), which group 0 first reads behind that same barrier, in the second half of its step t+1.  Nothing a
// query's sums are made of or their order depends on QS.
#include <type_traits>

#include "attn_common.h"

namespace shplb {
namespace {

// Everything the kernel is given.  It reads fields through the kernel-argument segment where it needs
// them (see reload()): kept in scalar registers across the tile loop they do not fit.
struct AttnArgs {
  const uint16_t *q, *k, *v;
  const int64_t* sel_ptr;
  const int32_t* sel_idx;
  uint16_t* out;
  float* lse;
  shplb_wg_stats* stats;
  int32_t n_stats;
  int32_t rows, rows_per_die, compute_units;   // how rows without queues are dealt, see row_place()
  int32_t group;                               // query heads per KV head; 0: meta.kv_of names them
  float scale_log2;
  int64_t total_tokens;
  Strides st;
  WorkQueues wq;
  SplitBuffers sb;
  SeqMeta meta;
};
typedef const __attribute__((address_space(4))) AttnArgs* ArgsPtr;
typedef const __attribute__((address_space(4))) int32_t* ConstInts;   // read by scalar loads
typedef const __attribute__((address_space(4))) int64_t* ConstLongs;

// The same pointer, but the compiler may not carry values loaded through it from before this point.
__device__ __forceinline__ ArgsPtr reload(ArgsPtr a) {
  asm volatile("" : "+s"(a));
  return a;
}

// A pointer that is the same in all lanes, said explicitly: in scalar registers.
__device__ __forceinline__ const char* uniform(const char* p) {
  const uint64_t x = reinterpret_cast<uint64_t>(p);
  return reinterpret_cast<const char*>(uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(x)))) |
                                       uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(x >> 32)))) << 32);
}

// What a wave keeps of the item it works on (uniform values).
struct Item {
  int pos;                            // its place in the queues
  int n_sel, slot, head, q_block, n_blocks, kv_head, seq_begin, seq_end, first_block, second_block;
  int64_t sel_begin;
  int half;                           // 0: the row; 1, 2: the first, second half of its queries
};

// The row of workgroup b in a launch that gives every row a workgroup of its own.  False: no row.
// The dispatcher puts workgroup b on die b % 8 and, one lap of all compute units after the other, beside workgroup
// b - (compute units).
// * No more rows than compute units: die x takes a run of consecutive rows (rows_per_die), i.e. few K/V streams.
// * More: rows that lie next to each other (of one head, all long or all short) go to different compute units and
//   dies, and every other lap runs backwards, so that the long end of a head mostly meets the short end of another.
//   In runs, the long rows of a dense head shared few compute units.  The attention step for 4/2 heads x 16K with
//   one dense head takes 257 us (in runs 335, with the ordering launch 266), for 2/1 x 32K 507 (782, 517), 8/2 x 8K
//   131 (152, 140).  Of some 200 shapes of 256 to 1024 rows one is slower than with the ordering launch: dense heads
//   among five of 200 64-token blocks, whose long ends meet (two 283 against 261, three 286 against 270).  Runs
//   are the faster ones for up to one row per compute unit (2K x 8 heads, 64-token blocks: 25.2 against 26.5) and
//   for equally short rows (32/8 heads x 2K at budgets of 2 to 4 blocks 21 against 23).
// What a single sequence needs of the arguments is loaded together, before the first use: each load that waits for
// another one costs some 500 cycles here, at the start of the launch.
__device__ __forceinline__ bool row_place(ArgsPtr a, int b, Item& it) {
  const int n_seq = a->meta.n_seq, hq = a->meta.n_q_heads, rows = a->rows, per_die = a->rows_per_die, cus = a->compute_units;
  const int group = a->group, nb0 = a->meta.blk_begin[1], t0 = a->meta.tok_begin[0], t1 = a->meta.tok_begin[1];
  asm volatile("" ::"s"(n_seq), "s"(hq), "s"(rows), "s"(per_die), "s"(cus), "s"(group), "s"(nb0), "s"(t0), "s"(t1), "s"(a->q),
               "s"(a->st.q_t));
  int row = (b % kXcds) * per_die + b / kXcds;
  bool any = b / kXcds < per_die && row < rows;
  if (per_die == 0) {
    int begin = 0, odd = 0;                          // first row of the lap
    for (; begin + cus <= b; begin += cus) odd ^= 1;
    const int place = b - begin, n = min(cus, rows - begin);
    row = begin + (odd ? n - 1 - place : place);
    any = place < n;
  }
  if (!any) return false;
  auto scalar = [](int x) { return int(__builtin_amdgcn_readfirstlane(x)); };
  // x / y of small non-negative numbers (there are no more rows than workgroups here)
  auto quotient = [&](int x, int y) {
    const int q = scalar(int(float(x) * __builtin_amdgcn_rcpf(float(y)))), r = x - q * y;
    return q + (r >= y ? 1 : 0) - (r < 0 ? 1 : 0);
  };
  int s = 0, local = row;
  it.n_blocks = nb0;
  it.seq_begin = t0;
  it.seq_end = t1;
  if (n_seq > 1) {
    // how many sequences end at or before the row (one lane per sequence)
    const int lane = threadIdx.x & 63;
    s = __builtin_popcountll(__ballot(lane < n_seq && row >= a->meta.blk_begin[min(lane, n_seq - 1) + 1] * hq));
    const int b0 = scalar(a->meta.blk_begin[s]);
    local = row - b0 * hq;
    it.n_blocks = scalar(a->meta.blk_begin[s + 1]) - b0;
    it.seq_begin = scalar(a->meta.tok_begin[s]);
    it.seq_end = scalar(a->meta.tok_begin[s + 1]);
  }
  it.pos = row;
  it.head = quotient(local, it.n_blocks);
  it.q_block = local - it.head * it.n_blocks;
  it.kv_head = group > 0 ? quotient(it.head, group) : scalar(int(a->meta.kv_of[it.head >> 2] >> (8 * (it.head & 3)) & 0xff));
  it.slot = -1;
  it.half = 0;
  return true;
}

// The wave that copies the tiles of group `grp` of a row without a record (see COPIERS).  It meets the others at the barriers of
// the kernel: one in front of S(0), one at the start of each step, three around the combination of the groups.
template <int BQ, int KT, int kStages>
__device__ __forceinline__ void copy_row(ArgsPtr args, const Item& it, int grp, int lane, uint32_t k_lds, uint32_t v_lds) {
  static_assert(kStages == 4 && KT == 32, "counts of copies below");
  constexpr int kTileBytes = KT * kRowBytes, kRounds = KT / 4;      // four rows a copy
  const int64_t row_bytes = args->st.kv_t * 2;
  const char* const k_head = reinterpret_cast<const char*>(args->k + int64_t(it.kv_head) * args->st.kv_h);
  const char* const v_head = reinterpret_cast<const char*>(args->v + int64_t(it.kv_head) * args->st.kv_h);
  const int r4 = lane >> 4;
  uint32_t off[4];                                   // of a lane in rounds 0 .. 3 mod 4, without the round's first row
#pragma unroll
  for (int x = 0; x < 4; ++x) off[x] = uint32_t(r4) * uint32_t(row_bytes) + (((lane & 15) ^ swz(4 * x + r4)) << 4);
  auto copy_tile = [&](const char* head, int j, int half, uint32_t dst) {
    const int key_base = min(it.seq_begin + min(max(j, 0), it.n_blocks - 1) * BQ + KT * half, it.seq_end - 1);
    const int last = it.seq_end - 1 - key_base;
    const char* tile = uniform(head + int64_t(key_base) * row_bytes);
    dst = __builtin_amdgcn_readfirstlane(dst);
    if (last >= KT - 1) {
#pragma unroll
      for (int rd = 0; rd < kRounds; ++rd) copy_g2l_16(tile + int64_t(4 * rd) * row_bytes, off[rd & 3], dst + rd * 4 * kRowBytes);
    } else {                                         // rows past the end re-read the last valid key (masked)
#pragma unroll
      for (int rd = 0; rd < kRounds; ++rd) {
        const int r = 4 * rd + r4;
        copy_g2l_16(tile, uint32_t(min(r, last)) * uint32_t(row_bytes) + (((lane & 15) ^ swz(r)) << 4), dst + rd * 4 * kRowBytes);
      }
    }
  };
  auto k_tile = [&](int j, int t) { copy_tile(k_head, j, t & 1, k_lds + (t & 3) * kTileBytes); };
  auto v_tile = [&](int j, int t) { copy_tile(v_head, j, t & 1, v_lds + (t & 3) * kTileBytes); };
  auto first_block = [&](int j) {
    k_tile(j, 0);
    v_tile(j, 0);
    k_tile(j, 1);
    v_tile(j, 1);
  };
  // (block 0, the sink, is nearly always a row's first: its copies start before the selection is known)
  const ConstLongs ptr = (ConstLongs)uintptr_t(args->sel_ptr + it.pos);
  const int64_t begin = ptr[0], end = ptr[1];
  if (grp == 0) first_block(0);
  const int n_sel = int(end - begin);
  if (n_sel <= 0) {
    wait_vmem_all();
    return;
  }
  const ConstInts sel = (ConstInts)uintptr_t(args->sel_idx + begin);
  auto block_of = [&](int b) { return sel[min(2 * b + grp, n_sel - 1)]; };
  const int n_tiles = 2 * ((n_sel + 1) / 2);         // of either group
  const int j0 = block_of(0);
  int jv = block_of(1), jk = block_of(2);            // the blocks of V(t+3) and K(t+4)
  if (grp == 1 || j0 != 0) {
    wait_vmem_all();                                 // (of the copies that went to the same stages)
    first_block(j0);
  }
  if (n_tiles > 2) {
    k_tile(jv, 2);
    v_tile(jv, 2);
    k_tile(jv, 3);
  }
  // tile t + 1's K and tile t's V are wanted at the start of step t, K(0) before the first: what was issued after them may be under way
  if (n_tiles > 2) wait_vmem_but(std::integral_constant<int, 6 * kRounds>{});
  else wait_vmem_but(std::integral_constant<int, 3 * kRounds>{});
  __syncthreads();
  for (int t = 0; t < n_tiles; ++t) {
    if (t + 3 < n_tiles) wait_vmem_but(std::integral_constant<int, 4 * kRounds>{});
    else wait_vmem_all();
    __syncthreads();
    // the stages of K(t) and V(t-1) are free
    if (t + 3 < n_tiles) v_tile(jv, t + 3);
    if (t + 4 < n_tiles) k_tile(jk, t + 4);
    jv = jk;
    jk = block_of((t + 5) / 2);
  }
  __syncthreads();
  __syncthreads();
  __syncthreads();
}

// BQ: tokens per block.  GROUPS: groups of BQ/32 waves that share a row, see KS, QS, SCORES_FIRST and COPIERS in the header.
template <int BQ, int GROUPS, bool SCORES_FIRST, bool COPIERS, bool HALVES>
__global__ __launch_bounds__(64 * (GROUPS * BQ / 32 + (COPIERS ? GROUPS : 0))) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_pipe_kernel(AttnArgs) {
  static_assert(GROUPS == 1 || GROUPS == 2, "an item's record names its first two blocks");
  constexpr int KS = BQ == 64 ? GROUPS : 1, QS = BQ == 128 ? GROUPS : 1;   // groups that share a row, by keys and by queries
  constexpr int kWaves = BQ / 32;                    // waves of a group: 32 query rows each, or 16
  static_assert(!COPIERS || (KS == 2 && SCORES_FIRST), "rows without queues, shared by their keys");
  constexpr int kThreads = 64 * (GROUPS * kWaves + (COPIERS ? GROUPS : 0));
  constexpr int kStages = COPIERS ? 4 : 2;           // of K and V tiles each: tile t is in stage t mod kStages
  constexpr int KT = BQ / 2;                         // keys per tile: two tiles per key block
  static_assert(!HALVES || GROUPS == 1, "rows from queues");
  constexpr int QGM = 2 / QS, MT = KT / 16;          // 16-query and 16-key MFMA tiles of a tile's scores
  constexpr int kTileBytes = KT * kRowBytes;
  constexpr int kRoundRows = 4 * kWaves;             // rows one round of copies moves (4 per wave)
  constexpr int kRounds = KT / kRoundRows;
  constexpr int kQK = 4 * MT;                        // K operands of a tile's first contraction, index MT*ks + mt ...
  constexpr int kPV = 8 * (KT / 32);                 // ... V operands of its second, index 8*gq + dt: QG MFMAs each
  // LDS operand fetches run this many operands ahead.  (A row to a workgroup: 12 no change.  Shared by two groups: 1/1 heads
  // x 20000 take 266 us with 4, 281 with 2, 273 with 8, 292 with 16; 2/1 x 8000 with 64-token blocks 109.5 with 4, 111.5 with 8.)
  constexpr int kLook = GROUPS > 1 ? 4 : HALVES ? 6 : 8;
  constexpr float kSumLimit = 4.0f * MT * 256.0f;    // a lane's 4 MT probabilities of a query and tile can only sum to
                                                     // more if one of them exceeds 2^8
  constexpr int kHelp = -2;                          // s_next: the home queue is empty

  // stages of group g: K tiles from 2 kStages g * kTileBytes on, V tiles kStages behind them
  __shared__ __attribute__((aligned(1024))) char lds[KS * 2 * kStages * kTileBytes];
  __shared__ float s_ml[KS > 1 ? KS * 2 * BQ : 1];   // groups' reference exponents and denominators
  __shared__ int32_t s_next, s_flag, s_empty;
  __shared__ int32_t s_home[HALVES ? 3 : 1];         // the home queue's begin, halved rows and size (thread 0's own)
  __shared__ int32_t s_merge[kDeferredMerges];       // items whose row this workgroup still has to combine

  ArgsPtr args = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int team = GROUPS > 1 ? wave_all / kWaves : 0, wave = GROUPS > 1 ? wave_all % kWaves : wave_all;
  const bool computes = !COPIERS || wave_all < GROUPS * kWaves;
  const int grp = COPIERS && !computes ? wave_all - GROUPS * kWaves : KS > 1 ? team : 0, q_grp = QS > 1 ? team : 0;         // group of waves, by keys or by queries
  const int q_wave = 16 * QGM * (q_grp * kWaves + wave);                // the wave's first query
  const int n = lane & 15, hi = lane >> 4;
  const int64_t row_bytes = args->st.kv_t * 2;
  const float scale_log2 = args->scale_log2;

  // ---- per-lane constants
  // copies: lane (r4 = lane>>4, slot = lane&15) of a wave fills, in round rd, LDS row
  // rd*kRoundRows + cp_row, slot `slot`, with the source chunk slot ^ swz(row).  Rounds of 8
  // rows alternate bit 3 of the row, which flips the two low bits of the swizzle: two per-lane
  // source offsets cover all rounds.
  // K operand reads: lane (n, hi) reads row 16mt + n, chunk 4ks + hi.
  // V transpose reads: lane = 16*hi + 4e + a supplies the piece (key 32gq + 16half + 4hi + e, dims 16dt + 4a ..)
  // and receives keys 4hi+0..3 (+16half, +32gq) of dim 16dt + n.
  const int cp_row = 4 * wave + (lane >> 4);
  const uint32_t cp_off0 = uint32_t(cp_row) * uint32_t(row_bytes) + (((lane & 15) ^ swz(cp_row)) << 4);
  const uint32_t cp_off1 = uint32_t(cp_row) * uint32_t(row_bytes) + (((lane & 15) ^ swz(cp_row) ^ 3) << 4);
  const int k_rd0 = n * kRowBytes + ((hi ^ swz(n)) << 4);
  const int tr_row = 4 * hi + ((lane >> 2) & 3), tr_a = lane & 3;
  const int v_rd0 = tr_row * kRowBytes + (((tr_a >> 1) ^ swz(tr_row)) << 4) + 8 * (tr_a & 1);
  const char* const k_lds = lds + grp * 2 * kStages * kTileBytes;
  const char* const v_lds = k_lds + kStages * kTileBytes;
  const uint32_t k_stage0 = __builtin_amdgcn_readfirstlane(lds_offset_of(lds) + grp * 4 * kTileBytes + 4 * wave * kRowBytes);
  const uint32_t v_stage0 = k_stage0 + 2 * kTileBytes;

  uint32_t my_items = 0, my_cost = 0;
  uint64_t t_first = 0, t_last = 0;
  int n_merge = 0;                       // rows whose last piece finished here; combined after the loop
  const int home = my_xcd();
  bool home_open = false;                // the home die's queue may still hold items
  int home_begin = 0;                    // ... which starts at this place
  uint32_t home_size = 0;                // ... and held so many (HALVES: s_home, for want of scalar registers)

  // The record of queue place pos, one word per lane (every 16 lanes): a vector load, so that waiting
  // for it does not wait for LDS operands.
  // (No place: any words.  No branch around the load, which would make the wave wait for it on the spot.)
  auto record_words = [&](int pos) {
    ArgsPtr a = reload(args);
    const uint32_t* at = pos >= 0 ? reinterpret_cast<const uint32_t*>(a->wq.items + (HALVES ? pos & kPlaceMask : pos)) : reinterpret_cast<const uint32_t*>(a->q);
    return at[lane & 15];
  };
  auto read_record = [&](int pos, uint32_t words, Item& it) {
    auto word = [&](int x) { return int(__builtin_amdgcn_readlane(words, x)); };
    it.pos = HALVES ? pos & kPlaceMask : pos;
    it.n_sel = word(1);
    it.sel_begin = int64_t(uint32_t(word(2))) | int64_t(word(3)) << 32;
    it.slot = word(4);
    it.seq_begin = word(8);
    it.seq_end = word(9);
    it.head = word(10);
    it.kv_head = word(11);
    it.q_block = word(12);
    it.n_blocks = word(13);
    it.first_block = word(14);
    it.second_block = word(15);
    it.half = HALVES ? pos >> kHalfShift : 0;
    // records come from the ordering kernel; a malformed one must not index out of bounds
    return it.n_sel > 0 && it.slot < reload(args)->sb.slot_capacity;
  };
  // Place of an item from another die's queue, to all threads (-1: every queue is empty).
  auto help = [&]() {
    if (wave_all == 0) {
      const int at = help_item<HALVES>(reload(args)->wq.queue_begin, reload(args)->wq.tickets, home, &s_empty);
      if (lane == 0) s_next = at;
    }
    __syncthreads();
    const int pos = __builtin_amdgcn_readfirstlane(s_next);
    __syncthreads();
    return pos;
  };

  // ---- first item.  Queue x starts with one item for each workgroup of the grid that the dispatcher puts
  // on die x (the tickets start behind them): no atomic and no waiting for one.
  Item it;
  bool have;
  if (args->wq.items == nullptr) {
    have = row_place(args, blockIdx.x, it);
  } else {
    if (tid < 64) s_empty = 0;                       // (wave 0's own)
    const int x = blockIdx.x % kXcds, begin = args->wq.queue_begin[x];
    const int halved = HALVES ? args->wq.queue_begin[kHalvedRows + x] : 0;
    int pos = queue_place(begin, halved, int(blockIdx.x / kXcds));
    if (int(blockIdx.x / kXcds) >= args->wq.queue_begin[x + 1] - begin + halved) pos = help();
    have = pos >= 0 && read_record(pos, record_words(pos), it);
    while (!have && pos >= 0) {                      // rows without a block (at the end of their queues)
      pos = help();
      have = pos >= 0 && read_record(pos, record_words(pos), it);
    }
    home_open = true;
    if constexpr (HALVES) {
      if (tid == 0) {
        s_home[0] = args->wq.queue_begin[home];
        s_home[1] = args->wq.queue_begin[kHalvedRows + home];
        s_home[2] = args->wq.queue_begin[home + 1] - s_home[0] + s_home[1];
      }
    } else {
      home_begin = __builtin_amdgcn_readfirstlane(args->wq.queue_begin[home]);
      home_size = uint32_t(__builtin_amdgcn_readfirstlane(args->wq.queue_begin[home + 1]) - home_begin);
    }
  }

  if constexpr (COPIERS) {
    if (!computes) {
      if (have) copy_row<BQ, KT, kStages>(args, it, grp, lane, lds_offset_of(k_lds), lds_offset_of(v_lds));
      return;
    }
  }
  const char *k_head = nullptr, *v_head = nullptr;
  bf16x8 qf[QGM][4];
  int64_t next_off = 0;                  // byte offset (from k_head, v_head) of the tile whose K copies were issued last ...
  int next_last = 0;                     // ... and the row in it that holds the sequence's last token (or a larger number)

  // Tile `half` of block j: where its rows start.
  auto locate = [&](int j_raw, int half) {
    const int j = min(max(j_raw, 0), it.n_blocks - 1);
    // a sub-tile that starts past the end of a ragged last block is moved back onto the
    // last token: row offsets must stay non-negative (they are added unsigned)
    const int key_base = min(it.seq_begin + j * BQ + KT * half, it.seq_end - 1);
    next_last = it.seq_end - 1 - key_base;
    next_off = int64_t(key_base) * row_bytes;
  };
  // Copy the K or V rows of the located tile into an LDS stage.
  auto issue = [&](const char* head, uint32_t dst) {
    const char* tile = uniform(head + next_off);
    if (next_last >= KT - 1) {
#pragma unroll
      for (int rd = 0; rd < kRounds; ++rd) {
        const bool odd8 = ((rd * kRoundRows) >> 3) & 1;       // round starts at an odd multiple of 8 rows
        copy_g2l_16(tile + int64_t(rd * kRoundRows) * row_bytes, odd8 ? cp_off1 : cp_off0,
                    dst + rd * kRoundRows * kRowBytes);
      }
    } else {                                     // ragged: rows past the end re-read the last valid key (masked)
#pragma unroll
      for (int rd = 0; rd < kRounds; ++rd) {
        const int r = rd * kRoundRows + cp_row;
        const uint32_t off = uint32_t(min(r, next_last)) * uint32_t(row_bytes) + (((lane & 15) ^ swz(r)) << 4);
        copy_g2l_16(tile, off, dst + rd * kRoundRows * kRowBytes);
      }
    }
  };
  // Everything an item can start before its turn: its first tile copies and its Q fragments (B operand of
  // S^T = K Q^T, lane (n, hi) holds dims 32ks+8hi.. of queries n and 16 + n).  The stages must be free.
  auto load_queries = [&](ArgsPtr a) {
    const uint16_t* src[QGM];
    const int first = HALVES && it.half > 0 ? BQ / 2 * (it.half - 1) + 16 * wave : q_wave, group = HALVES && it.half > 0 ? 0 : 16;
#pragma unroll
    for (int qg = 0; qg < QGM; ++qg) {
      const int tok = min(it.seq_begin + it.q_block * BQ + first + group * qg + n, it.seq_end - 1);
      src[qg] = a->q + int64_t(tok) * a->st.q_t + int64_t(it.head) * a->st.q_h + 8 * hi;
    }
#pragma unroll
    for (int qg = 0; qg < QGM; ++qg)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) qf[qg][ks] = *reinterpret_cast<const bf16x8*>(src[qg] + 32 * ks);
  };
  const std::true_type yes{};
  const std::false_type no{};
  const bool copies = !COPIERS && (QS == 1 || q_grp == 1);   // of query groups the later one copies, for both (see the header)
  auto start_item = [&](auto copies_c, auto queries_c) {
    constexpr bool kCopies = decltype(copies_c)::value, kQueries = decltype(queries_c)::value;
    ArgsPtr a = reload(args);
    k_head = reinterpret_cast<const char*>(a->k + int64_t(it.kv_head) * a->st.kv_h);
    v_head = reinterpret_cast<const char*>(a->v + int64_t(it.kv_head) * a->st.kv_h);
    if (kCopies && copies) {
      locate(it.first_block, 0);
      issue(k_head, k_stage0);
    }
    if (kQueries) load_queries(a);
    if (kCopies && copies) {
      issue(v_head, v_stage0);
      locate(it.first_block, 1);
      issue(k_head, k_stage0 + kTileBytes);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // the group's own first block
  auto own_first = [&]() {
    if (KS > 1 && grp == 1) it.first_block = it.second_block;
  };
  if (have && args->wq.items != nullptr) {
    own_first();
    start_item(yes, yes);
  } else if (have) {
    // A row without a record: which blocks it has selected is two dependent loads away.  Block 0, the sink, is
    // nearly always the first of them: its copies start meanwhile, and are done again if it is not.
    const ConstLongs ptr = (ConstLongs)uintptr_t(args->sel_ptr + it.pos);
    const int64_t begin = ptr[0], end = ptr[1];
    it.first_block = 0;
    if ((KS == 1 || grp == 0) && !COPIERS) start_item(yes, yes);
    else start_item(no, yes);
    it.sel_begin = begin;
    it.n_sel = int(end - begin);
    have = it.n_sel > 0;
    if (have) {
      const ConstInts sel = (ConstInts)uintptr_t(args->sel_idx + begin);
      it.first_block = sel[0];
      it.second_block = sel[min(1, it.n_sel - 1)];
      own_first();
      if (!COPIERS && (it.first_block != 0 || (KS > 1 && grp == 1))) {
        wait_vmem_all();                             // (of the copies that went to the same stages)
        start_item(yes, no);
      }
    }
  }
  wait_vmem_all();

  // QG: query groups of a wave, one in a half of a row.
  auto process = [&](auto qg_c) __attribute__((always_inline)) {
    constexpr int QG = decltype(qg_c)::value;
    const int q_first = HALVES && QG != QGM ? BQ / 2 * (it.half - 1) + 16 * wave : q_wave;
    if (t_first == 0) t_first = wall_clock64();      // (my_items may still be 0: a second half is not counted)
    my_items += HALVES && it.half == 2 ? 0 : 1;      // (a row in halves is one item, and half of its blocks to either)
    my_cost += uint32_t(HALVES && it.half > 0 ? (it.n_sel + 2 - it.half) / 2 : it.n_sel);
    const int i = it.q_block;
    const int n_pairs = KS > 1 ? (it.n_sel + KS - 1) / KS : it.n_sel;   // tile pairs of every group
    // selected block of the group's tile pair b; read one pair ahead of its first use so
    // that the scalar-memory latency never sits in front of a copy
    const ConstInts sel = (ConstInts)uintptr_t(reload(args)->sel_idx + it.sel_begin);
    auto block_of = [&](int b) { return sel[min(KS > 1 ? b * KS + grp : b, it.n_sel - 1)]; };
    // a group whose blocks ran out repeats the last one with every key masked and leaves its values out
    // (an infinite one, with a probability of zero, would be NaN)
    auto beyond = [&](int b) { return KS > 1 && b * KS + grp >= it.n_sel; };
    int j0 = it.first_block, j1 = KS > 1 ? block_of(1) : it.second_block;

    typedef f32x4 Scores[QG][MT];
    f32x4 acc_o[QG][8];
    float m_ref[QG], l_run[QG];
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) {
      l_run[qg] = 0.0f;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) acc_o[qg][dt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    auto clear_scores = [&](Scores& sc) {
#pragma unroll
      for (int qg = 0; qg < QG; ++qg)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) sc[qg][mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    auto mask_scores = [&](Scores& sc, int half, bool all) {         // diagonal block: keys above the query
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) {
        // key position minus query position, up to the part that depends on the register: taken
        // through an opaque move so that the comparisons are made here, on the rare diagonal
        // tile, instead of being hoisted out of the item loop into 64 scalar registers of masks
        int d = all ? BQ : KT * half + 4 * hi - (q_first + 16 * qg + n);
        asm volatile("" : "+v"(d));
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (d + (16 * mt + r) > 0) sc[qg][mt][r] = -INFINITY;
          asm volatile("" : "+v"(sc[qg][mt]));         // (four masks at a time, not all of them in scalar registers)
        }
      }
    };
    auto read_k = [&](const char* kt, int gi) {       // operand gi = MT*ks + mt of the first contraction
      const int ks = gi / MT, mt = gi % MT;
      return *reinterpret_cast<const bf16x8*>(kt + (k_rd0 ^ (ks << 6)) + mt * 16 * kRowBytes);
    };
    // in-lane maximum of a tile's scores of a query
    auto tile_max = [&](const Scores& sc, int qg) {
      float mx = sc[qg][0][0];
#pragma unroll
      for (int x = 1; x < 4 * MT; ++x) mx = fmaxf(mx, sc[qg][x >> 2][x & 3]);
      return mx;
    };
    auto read_v = [&](const char* vt, int gi) {       // operand gi = 8*gq + dt of the second
      const int gq = gi >> 3, dt = gi & 7;
      const char* at = vt + (v_rd0 ^ (dt << 5)) + gq * 32 * kRowBytes;
      const s16x4 lo = lds_read_tr16(at), up = lds_read_tr16(at + 16 * kRowBytes);
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    // a workgroup that owes (nearly) as many merges as it can note stops taking items; the others carry on
    // (there are far fewer split rows in a launch than the workgroups together can note)
    const bool more = n_merge < kDeferredMerges - 1 && reload(args)->wq.items != nullptr;
    home_open = more && home_open;
    // The next item is asked for two steps before the last one (an item of two tiles: here).
    uint32_t ticket = 0, words = 0;
    int pos = -1;
    auto ask = [&]() {
      if (home_open && tid == 0) {
        int at = home * kTicketStride;               // (in a vector register: for a uniform address the compiler
        asm volatile("" : "+v"(at));                 // would add a use of the result right behind the atomic)
        ticket = __hip_atomic_fetch_add(reload(args)->wq.tickets + at, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    };
    if (n_pairs == 1) ask();

    // ---- S(0).  (The item's copies have landed in this wave: see the end of the loop.)
    Scores sc_a, sc_b;
    if (QS > 1 && q_grp == 1) __builtin_amdgcn_s_barrier();   // half a step behind group 0, which waits at the end
    __syncthreads();
    {
      bf16x8 kf[kQK];
#pragma unroll
      for (int gi = 0; gi < kQK; ++gi) kf[gi] = read_k(k_lds, gi);
      clear_scores(sc_a);
#pragma unroll
      for (int gi = 0; gi < kQK; ++gi)
#pragma unroll
        for (int qg = 0; qg < QG; ++qg)
          sc_a[qg][gi % MT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[gi], qf[qg][gi / MT], sc_a[qg][gi % MT], 0, 0, 0);
      if (j0 == i || beyond(0)) mask_scores(sc_a, 0, beyond(0));
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) m_ref[qg] = quad_max(tile_max(sc_a, qg)) * scale_log2;
    }

    // One step: tile t's softmax and PV from sc_cur, tile t+1's scores into sc_nxt.
    //   stage: t & 1.  jk: block of tile t+2 (kMid only).  mask: tile t+1 is (in) the diagonal block, or `all`
    //   of its keys are to be masked.  drop: tile t belongs to a repeated block.
    // kPlace: kMid inside the item; kRecord the last step but one, kFinal the last one.
    enum { kMid, kRecord, kFinal };
    const Item cur = it;                             // (the last step starts the next item)
    auto step = [&](auto place_c, auto stage_c, Scores& sc_cur, Scores& sc_nxt, int jk, bool mask, bool all,
                    bool drop, bool ask_now, int pair) {   // pair: t / 2
      constexpr int kPlace = decltype(place_c)::value, kStage = decltype(stage_c)::value;
      constexpr bool kHasNext = kPlace != kFinal;
      if (!SCORES_FIRST) __builtin_amdgcn_s_setprio(0);
      if (!COPIERS) wait_vmem_all();    // own copies of K(t+1), V(t) have landed
      if (kPlace == kRecord && home_open && tid == 0) {
        // the ticket asked for one step ago
        if constexpr (HALVES) s_next = ticket < uint32_t(s_home[2]) ? queue_place(s_home[0], s_home[1], int(ticket)) : kHelp;
        else s_next = ticket < home_size ? home_begin + int(ticket) : kHelp;
      }
      __syncthreads();                  // everyone's have; stages of K(t) and V(t-1) are free
      if (kPlace == kMid && kStage == 1 && ask_now) ask();
      if constexpr (kPlace == kRecord) {
        // the next item's record arrives behind this step's work
        pos = home_open ? __builtin_amdgcn_readfirstlane(s_next) : kHelp;
        words = record_words(pos);
      }
      if constexpr (kPlace == kFinal && KS == 1) {
        // all stages but that of V(t) are free and the last scores have been taken: the next item starts
        if (pos >= 0 && read_record(pos, words, it)) start_item(yes, yes);
        else it.n_sel = 0;
      }

      const int odd_pair = COPIERS ? pair & 1 : 0;
      const char* kn = k_lds + (COPIERS ? (kStage == 0 ? 2 * odd_pair + 1 : 2 - 2 * odd_pair) : kStage ^ 1) * kTileBytes;
      const char* vc = v_lds + (2 * odd_pair + kStage) * kTileBytes;

      bf16x8 kf[kQK], vf[kPV];
      if (kHasNext) clear_scores(sc_nxt);

      // ---- the first LDS operands, and the copies of this step
      auto fetch_first = [&]() {
        if (kHasNext) {
#pragma unroll
          for (int gi = 0; gi < kLook; ++gi) kf[gi] = read_k(kn, gi);
        } else {
#pragma unroll
          for (int gi = 0; gi < kLook; ++gi) vf[gi] = read_v(vc, gi);
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      if constexpr (QS == 1) fetch_first();
      if (kHasNext && copies) {
        issue(v_head, v_stage0 + (kStage ^ 1) * kTileBytes);
        if constexpr (kPlace == kMid) {
          locate(jk, kStage);
          issue(k_head, k_stage0 + kStage * kTileBytes);
        }
      }
      __builtin_amdgcn_sched_barrier(0);

      // S(t+1): its MFMAs back to back (the operands of the second contraction are fetched behind the last K operands)
      auto next_scores = [&]() {
        if (kHasNext) {
#pragma unroll
          for (int gi = 0; gi < kQK; ++gi) {
            if (gi + kLook < kQK) kf[gi + kLook] = read_k(kn, gi + kLook);
            if (gi + kLook >= kQK) vf[gi + kLook - kQK] = read_v(vc, gi + kLook - kQK);
#pragma unroll
            for (int qg = 0; qg < QG; ++qg)
              sc_nxt[qg][gi % MT] =
                  __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[gi], qf[qg][gi / MT], sc_nxt[qg][gi % MT], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
          if (mask) mask_scores(sc_nxt, kStage ^ 1, all);
        }
      };
      if (SCORES_FIRST) next_scores();

      // ---- probabilities of tile t, in one run of VALU work: the first K operands arrive behind it, and the other
      // wave of the SIMD is usually inside an MFMA block.
      uint32_t pk[QG][MT][2];
      float rs[QG];
      auto probabilities = [&]() {
        float sum[QG][2];
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) sum[qg][0] = sum[qg][1] = 0.0f;
#pragma unroll
        for (int u = 0; u < 2 * QG * MT; ++u) {       // two probabilities of a query group, the groups in turn
          const int qg = u % QG, mt = u / (2 * QG), c = u / QG % 2;
          const float m_use = m_ref[qg] == -INFINITY ? 0.0f : m_ref[qg];
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc_cur[qg][mt][2 * c], scale_log2, -m_use));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc_cur[qg][mt][2 * c + 1], scale_log2, -m_use));
          pk[qg][mt][c] = pack_bf16(p0, p1);
          // row sums of the rounded probabilities (what the second contraction multiplies with)
          sum[qg][c] = dot2_ones(pk[qg][mt][c], sum[qg][c]);
        }
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) rs[qg] = sum[qg][0] + sum[qg][1];
      };
      probabilities();
      // The reference m_ref was fixed by earlier tiles.  It is too low for this tile exactly
      // when a probability came out large, and then the tile's row sum is large: no maximum
      // over the scores is needed to notice.  In that (rare) case take the tile's true
      // maximum, raise the reference, rescale O and l, and redo the tile's probabilities.  (For 16 queries at a time,
      // so that what a row comes to does not depend on how many a wave has.)
      auto too_low = [&](int qg) { return !(rs[qg] <= kSumLimit); };
      if (__any(too_low(0) || too_low(QG - 1))) {
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) {
          const float m_tile = quad_max(tile_max(sc_cur, qg)) * scale_log2;
          const float m_new = QG == 1 || __any(too_low(qg)) ? fmaxf(m_ref[qg], m_tile) : m_ref[qg];
          const float alpha = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m_ref[qg] - m_new);
          m_ref[qg] = m_new;
          l_run[qg] *= alpha;
#pragma unroll
          for (int dt = 0; dt < 8; ++dt) acc_o[qg][dt] *= alpha;
        }
        probabilities();
      }
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) l_run[qg] += rs[qg];
      __builtin_amdgcn_sched_barrier(0);

      // ---- S(t+1)
      if constexpr (QS > 1) {
        // (group 1 has waited for the copies of K(t+1) and V(t) in front of the barrier that is group 0's this one)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        fetch_first();
      }
      if (!SCORES_FIRST) __builtin_amdgcn_s_setprio(1);
      __builtin_amdgcn_sched_barrier(0);
      if (!SCORES_FIRST) next_scores();

      // ---- O^T += V(t)^T P(t)^T: its MFMAs back to back
      if (KS > 1 && drop) return;
#pragma unroll
      for (int gi = 0; gi < kPV; ++gi) {
        if (gi + kLook < kPV) vf[gi + kLook] = read_v(vc, gi + kLook);
        const int gq = gi >> 3, dt = gi & 7;
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) {
          const u32x4 w = {pk[qg][2 * gq][0], pk[qg][2 * gq][1], pk[qg][2 * gq + 1][0], pk[qg][2 * gq + 1][1]};
          acc_o[qg][dt] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[gi], __builtin_bit_cast(bf16x8, w), acc_o[qg][dt], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };

    using std::integral_constant;
    const integral_constant<int, 0> even{};
    const integral_constant<int, 1> odd{};
    int b = 0;
    for (; b + 1 < n_pairs; ++b) {
      const int j2 = block_of(b + 2);
      step(integral_constant<int, kMid>{}, even, sc_a, sc_b, j1, j0 == i || beyond(b), beyond(b), beyond(b), false, b);
      step(integral_constant<int, kMid>{}, odd, sc_b, sc_a, j1, j1 == i || beyond(b + 1), beyond(b + 1), beyond(b),
           b + 2 == n_pairs, b);
      j0 = j1;
      j1 = j2;
    }
    step(integral_constant<int, kRecord>{}, even, sc_a, sc_b, 0, j0 == i || beyond(b), beyond(b), beyond(b), false, b);
    step(integral_constant<int, kFinal>{}, odd, sc_b, sc_a, 0, false, false, beyond(b), false, b);

    // ---- the next item starts before this one's results are written
    float l_tot[QG];
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) l_tot[qg] = quad_sum(l_run[qg]);
    if (QS > 1 && q_grp == 0) __builtin_amdgcn_s_barrier();
    auto own = [&](int dt) { return KS == 1 || dt / (8 / KS) == grp; };   // dim tiles a group ends up with
    if constexpr (KS > 1) {
      __syncthreads();                               // every wave is done with the stages
      // The groups combine their partial results (the softmax of Eq. 1 over the union of their keys): group g
      // ends up with the dims 16 dt .. of the dt's that are its own.
      f32x4* xo = reinterpret_cast<f32x4*>(lds);
      auto chunk = [&](int g, int qg, int dt) { return ((((g * QG + qg) * 8 + dt) * kWaves + wave) << 6) + lane; };
      float* const ml = s_ml + wave * 32 + n;        // + 2 BQ group + 16 qg (+ BQ: denominators)
      constexpr int kOwn = 8 / KS;
      auto combine = [&](auto own_c) {               // (the group as a constant: no branch per dim tile)
        constexpr int kGroup = decltype(own_c)::value, kOther = KS - 1 - kGroup;
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) {
          if (hi == 0) {
            ml[kGroup * 2 * BQ + 16 * qg] = m_ref[qg];
            ml[kGroup * 2 * BQ + BQ + 16 * qg] = l_tot[qg];
          }
#pragma unroll
          for (int x = 0; x < kOwn; ++x) xo[chunk(kGroup, qg, kOther * kOwn + x)] = acc_o[qg][kOther * kOwn + x];
        }
        __syncthreads();
        f32x4 other[QG][kOwn];
        float m_other[QG], l_other[QG];
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) {
          m_other[qg] = ml[kOther * 2 * BQ + 16 * qg];
          l_other[qg] = ml[kOther * 2 * BQ + BQ + 16 * qg];
#pragma unroll
          for (int x = 0; x < kOwn; ++x) other[qg][x] = xo[chunk(kOther, qg, kGroup * kOwn + x)];
        }
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) {
          const float m_all = fmaxf(m_ref[qg], m_other[qg]);
          const float w = m_ref[qg] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m_ref[qg] - m_all);
          const float w_other = m_other[qg] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m_other[qg] - m_all);
          l_tot[qg] = kGroup == 0 ? w * l_tot[qg] + w_other * l_other[qg] : w_other * l_other[qg] + w * l_tot[qg];
          m_ref[qg] = m_all;
#pragma unroll
          for (int x = 0; x < kOwn; ++x) acc_o[qg][kGroup * kOwn + x] = w * acc_o[qg][kGroup * kOwn + x] + w_other * other[qg][x];
        }
      };
      if (grp == 0) combine(std::integral_constant<int, 0>{});
      else combine(std::integral_constant<int, KS - 1>{});
      __syncthreads();                               // the stages are free again
    }
    home_open = pos != kHelp;
    if (KS > 1 || (more && it.n_sel <= 0)) {
      if (KS == 1) __syncthreads();                  // every wave is done with the stages
      have = KS > 1 && pos >= 0 && read_record(pos, words, it);
      while (more && !have) {                        // (again after a row without a block)
        pos = help();
        if (pos < 0) break;
        have = read_record(pos, record_words(pos), it);
      }
      if (have) {
        own_first();
        start_item(yes, yes);
      }
    } else {
      have = more && it.n_sel > 0;
    }

    // ---- normalise and store: lane holds, for its queries, dims 16dt + 4hi + r
    int q_in = q_first + n;                          // + 16 qg
    asm volatile("" : "+v"(q_in));                   // output addresses are made here, not carried through the loop
    ArgsPtr a = reload(args);
    const int q0 = cur.seq_begin + cur.q_block * BQ;
    if (!COPIERS && cur.slot >= 0) {
      // a piece of a split row: O and l as they stand (relative to 2^m_ref), for merge_row()
      float* part = a->sb.part_o + int64_t(cur.slot) * kSlotFloatsO;
      float* ml = a->sb.part_ml + int64_t(cur.slot) * kSlotFloatsML;
#pragma unroll
      for (int qg = 0; qg < QG; ++qg) {
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
          if (own(dt)) {
            float* dst = part + slot_chunk(q_first / 16 + qg, dt, lane);
            slot_store(dst, acc_o[qg][dt][0], acc_o[qg][dt][1]);
            slot_store(dst + 2, acc_o[qg][dt][2], acc_o[qg][dt][3]);
          }
        if (hi == 0 && grp == 0) {
          slot_store1(ml + q_in + 16 * qg, m_ref[qg]);
          slot_store1(ml + 128 + q_in + 16 * qg, l_tot[qg]);
        }
      }
      // count the piece; if it completes its row, note the row for the merge after the loop
      const ItemRec* rec = a->wq.items + cur.pos;
      const SplitBuffers sb = {a->sb.part_o, a->sb.part_ml, a->sb.done, a->sb.slot_capacity};
      if (count_piece(sb, rec->pieces, rec->split_index, &s_flag)) {
        if (tid == 0) s_merge[n_merge] = cur.pos;
        n_merge += 1;
      }
      wait_vmem_all();
    } else {
      // The four lanes of a query hold runs of four dims (8 bytes as bf16) of every dim tile.  Neighbours trade
      // runs of two tiles so that each ends up with eight consecutive dims of one of them, and a row goes out in
      // 16-byte stores, four lanes per 64 bytes.
      const int n_valid = cur.seq_end - q0;
      constexpr int kPairs = 4, kStores = QG * kPairs;   // pairs of dim tiles; 16-byte stores of a lane
      auto store_rows = [&](bool all) {
#pragma unroll
        for (int qg = 0; qg < QG; ++qg) {
          const int q_at = q_in + 16 * qg;
          const bool valid = all || q_at < n_valid;
          const float inv = 1.0f / l_tot[qg];
          if (a->lse != nullptr && hi == 0 && grp == 0 && valid)
            a->lse[int64_t(cur.head) * a->total_tokens + q0 + q_at] =
                (m_ref[qg] + __builtin_amdgcn_logf(l_tot[qg])) * 0.6931471805599453f;
          uint16_t* dst = a->out + int64_t(q0 + min(q_at, n_valid - 1)) * a->st.q_t + int64_t(cur.head) * a->st.q_h +
                          16 * (hi & 1) + 8 * (hi >> 1);
#pragma unroll
          for (int p = 0; p < kPairs; ++p)
            if (own(2 * p)) {
              const f32x4 &x = acc_o[qg][2 * p], &y = acc_o[qg][2 * p + 1];
              uint32_t e0 = pack_bf16(x[0] * inv, x[1] * inv), e1 = pack_bf16(x[2] * inv, x[3] * inv);
              uint32_t o0 = pack_bf16(y[0] * inv, y[1] * inv), o1 = pack_bf16(y[2] * inv, y[3] * inv);
              swap_rows(e0, o0);                         // lanes of even hi: both runs of the even tile; of odd hi: of the odd one
              swap_rows(e1, o1);
              if (valid) *reinterpret_cast<u32x4*>(dst + 32 * p) = u32x4{e0, e1, o0, o1};
            }
        }
      };
      // The next item's copies and Q loads were issued before these stores, and the vector memory operations of
      // a wave are reported complete in the order they were issued, loads and stores alike (LLVM's AMDGPU usage
      // guide, memory model of gfx6 to gfx9 and of gfx942; flat accesses to LDS are the exception, and none is under
      // way here): with at most the stores outstanding the copies have landed.  For that the stores must stay in
      // front of the wait.
      if (KS == 1 && q_first + 16 * QG <= n_valid) {
        store_rows(true);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        wait_vmem_but(std::integral_constant<int, kStores>{});
      } else {
        store_rows(false);
        wait_vmem_all();
      }
    }
    // (said to the compiler too, which would else wait for the stores in front of the first use)
#pragma unroll
    for (int qg = 0; qg < QGM; ++qg)
      asm volatile("" : "+v"(qf[qg][0]), "+v"(qf[qg][1]), "+v"(qf[qg][2]), "+v"(qf[qg][3]));
    t_last = wall_clock64();
  };
  while (have) {
    if (HALVES && it.half > 0) process(std::integral_constant<int, HALVES ? 1 : QGM>{});
    else process(std::integral_constant<int, QGM>{});
  }

  // ---- rows whose pieces are all done and whose last piece this workgroup computed (COPIERS: rows are whole)
  if constexpr (!COPIERS) for (int x = 0; x < n_merge; ++x) {
    __syncthreads();                                   // s_merge as thread 0 left it
    ArgsPtr a = reload(args);
    const ItemRec* item = a->wq.items + s_merge[x];
    const int q0 = item->seq_begin + item->query_block * BQ, h = item->head;
    const SplitBuffers sb = {a->sb.part_o, a->sb.part_ml, a->sb.done, a->sb.slot_capacity};
    merge_row<BQ, kThreads>(sb, item->pieces, item->first_slot, a->out + int64_t(q0) * a->st.q_t + int64_t(h) * a->st.q_h,
                            a->st.q_t, a->lse != nullptr ? a->lse + int64_t(h) * a->total_tokens + q0 : nullptr,
                            min(BQ, item->seq_end - q0), reinterpret_cast<float*>(lds),
                            reinterpret_cast<float*>(lds) + kMaxPieces * BQ);
    t_last = wall_clock64();
  }

  if (args->stats != nullptr && tid == 0) {
    shplb_wg_stats rec;
    rec.xcc_id = uint32_t(my_xcd());
    rec.cu_id = (__builtin_amdgcn_s_getreg((16 - 1) << 11 | 0 << 6 | 4) >> 8) & 0xff; // HW_ID[15:8]
    rec.n_items = my_items;
    rec.cost_blocks = my_cost;
    rec.t_first = t_first;
    rec.t_last = t_last;
    args->stats[blockIdx.x] = rec;
    // a launch with fewer workgroups than records
    for (int x = blockIdx.x + gridDim.x; x < args->n_stats; x += gridDim.x) args->stats[x] = shplb_wg_stats{};
  }
}

template <int BQ, int GROUPS, bool SCORES_FIRST = false, bool COPIERS = false, bool HALVES = false>
void launch_one(const AttnArgs& args, int n_wg, hipStream_t stream) {
  hipLaunchKernelGGL((attn_pipe_kernel<BQ, GROUPS, SCORES_FIRST, COPIERS, HALVES>), dim3(n_wg), dim3(64 * (GROUPS * BQ / 32 + (COPIERS ? GROUPS : 0))),
                     0, stream, args);
}

}  // namespace

AttentionPlan plan_attention(const Geometry& g, int32_t n_wg, int64_t slot_capacity) {
  AttentionPlan plan;
  const int cus = plan.compute_units = n_wg / (g.meta.block == 64 ? 4 : 2);
  // A launch of few 64-token rows leaves half of every compute unit's SIMDs without a wave (a row is two
  // waves), and its length is that of the chain of tiles of the longest row: two groups of waves per row
  // halve that chain.  256 rows of up to 16 blocks 24.6 -> 18.1 us, 512 rows 28.2 -> 21.6 us, 64 rows of up to
  // 8 blocks 14.8 -> 11.8 us; at 1024 rows, where the chip is full without them, 54 -> 57 and 38 -> 51 us.
  // A 128-token row fills the SIMDs by itself, but with no more rows than compute units every SIMD has one wave and its
  // MFMAs and softmax wait for each other: two groups of waves share it, 64 queries each and half a step apart.  Not by
  // its keys: a query's sums are taken in the order of the other launches, bit for bit, and short rows combine nothing.
  // Whole path, one group against two: 32/8 heads x 777 tokens 32.0 -> 28.4 us, with two blocks a row 22.0 -> 21.1, 8/2 x
  // 4096 at 20 to 100% 68.7 -> 57.4, 16/4 x 2048 with two or three blocks a row 27.2 -> 25.8, 4/1 x 8000 with a dense one
  // 155 -> 125, 1/1 x 20000 dense 347 -> 266 (by keys 31.0, 23.2, 58.4, 29.3, 120 and 251), in pieces 4/1 x 8000 82.0 -> 74.1,
  // 2/1 x 16384 151 -> 141, 16/4 x 2048 63.9 -> 56.0.  512 rows are two rows a compute unit, which fill it.
  plan.groups = g.rows <= (g.meta.block == 64 ? 2 * cus : cus) ? 2 : 1;
  plan.grid = n_wg / plan.groups;
  // No more rows than workgroups and none to be cut: there is nothing to order, every row gets a workgroup
  // of its own (777 tokens x 32 heads: 42.6 us for the whole path with the ordering launch, 35.5 without).
  plan.ordered = slot_capacity > 0 || g.rows > plan.grid - plan.grid % kXcds;
  // Whole rows from queues: the ordering kernel may have long ones worked on in halves, if a row can be that long (every row of
  // two blocks and more selects at least two), by an instance of the kernel that has both.  Where there is nothing to halve, the
  // attention call takes 0.2 to 3% longer by it (8231 tokens x 32/8 heads 144.9 -> 148.1 us, x 28/4 130.4 -> 131.4, 12000 x 32/8 263.9 -> 271.0,
  // 6000 x 40/8 109.4 -> 113.1), on long launches, whose rows
  // hardly reach the share, 0.9% (32K x 32/8, 64K x 8/2): up to six rows a workgroup.  With 64-token blocks, where a half has as many
  // copies for half of the products of which there are few, 6933 x 32/8 with a dense head gains 10%, 8/8 x (1265, 6884, 1553) loses 4%.
  const int64_t n_sh = int64_t(g.meta.n_seq) * g.meta.n_q_heads;
  plan.halves = plan.ordered && slot_capacity == 0 && plan.groups == 1 && g.meta.block == 128 && g.rows <= 6 * n_wg &&
                places_counted(g, false) && worth_halves(g.max_nb, 2 * g.rows - n_sh, n_wg);
  return plan;
}

int32_t launch_attention(const Geometry& g, const AttentionPlan& plan, const void* q, const void* k, const void* v,
                         const int64_t* sel_ptr, const int32_t* sel_idx, void* out, float* lse,
                         shplb_wg_stats* stats, WorkQueues wq, SplitBuffers sb, int32_t n_wg, hipStream_t stream) {
  AttnArgs args{};
  args.q = static_cast<const uint16_t*>(q);
  args.k = static_cast<const uint16_t*>(k);
  args.v = static_cast<const uint16_t*>(v);
  args.sel_ptr = sel_ptr;
  args.sel_idx = sel_idx;
  args.out = static_cast<uint16_t*>(out);
  args.lse = lse;
  args.stats = stats;
  args.n_stats = n_wg;
  args.rows = int32_t(g.rows);
  args.rows_per_die = g.rows <= plan.compute_units ? int32_t((g.rows + kXcds - 1) / kXcds) : 0;
  args.compute_units = plan.compute_units;
  args.group = g.meta.kv_map ? 0 : g.meta.n_q_heads / g.meta.n_kv_heads;
  args.scale_log2 = g.scale * 1.4426950408889634f;
  args.total_tokens = g.total_tokens;
  args.st = g.st;
  args.wq = wq;
  args.sb = sb;
  args.meta = g.meta;
  if (g.meta.block == 128) {
    if (plan.groups == 2) launch_one<128, 2>(args, plan.grid, stream);
    else if (plan.halves) launch_one<128, 1, false, false, true>(args, plan.grid, stream);
    else launch_one<128, 1>(args, plan.grid, stream);
  } else {
    if (plan.groups == 2 && wq.items == nullptr && args.rows_per_die > 0) launch_one<64, 2, true, true>(args, plan.grid, stream);
    else if (plan.groups == 2 && wq.items == nullptr) launch_one<64, 2, true>(args, plan.grid, stream);
    else if (plan.groups == 2) launch_one<64, 2>(args, plan.grid, stream);
    else launch_one<64, 1>(args, plan.grid, stream);
  }
  if (hipGetLastError() != hipSuccess) return SHPLB_E_HIP;
  return SHPLB_OK;
}

}  // namespace shplb
