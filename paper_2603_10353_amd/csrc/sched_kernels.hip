// Work-item ordering for the persistent attention launch.
//
// The paper's greedy (Section 3.3) sorts units by descending cost and hands each to the
// least-loaded worker.  On one GPU the workers are compute units: the rows (sequence,
// head, query block) are sorted by descending selected-block count and consumed through
// atomic tickets, so the next-largest item always goes to a workgroup that just became
// free.  MI355X has eight dies (XCDs), each with its own L2, so there is one sorted queue
// per die: all rows that stream one KV head of one sequence share a home die, whose L2 then
// sees that K/V once.  A workgroup drains its die's queue first and then helps whichever die
// has the most items left (see help_item()), which keeps the greedy's balance when the dies'
// queues hold very different amounts of work.
//
// Rows of up to 2048 (sequence, head) pairs find their places without a sort: see place_kernel.  Launches of more pairs
// go through one launch of eight workgroups (order_kernel); workgroup x builds the queue of die x with a counting sort
// whose histogram (one entry per possible cost) lies in LDS: count, scan, place.  It looks
// only at the rows that live on its die; where its queue begins follows from the shapes
// alone, so the workgroups need nothing from each other.  Rows of equal cost are placed in
// the order their LDS atomics arrive: that decides only which workgroup takes which of two
// equally long rows, results do not depend on it.
//
// When the caller provides slots for partial results (shplb_sparse_attn_prefill_split), rows
// longer than split_length() are cut along their selected key blocks into near-equal pieces,
// each an item of its own (the pieces of a row sit next to each other, where the row would).
// A piece leaves a partial result in a slot of the workspace; the piece of a row that finishes
// last combines them (count_piece() and merge_row() in attn_common.h).  Slots and counter
// entries are handed out in the same arbitrary order; what is computed does not depend on it.
//
// Launches without splitting that have no more rows than workgroups skip all this: see row_place() in
// attn_pipe_kernel.hip.
//
// What bounds order_kernel: a chain of dependent memory round trips (geometry, row pointer, first
// selected blocks, record) on eight compute units.  A thread works out one (sequence, head)
// pair, a prefix sum over the pairs lies in LDS, and threads then find their rows in it by
// bisection: nothing loops over sequences and no lane is idle when sequences are short.
#include <type_traits>

#include "shplb_internal.h"

namespace shplb {
namespace {

constexpr int kOrderThreads = 1024;
constexpr int kOrderWaves = kOrderThreads / 64;
constexpr int kPairs = 2;                 // (sequence, head) pairs of a thread
constexpr int kBatch = kPairs * kOrderThreads;   // pairs looked at together
constexpr int kInFlight = 4;              // rows a thread has in flight

// Which rows of a (sequence, head) pair die x holds.  All rows that stream the same K/V (one
// KV head of one sequence) go to the same die, so its L2 sees one K/V stream per resident head
// instead of all of them; with fewer streams than dies a stream is spread over `per` dies by
// query block.  The rows are those whose query block i has i % mod in [first, first + width).
struct PairRows {
  int count, first, width, mod;
  // query block of the pair's r-th row here
  static __device__ __forceinline__ int block_of(int r, int first, int width, int mod) {
    return mod == 1 ? r : (r / width) * mod + first + r % width;
  }
};
// and_earlier: the rows of the dies before x too.
__device__ __forceinline__ PairRows pair_rows(const SeqMeta& m, int stream, int nb, int x, bool and_earlier) {
  const int n_streams = m.n_seq * m.n_kv_heads;
  PairRows r{0, 0, 1, 1};
  if (n_streams >= kXcds) {
    const int die = stream % kXcds;
    r.count = die == x || (and_earlier && die < x) ? nb : 0;
    return r;
  }
  r.mod = kXcds / n_streams;
  const int last = x - stream * r.mod;                 // residue that belongs to die x, if in 0 .. mod-1
  r.first = and_earlier ? 0 : last;
  r.width = and_earlier ? min(last, r.mod - 1) + 1 : 1;
  if (last < 0 || (!and_earlier && last >= r.mod)) return PairRows{0, 0, 1, r.mod};
  r.count = nb / r.mod * r.width + min(max(nb % r.mod - r.first, 0), r.width);
  return r;
}

// Inclusive sum over the lanes of a wave, by data-parallel-primitive shifts (no LDS round trips).
__device__ __forceinline__ int wave_scan(int v) {
  auto dpp = [](int x, auto ctrl, auto rows) {
    return __builtin_amdgcn_update_dpp(0, x, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
  };
  using std::integral_constant;
  v += dpp(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});   // row_shr 1, 2, 4, 8: rows of 16
  v += dpp(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
  v += dpp(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
  v += dpp(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
  v += dpp(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});   // last lane of rows 0, 2 into rows 1, 3
  v += dpp(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});   // last lane of row 1 into rows 2, 3
  return v;
}
// Sum over the threads before this one, and over all.  One barrier; s_wave must be free before the call.
__device__ __forceinline__ int block_scan(int v, int32_t (&s_wave)[kOrderWaves], int& total) {
  static_assert(kOrderWaves == 16, "the waves' sums are scanned inside a row of 16 lanes");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int inc = wave_scan(v);
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  const int waves = wave_scan(lane < kOrderWaves ? s_wave[lane] : 0);
  total = __builtin_amdgcn_readlane(waves, kOrderWaves - 1);
  return inc - v + (wave > 0 ? __builtin_amdgcn_readlane(waves, wave - 1) : 0);
}

// Add one to bins[bin] for every active lane; returns the lane's own position.  The rows of a wave are
// mostly neighbours of one head: their cost climbs with the query block and then stays at the head's
// budget, so one entry gets most of the wave (and the next head's plateau a second one): LDS atomics on
// one address go one lane at a time.  Those two are counted by ballot, the rest lane by lane.
__device__ __forceinline__ int take_places(int32_t* bins, int bin, bool active) {
  int pos = 0;
#pragma unroll
  for (int round = 0; round < 2; ++round) {
    const uint64_t open = __ballot(active);
    if (open == 0) break;
    const int lead = round == 0 ? 63 - __builtin_clzll(open) : __builtin_ctzll(open);
    const int b = __builtin_amdgcn_readlane(bin, lead);
    const uint64_t same = __ballot(active && bin == b);
    int at = 0;
    if ((threadIdx.x & 63) == lead) at = atomicAdd(&bins[b], __builtin_popcountll(same));
    at = __builtin_amdgcn_readlane(at, lead);
    if (active && bin == b) {
      pos = at + int(__builtin_amdgcn_mbcnt_hi(uint32_t(same >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(same), 0u)));
      active = false;
    }
  }
  if (active) pos = atomicAdd(&bins[bin], 1);
  return pos;
}

__global__ __launch_bounds__(kOrderThreads) void order_kernel(
    SeqMeta meta, const int64_t* __restrict__ sel_ptr, const int32_t* __restrict__ sel_idx,
    ItemRec* __restrict__ items, int32_t* __restrict__ queue_begin, uint32_t* __restrict__ tickets,
    uint32_t* __restrict__ split_done, int rows, int n_bins, int item_capacity, int slot_capacity, int n_wg,
    int grid) {
  __shared__ int32_t bins[kCostBins];     // items per cost, then next free position per cost
  __shared__ int32_t s_wave[4][kOrderWaves];
  __shared__ int32_t s_slots, s_split;    // next free slot and finished-pieces counter
  __shared__ int32_t s_pre[kBatch];       // rows of the batch's earlier pairs, per pair
  __shared__ int32_t s_row0[kBatch];      // row of the pair's query block 0
  __shared__ uint32_t s_res[kBatch];      // PairRows.first | width << 8 | sequence << 16
  // the geometry, which is read by lane-dependent index
  __shared__ int32_t s_blk[SHPLB_MAX_SEQ + 1], s_tok[SHPLB_MAX_SEQ + 1];
  __shared__ uint32_t s_kv[SHPLB_MAX_MAPPED_HEADS / 4];
  const int x = blockIdx.x;               // the die
  const int tid = threadIdx.x;
  const int hq = meta.n_q_heads, n_pairs = meta.n_seq * hq;
  const bool spread = meta.n_seq * meta.n_kv_heads < kXcds;
  const int mod = spread ? kXcds / (meta.n_seq * meta.n_kv_heads) : 1;
  const bool split = slot_capacity >= 2;
  for (int b = tid; b < n_bins; b += kOrderThreads) bins[b] = 0;
  if (tid <= meta.n_seq) {
    s_blk[tid] = meta.blk_begin[tid];
    s_tok[tid] = meta.tok_begin[tid];
  }
  if (meta.kv_map && tid < SHPLB_MAX_MAPPED_HEADS / 4) s_kv[tid] = meta.kv_of[tid];
  const int group = meta.kv_map ? 1 : hq / meta.n_kv_heads;
  auto kv_head = [&](int h) { return meta.kv_map ? int(s_kv[h >> 2] >> (8 * (h & 3)) & 0xff) : h / group; };
  __syncthreads();
  const int64_t split_len = split ? split_length(sel_ptr[rows] - sel_ptr[0], slot_capacity, n_wg, meta.block) : 0;

  // Lay the batch of pairs from `base` on out in LDS (its arrays and s_wave[0], s_wave[1] must be free);
  // returns its number of rows, adds to `earlier` the rows its pairs have on dies before this one.
  auto load_batch = [&](int base, bool and_earlier, int& earlier) {
    PairRows r[kPairs];
    int row0[kPairs], seq_of[kPairs], mine = 0, mine_earlier = 0, n_batch = 0, n_earlier = 0;
#pragma unroll
    for (int u = 0; u < kPairs; ++u) {
      const int p = base + kPairs * tid + u;
      r[u] = PairRows{0, 0, 1, mod};
      row0[u] = seq_of[u] = 0;
      if (p >= n_pairs) continue;
      const int s = p / hq, h = p - s * hq, b0 = s_blk[s], nb = s_blk[s + 1] - b0;
      const int stream = s * meta.n_kv_heads + kv_head(h);
      row0[u] = b0 * hq + h * nb;
      seq_of[u] = s;
      r[u] = pair_rows(meta, stream, nb, x, and_earlier);
      mine += r[u].count;
      if (!and_earlier) mine_earlier += pair_rows(meta, stream, nb, x - 1, true).count;
    }
    int pre = block_scan(mine, s_wave[0], n_batch);
    if (!and_earlier) block_scan(mine_earlier, s_wave[1], n_earlier);
#pragma unroll
    for (int u = 0; u < kPairs; ++u) {
      const int at = kPairs * tid + u;
      s_pre[at] = pre;
      s_row0[at] = row0[u];
      s_res[at] = uint32_t(r[u].first | r[u].width << 8 | seq_of[u] << 16);
      pre += r[u].count;
    }
    __syncthreads();
    earlier += n_earlier;
    return n_batch;
  };
  // Rows r0, r0 + kOrderThreads, ... of the batch (-1: past its end), all their loads in flight together.
  int row[kInFlight], pair[kInFlight], seq[kInFlight], block[kInFlight], n_sel[kInFlight];
  int first_j[kInFlight], second_j[kInFlight];
  int64_t sel_begin[kInFlight];
  auto fetch = [&](int r0, int n_rows, bool with_blocks) {
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const int r = r0 + u * kOrderThreads;
      row[u] = -1;
      if (r >= n_rows) continue;
      int lo = 0;
#pragma unroll
      for (int d = kBatch / 2; d >= 1; d >>= 1)
        if (s_pre[lo + d] <= r) lo += d;
      const int res = int(s_res[lo]);
      pair[u] = lo;
      seq[u] = res >> 16;
      block[u] = PairRows::block_of(r - s_pre[lo], res & 0xff, res >> 8 & 0xff, mod);
      row[u] = s_row0[lo] + block[u];
    }
    int64_t end[kInFlight];
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const int at = max(row[u], 0);
      sel_begin[u] = sel_ptr[at];
      end[u] = sel_ptr[at + 1];
    }
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      n_sel[u] = row[u] < 0 ? 0 : int(min(max(end[u] - sel_begin[u], int64_t(0)), int64_t(kCostBins - 1)));
      first_j[u] = with_blocks && n_sel[u] > 0 ? sel_idx[sel_begin[u]] : 0;
      second_j[u] = with_blocks && n_sel[u] > 0 ? sel_idx[sel_begin[u] + min(1, n_sel[u] - 1)] : 0;
    }
  };

  // ---- count: items per cost on this die; items (and slots, split rows) of the dies before it
  int begin = 0, before = 0, slots = 0, splits = 0;   // without splitting every row is one item and the shapes say `begin`
  int n_rows = 0;
  for (int base = 0; base < n_pairs; base += kBatch) {
    if (base > 0) __syncthreads();
    n_rows = load_batch(base, split, begin);
    for (int r0 = tid; r0 - tid < n_rows; r0 += kInFlight * kOrderThreads) {
      fetch(r0, n_rows, false);
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        if (!split) {
          take_places(bins, min(n_sel[u], n_bins - 1), row[u] >= 0);
        } else if (row[u] >= 0) {
          const int pieces = pieces_of(n_sel[u], split_len);
          const int stream = seq[u] * meta.n_kv_heads + kv_head(base + pair[u] - seq[u] * hq);
          const int die = spread ? stream * mod + block[u] % mod : stream % kXcds;
          if (die == x) {
            atomicAdd(&bins[min(n_sel[u], n_bins - 1)], pieces);
          } else {
            before += pieces;
            slots += pieces > 1 ? pieces : 0;
            splits += pieces > 1;
          }
        }
      }
    }
  }
  __syncthreads();
  if (split) {
    block_scan(before, s_wave[0], begin);
    block_scan(slots, s_wave[1], slots);
    block_scan(splits, s_wave[2], splits);
  }
  if (tid == 0) {
    queue_begin[x] = begin;
    tickets[x * kTicketStride] = uint32_t(grid - x + kXcds - 1) / kXcds;   // workgroups x, x + 8, ... take one item each without asking
    s_slots = slots;
    s_split = splits;
  }

  // ---- exclusive scan in descending-cost order (position k <-> bin n_bins-1-k), a thread owns a run of bins
  const int per = (n_bins + kOrderThreads - 1) / kOrderThreads;
  const int k0 = min(tid * per, n_bins), k1 = min(k0 + per, n_bins);
  int mine = 0, n_items = 0;
  for (int k = k0; k < k1; ++k) mine += bins[n_bins - 1 - k];
  int run = begin + block_scan(mine, s_wave[3], n_items);
  for (int k = k0; k < k1; ++k) {
    const int c = bins[n_bins - 1 - k];
    bins[n_bins - 1 - k] = run;
    run += c;
  }
  if (x == kXcds - 1 && tid == 0) queue_begin[kXcds] = begin + n_items;
  __syncthreads();

  // ---- place
  for (int base = 0; base < n_pairs; base += kBatch) {
    int unused = 0;
    if (base > 0) __syncthreads();
    n_rows = load_batch(base, false, unused);
    for (int r0 = tid; r0 - tid < n_rows; r0 += kInFlight * kOrderThreads) {
      fetch(r0, n_rows, true);
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        const int n = n_sel[u], bin = min(n, n_bins - 1), pieces = split ? pieces_of(n, split_len) : 1;
        int dst = 0;
        if (!split) dst = take_places(bins, bin, row[u] >= 0);
        else if (row[u] >= 0) dst = atomicAdd(&bins[bin], pieces);
        if (row[u] < 0) continue;
        const int h = base + pair[u] - seq[u] * hq;
        ItemRec rec;
        rec.unused = 0;
        rec.n_sel = n;
        rec.sel_begin = sel_begin[u];
        rec.slot = rec.first_slot = rec.split_index = -1;
        rec.pieces = pieces;
        rec.seq_begin = s_tok[seq[u]];
        rec.seq_end = s_tok[seq[u] + 1];
        rec.head = h;
        rec.kv_head = kv_head(h);
        rec.query_block = block[u];
        rec.n_blocks = s_blk[seq[u] + 1] - s_blk[seq[u]];
        rec.first_block = first_j[u];
        rec.second_block = second_j[u];
        if (dst < 0 || dst + pieces > item_capacity) continue;   // ruled out by split_length(); keeps stores in bounds
        if (pieces <= 1) {
          items[dst] = rec;
          continue;
        }
        const int slot = atomicAdd(&s_slots, pieces), entry = atomicAdd(&s_split, 1);
        if (slot + pieces > slot_capacity || entry >= slot_capacity / 2 + 1) continue;   // likewise
        split_done[entry] = 0;
        rec.first_slot = slot;
        rec.split_index = entry;
        for (int c = 0; c < pieces; ++c) {
          const int64_t first = piece_begin(n, pieces, c);
          rec.n_sel = int(piece_begin(n, pieces, c + 1) - first);
          rec.sel_begin = sel_begin[u] + first;
          rec.slot = slot + c;
          rec.first_block = sel_idx[rec.sel_begin];
          rec.second_block = sel_idx[rec.sel_begin + min(1, rec.n_sel - 1)];
          items[dst + c] = rec;
        }
      }
    }
  }
}

// The queues without a sort: where a row goes follows from its own number of blocks and
// from the budgets of the heads on its die, and every row works it out for itself.
//
// A row of query block i selects c = min(k, i + 1) blocks, k being what the last row of its (sequence, head) pair
// selects.  So the rows with more than c blocks are counted pair by pair, nb - c of each pair with k > c, and so are those with
// as many in front of it (pairs in order, then query blocks).  Keys are taken from k and i alone, never from a row's own entry in sel_ptr: the
// places are then a permutation whatever sel_ptr holds (a caller may list other blocks than a budget's), only
// the order is by cost just where rows are those of a budget.  The record holds what sel_ptr says.
//
// Pieces (kPieces): a row of c blocks is cut into one piece more for every m with m len < c, so the items in front of a row are
// the rows with more than max(c, m len) blocks, summed over m.  The length is split_length() of the budgets' cost, which is the selection's where
// rows are those of a budget: never more pieces than slots.  Split rows are the first of their queues, so slots and counters are
// numbered like items and rows, behind those of the dies before.  A row that is not its budget's is cut into as many pieces
// as its place has room for, or as it has blocks.
//
// A workgroup takes 32 consecutive rows of a stream (the heads of one KV head of one sequence; with a caller's map of heads,
// of one head), eight lanes each, which share the pairs of the die between them and write the record together.  An extra
// workgroup at the end writes the queues' beginnings and tickets, and with `halves` how many rows of each queue are worked on in
// halves (the longest ones, so the first; see halved_above()).
// What bounds it is the chain arguments -> row pointer -> first blocks, with the pairs' budgets behind the
// arguments at the same time; nothing is sorted, and it takes as many compute units as there are rows for.  Under
// the tracer, order_kernel against this: 8K prompt x 32 heads 9.7 -> 5.6 us, 48 sequences x 28 heads 10.2 -> 6.5, 32K x 32
// heads 12.0 -> 5.2, 128K 26 -> 5.7 (whole path: 8K 180.6 -> 175.1 us, the 48 sequences 145.4 -> 143.3).  With the pairs
// listed one by one, a division each, instead of by streams the 48 sequences took 7.9.  In pieces, whole path: 16K x 32 heads
// with four dense ones 546 -> 538 us, 3000 x 32 with a dense one 75.1 -> 70.0, 9000 x 28 with 64-token blocks 276 -> 268.
constexpr int kPlaceThreads = 256, kPlaceLanes = 8, kPlaceRows = kPlaceThreads / kPlaceLanes;

template <bool kPieces>
__global__ __launch_bounds__(kPlaceThreads) void place_kernel(
    SeqMeta meta, const int64_t* __restrict__ sel_ptr, const int32_t* __restrict__ sel_idx,
    ItemRec* __restrict__ items, int32_t* __restrict__ queue_begin, uint32_t* __restrict__ tickets, uint32_t* __restrict__ split_done,
    int item_capacity, int slot_capacity, int n_wg, int grid, int halves) {
  __shared__ int32_t s_blk[SHPLB_MAX_SEQ + 1], s_tok[SHPLB_MAX_SEQ + 1];
  __shared__ uint32_t s_kv[SHPLB_MAX_MAPPED_HEADS / 4];
  __shared__ uint32_t s_unit[kPlacePairs];   // units on this die: number of the first pair | blocks << 16 ...
  __shared__ int32_t s_row[kPlacePairs];     // ... and first row
  __shared__ uint32_t s_pair[kPlacePairs];   // their pairs: number | blocks << 16 ...
  __shared__ int32_t s_k[kPlacePairs];       // ... and blocks of the last row
  __shared__ int32_t s_count, s_before, s_total[kXcds], s_halved[kXcds];
  // pieces: of all pairs the blocks of the last row | blocks << 13 | die << 26 (0 the workgroup's, 1 before it, 2 behind it);
  // all blocks selected; slots and split rows on the dies before
  __shared__ uint32_t s_all[kPlacePairs];
  __shared__ unsigned long long s_cost;
  __shared__ int32_t s_slots, s_splits;
  static_assert(SHPLB_MAX_BLOCKS < 1 << 13, "");
  static_assert(SHPLB_MAX_SEQ < kPlaceThreads && SHPLB_MAX_BLOCKS < 1 << 16 && kPlacePairs <= 1 << 16, "");
  const int tid = threadIdx.x, lane = tid & 63;
  // asked for together: the geometry, of which a lane-dependent index is read
  const int my_blk = meta.blk_begin[min(tid, SHPLB_MAX_SEQ)], my_tok = meta.tok_begin[min(tid, SHPLB_MAX_SEQ)];
  const uint32_t my_kv = meta.kv_of[min(tid, SHPLB_MAX_MAPPED_HEADS / 4 - 1)];
  const int n_seq = meta.n_seq, hq = meta.n_q_heads, hkv = meta.n_kv_heads;
  const bool map = meta.kv_map != 0;
  auto scalar = [](int v) { return int(__builtin_amdgcn_readfirstlane(v)); };
  // x / y of non-negative numbers below 2^24, quotients below 2^16
  auto quotient = [](int x, int y) {
    const int q = int(float(x) * __builtin_amdgcn_rcpf(float(y))), r = x - q * y;
    return q + (r >= y ? 1 : 0) - (r < 0 ? 1 : 0);
  };
  const int group = map ? 1 : scalar(quotient(hq, hkv));      // heads of a unit, whose K/V is one stream ...
  const int units = map ? hq : hkv, n_units = n_seq * units;  // ... and how many units a sequence has, and all have
  const int n_pairs = n_seq * hq;
  const int n_streams = n_seq * hkv;
  const int mod = n_streams < kXcds ? scalar(quotient(kXcds, n_streams)) : 1;   // dies of a stream: 1, 2, 4 or 8
  const int log_mod = 31 - __builtin_clz(mod);
  if (tid <= SHPLB_MAX_SEQ) {
    s_blk[tid] = my_blk;
    s_tok[tid] = my_tok;
  }
  if (tid < SHPLB_MAX_MAPPED_HEADS / 4) s_kv[tid] = my_kv;
  if (tid < kXcds) s_total[tid] = s_halved[tid] = 0;
  if (tid == 0) {
    s_count = s_before = s_slots = s_splits = 0;
    s_cost = 0;
  }
  __syncthreads();
  auto kv_head = [&](int h) { return map ? int(s_kv[h >> 2] >> (8 * (h & 3)) & 0xff) : quotient(h, group); };
  struct Unit { int stream, nb, pair, row; };                 // (pair, row: its first)
  auto unit_of = [&](int u) {
    const int s = quotient(u, units), first = (u - s * units) * group, b0 = s_blk[s], nb = s_blk[s + 1] - b0;
    return Unit{map ? s * hkv + kv_head(first) : u, nb, s * hq + first, b0 * hq + first * nb};
  };

  // ---- pieces: what the pairs' last rows select, and the length that rows are cut at
  int len = 1 << 30;
  auto load_pairs = [&](int own_stream) {
    unsigned long long cost = 0;
    for (int p = tid; p < n_pairs; p += kPlaceThreads) {
      const int s = quotient(p, hq), h = p - s * hq, b0 = s_blk[s], nb = s_blk[s + 1] - b0, end = b0 * hq + (h + 1) * nb;
      const int k = int(min(max(sel_ptr[end] - sel_ptr[end - 1], int64_t(1)), int64_t(nb))), stream = s * hkv + kv_head(h);
      const int a = mod == 1 ? stream % kXcds : stream, b = mod == 1 ? own_stream % kXcds : own_stream;
      s_all[p] = uint32_t(k | nb << 13 | (a == b ? 0 : a < b ? 1 : 2) << 26);
      cost += uint32_t(k) * uint32_t(nb) - uint32_t(k) * uint32_t(k - 1) / 2;
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) cost += __shfl_xor(cost, d);
    if (lane == 0 && cost != 0) atomicAdd(&s_cost, cost);
    __syncthreads();
    if (kPieces) len = int(min(split_length(int64_t(s_cost), slot_capacity, n_wg, meta.block), int64_t(1 << 30)));
  };
  // f(t) for t = 0, len, 2 len .. below k: a row of more than t blocks has a piece more than one of t
  auto each_piece = [&](int k, auto&& f) {
    int t = 0;
    for (int m = 0; m < kSplitMaxPieces && t < k; ++m, t += len) f(t);
  };

  if (blockIdx.x == gridDim.x - 1) {                          // the queues' beginnings
    if constexpr (kPieces) {
      load_pairs(0);
      for (int p = tid; p < n_pairs; p += kPlaceThreads) {
        const int k = int(s_all[p] & 0x1fff), nb = int(s_all[p] >> 13 & 0x1fff), s = quotient(p, hq), stream = s * hkv + kv_head(p - s * hq);
        for (int r = 0; r < mod; ++r) {
          int n = 0;
          each_piece(k, [&](int t) { n += ((nb + mod - 1 - r) >> log_mod) - ((t + mod - 1 - r) >> log_mod); });
          atomicAdd(&s_total[mod == 1 ? stream % kXcds : stream * mod + r], n);
        }
      }
    } else for (int u = tid; u < n_units; u += kPlaceThreads) {
      const Unit e = unit_of(u);
      if (mod == 1) atomicAdd(&s_total[e.stream % kXcds], group * e.nb);
      else
        for (int r = 0; r < mod; ++r) atomicAdd(&s_total[e.stream * mod + r], group * ((e.nb + mod - 1 - r) >> log_mod));
    }
    if (!kPieces && halves) {
      // rows of more blocks than `above`, the first of every queue
      load_pairs(0);
      const int above = int(min(halved_above(int64_t(s_cost), n_wg), int64_t(SHPLB_MAX_BLOCKS)));
      for (int p = tid; p < n_pairs; p += kPlaceThreads) {
        const int k = int(s_all[p] & 0x1fff), nb = int(s_all[p] >> 13 & 0x1fff), s = quotient(p, hq), stream = s * hkv + kv_head(p - s * hq);
        for (int r = 0; k > above && r < mod; ++r)
          atomicAdd(&s_halved[mod == 1 ? stream % kXcds : stream * mod + r], ((nb + mod - 1 - r) >> log_mod) - ((above + mod - 1 - r) >> log_mod));
      }
    }
    __syncthreads();
    if (!kPieces && halves && tid < kXcds) queue_begin[kHalvedRows + tid] = s_halved[tid];
    if (tid <= kXcds) {
      int begin = 0;
      for (int x = 0; x < tid; ++x) begin += s_total[x];
      queue_begin[tid] = begin;
    }
    if (tid < kXcds) tickets[tid * kTicketStride] = uint32_t(grid - tid + kXcds - 1) / kXcds;   // see order_kernel
    return;
  }

  // ---- the workgroup's sequence, heads and rows
  int s = 0, part = int(blockIdx.x);
  if (n_seq > 1) {
    const int at = min(lane, n_seq - 1), nb = s_blk[at + 1] - s_blk[at];
    const int parts = lane < n_seq ? units * ((group * nb + kPlaceRows - 1) / kPlaceRows) : 0;
    const int end = wave_scan(parts);
    s = min(int(__builtin_popcountll(__ballot(lane < n_seq && part >= end))), n_seq - 1);
    part -= s > 0 ? __builtin_amdgcn_readlane(end, s - 1) : 0;
  }
  const int b0 = scalar(s_blk[s]), nb = scalar(s_blk[s + 1]) - b0;
  const int parts = (group * nb + kPlaceRows - 1) / kPlaceRows;
  const int unit = scalar(quotient(part, parts));
  const int at = (part - unit * parts) * kPlaceRows + tid / kPlaceLanes, e8 = tid % kPlaceLanes;
  const bool live = at < group * nb;
  const int head_in = live ? quotient(at, nb) : 0, i = live ? at - head_in * nb : 0;
  const int h = unit * group + head_in, row = b0 * hq + h * nb + i, own_pair = s * hq + h;
  const int64_t begin = sel_ptr[row], end = sel_ptr[row + 1];
  const int kv = map ? scalar(kv_head(unit)) : unit, stream = s * hkv + kv;
  const int res = i & (mod - 1);                              // the row's die is stream * mod + res, or stream % 8
  // query blocks below v whose rows are on the row's die
  auto below = [&](int v) { return (v + mod - 1 - res) >> log_mod; };

  // ---- the units of the die, and the rows of the dies before it
  int before = 0, slots = 0, splits = 0;
  for (int u0 = 0; !kPieces && u0 < n_units; u0 += kPlaceThreads) {
    const int u = u0 + tid;
    bool own = false;
    Unit e{0, 0, 0, 0};
    if (u < n_units) {
      e = unit_of(u);
      own = mod == 1 ? e.stream % kXcds == stream % kXcds : e.stream == stream;
      before += (mod == 1 ? e.stream % kXcds < stream % kXcds : e.stream < stream) ? group * e.nb : 0;
    }
    const uint64_t mask = __ballot(own);
    int first = 0;
    if (mask != 0) {
      if (lane == 0) first = atomicAdd(&s_count, __builtin_popcountll(mask));
      first = scalar(first);
    }
    if (own) {
      const int x = first + int(__builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0u)));
      s_unit[x] = uint32_t(e.pair | e.nb << 16);
      s_row[x] = e.row;
    }
  }
  if constexpr (kPieces) {
    load_pairs(stream);
    for (int p0 = 0; p0 < n_pairs; p0 += kPlaceThreads) {
      const int p = p0 + tid;
      const uint32_t e = p < n_pairs ? s_all[p] : 2u << 26;
      const int k = int(e & 0x1fff), rows = int(e >> 13 & 0x1fff);
      if (e >> 26 == 1) {
        each_piece(k, [&](int t) {
          before += rows - t;
          slots += max(t, len) < k ? rows - max(t, len) : 0;
        });
        splits += len < k ? rows - len : 0;
      }
      const uint64_t mask = __ballot(e >> 26 == 0);
      int first = 0;
      if (mask != 0) {
        if (lane == 0) first = atomicAdd(&s_count, __builtin_popcountll(mask));
        first = scalar(first);
      }
      if (e >> 26 == 0) {
        const int x = first + int(__builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0u)));
        s_pair[x] = uint32_t(p | rows << 16);
        s_k[x] = k;
      }
    }
    slots = wave_scan(slots);
    splits = wave_scan(splits);
    if (lane == 63 && splits != 0) {
      atomicAdd(&s_slots, slots);
      atomicAdd(&s_splits, splits);
    }
  }
  before = wave_scan(before);
  if (lane == 63 && before != 0) atomicAdd(&s_before, before);
  const int n_sel = int(min(max(end - begin, int64_t(0)), int64_t(kCostBins - 1)));
  const int first_j = n_sel > 0 ? sel_idx[begin] : 0, second_j = n_sel > 0 ? sel_idx[begin + min(1, n_sel - 1)] : 0;
  __syncthreads();
  const int n_own = kPieces ? s_count : s_count * group;
  for (int x = tid; !kPieces && x < n_own; x += kPlaceThreads) {
    const int u = quotient(x, group), head = x - u * group, rows = int(s_unit[u] >> 16);
    const int end = s_row[u] + (head + 1) * rows;
    s_pair[x] = s_unit[u] + head;
    s_k[x] = int(min(max(sel_ptr[end] - sel_ptr[end - 1], int64_t(1)), int64_t(rows)));
  }
  __syncthreads();

  // ---- the row's place
  const int own_end = b0 * hq + (h + 1) * nb;
  const int k = int(min(max(sel_ptr[own_end] - sel_ptr[own_end - 1], int64_t(1)), int64_t(nb)));
  const int c = min(k, i + 1), below_c = below(c), at_c = below_c - below(c - 1);
  // rows of the same stream's dies before this one: those of the first v query blocks
  auto earlier = [&](int v) { return (v >> log_mod) * res + min(v & (mod - 1), res); };
  const int pieces = kPieces ? pieces_of(c, len) : 1;
  int place = 0;                              // items in front of the row, on this die and those before
  int slot = 0, entry = 0;                    // its first slot and its counter: split rows are the first of a queue
  for (int x = e8; x < n_own; x += kPlaceLanes) {
    const int p = int(s_pair[x] & 0xffff), rows = int(s_pair[x] >> 16), k_p = s_k[x], all = below(rows);
    const int same = p < own_pair ? (c < k_p ? at_c : c == k_p ? all - below_c + at_c : 0) : p == own_pair && c == k_p ? below(i) - below(k_p - 1) : 0;
    if constexpr (kPieces) {
      each_piece(k_p, [&](int t) {
        place += earlier(rows) - earlier(t);
        if (max(t, len) < k_p) slot += earlier(rows) - earlier(max(t, len));
        if (max(t, c) < k_p) {
          place += all - below(max(t, c));
          slot += all - below(max(t, c));
        }
      });
      if (len < k_p) entry += earlier(rows) - earlier(len);
      place += pieces * same;
      slot += pieces * same;
      entry += (c < k_p ? all - below_c : 0) + same;
    } else {
      place += earlier(rows) + (c < k_p ? all - below_c : 0) + same;
    }
  }
  auto of_row = [](int v) {
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    return v + __shfl_xor(v, 4);
  };
  place = of_row(place) + s_before;
  if constexpr (kPieces) {
    slot = of_row(slot) + s_slots;
    entry = of_row(entry) + s_splits;
  }
  if (!live || uint32_t(place) + uint32_t(pieces) > uint32_t(item_capacity)) return;      // (the latter never: keeps stores in bounds)
  if constexpr (kPieces) {
    if (pieces > 1) {
      // A row that is not its budget's may have fewer blocks than pieces are reserved for it: the others are items without a block.
      const int real = min(pieces, n_sel);
      if (slot + pieces > slot_capacity || entry >= slot_capacity / 2 + 1) return;        // likewise
      if (e8 == 0) split_done[entry] = 0;
      for (int x = 0; x < pieces; ++x) {
        const int64_t from = x < real ? piece_begin(n_sel, real, x) : 0, to = x < real ? piece_begin(n_sel, real, x + 1) : 0;
        const int n = int(to - from);
        const int64_t at = begin + from;
        int lo = 0, hi = n;
        if (e8 == 1) lo = int(uint32_t(at)), hi = int(at >> 32);
        if (e8 == 2) lo = real > 1 ? slot + x : -1, hi = max(real, 1);                    // slot, pieces
        if (e8 == 3) lo = real > 1 ? slot : -1, hi = real > 1 ? entry : -1;               // first_slot, split_index
        if (e8 == 4) lo = s_tok[s], hi = s_tok[s + 1];
        if (e8 == 5) lo = h, hi = kv;
        if (e8 == 6) lo = i, hi = nb;
        if (e8 == 7 && n > 0) lo = sel_idx[at], hi = sel_idx[at + min(1, n - 1)];
        reinterpret_cast<int2*>(items + place + x)[e8] = int2{lo, hi};
      }
      return;
    }
  }
  // a lane's two words of the record
  int lo = 0, hi = n_sel;
  if (e8 == 1) lo = int(uint32_t(begin)), hi = int(begin >> 32);
  if (e8 == 2) lo = -1, hi = 1;                                         // slot, pieces
  if (e8 == 3) lo = hi = -1;                                            // first_slot, split_index
  if (e8 == 4) lo = s_tok[s], hi = s_tok[s + 1];
  if (e8 == 5) lo = h, hi = kv;
  if (e8 == 6) lo = i, hi = nb;
  if (e8 == 7) lo = first_j, hi = second_j;
  reinterpret_cast<int2*>(items + place)[e8] = int2{lo, hi};
}

}  // namespace

int32_t launch_order(const Geometry& g, const int64_t* sel_ptr, const int32_t* sel_idx, const WorkspaceLayout& w,
                     char* workspace, int32_t n_wg, int32_t grid, bool halves, hipStream_t stream) {
  const SeqMeta& m = g.meta;
  if (int64_t(m.n_seq) * m.n_q_heads <= kPlacePairs) {
    const int units = m.kv_map ? m.n_q_heads : m.n_kv_heads, group = m.n_q_heads / units;
    int64_t parts = 0;
    for (int s = 0; s < m.n_seq; ++s)
      parts += units * ((int64_t(group) * (m.blk_begin[s + 1] - m.blk_begin[s]) + kPlaceRows - 1) / kPlaceRows);
    hipLaunchKernelGGL(w.slot_capacity >= 2 ? place_kernel<true> : place_kernel<false>, dim3(uint32_t(parts + 1)), dim3(kPlaceThreads), 0,
                       stream, m, sel_ptr, sel_idx, reinterpret_cast<ItemRec*>(workspace + w.items),
                       reinterpret_cast<int32_t*>(workspace + w.queue_begin), reinterpret_cast<uint32_t*>(workspace + w.tickets),
                       reinterpret_cast<uint32_t*>(workspace + w.split_done), int(w.item_capacity), int(w.slot_capacity), n_wg, grid, int(halves));
    return hipGetLastError() == hipSuccess ? SHPLB_OK : SHPLB_E_HIP;
  }
  hipLaunchKernelGGL(order_kernel, dim3(kXcds), dim3(kOrderThreads), 0, stream, g.meta, sel_ptr, sel_idx,
                     reinterpret_cast<ItemRec*>(workspace + w.items),
                     reinterpret_cast<int32_t*>(workspace + w.queue_begin),
                     reinterpret_cast<uint32_t*>(workspace + w.tickets),
                     reinterpret_cast<uint32_t*>(workspace + w.split_done), int(g.rows),
                     min(g.max_nb + 1, kCostBins), int(w.item_capacity), int(w.slot_capacity), n_wg, grid);
  if (hipGetLastError() != hipSuccess) return SHPLB_E_HIP;
  return SHPLB_OK;
}

}  // namespace shplb
