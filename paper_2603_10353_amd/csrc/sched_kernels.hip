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
// Launches of up to 65536 rows (16384 where rows may be cut) and 2048 (sequence, head) pairs find their places without a sort: see
// place_kernel.  Larger ones go through one launch of eight workgroups (order_kernel); workgroup x builds the queue of die x with a counting sort
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
// last combines them (count_piece() and merge_row() in attn_common.h).  Which slots and counter
// entries a row gets depends on the kernel and, in order_kernel, on arrival; what is computed does not.
//
// Launches that cut no row (through the splitting entry point too, where all are short) and have no more rows than workgroups skip all
// this: see row_place() in attn_pipe_kernel.hip.
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

// The queues without a sort: every row counts the rows in front of it in its queue, those of its die that select more blocks, and of those
// that select as many the ones before it.
//
// A workgroup takes 64 consecutive rows of one die and one stream (the heads of one KV head of one sequence; with a caller's map of
// heads, of one head).  It goes through all rows of the die and counts them per number of selected blocks, in LDS, and apart those
// in front of its own 64; a sum over the bins from the longest rows on, and its rows' places are known.  All workgroups of a die
// count the same, so none waits for another one.  A row has eight lanes, which write its record together.  An extra workgroup at the
// end writes the queues' beginnings and tickets, and with `halves` how many rows of each queue are worked on in halves (the
// longest ones, so the first; see in_halves() and worth_halves()).
//
// Pieces (kPieces): a row is cut into pieces_of() its own number of blocks, and the items in front of it are the pieces of the rows
// in front.  Items of the dies before come first: their rows follow from the shapes, and all rows of the launch are looked at for those that are cut.
// Split rows are the first of their queues, so slots and counters are numbered like items and rows, behind those of the dies before.
//
// What bounds it is the chain arguments -> row pointers -> first blocks, on as many compute units as there are rows for, with code that is not in
// the instruction cache.  Every workgroup reads the row pointers of its die (with pieces of all rows), rows / 64 times in all: that is why
// larger launches are sorted (places_counted()).  Under the tracer, order_kernel against this: 8K prompt x 32 heads 9.7 -> 5.5 us, 48
// sequences x 28 heads 10.2 -> 5.8, 32K x 32 heads 12.0 -> 6.5, 128K 26 -> 10.2, 16K in pieces 18 -> 9.2.  (Workgroups of 256 threads take
// 1 to 5 us longer, of 1024 as long or up to 1 us longer.  With the dies of all rows worked out, not only of the long ones, the extra workgroup took
// 6.6 at 8K and the pieces 12.4; four rows in flight, and so twice the code, 0.4 longer.)  Counted in closed form from what the last row of
// every head selects it took 5.3, 6.7, 5.7, 7.3 and 6.8 us, but then a list that is no budget's, say a different number of blocks for every query
// block, is neither ordered nor cut by its length: attention call of 8231 tokens x 32/8 heads with such lists 176 us, ordered 148.
constexpr int kPlaceThreads = 512, kPlaceLanes = 8, kPlaceRows = kPlaceThreads / kPlaceLanes, kPlaceWaves = kPlaceThreads / 64;
constexpr int kPlaceInFlight = 2;         // rows a thread has in flight

template <bool kPieces>
__global__ __launch_bounds__(kPlaceThreads) void place_kernel(
    SeqMeta meta, const int64_t* __restrict__ sel_ptr, const int32_t* __restrict__ sel_idx,
    ItemRec* __restrict__ items, int32_t* __restrict__ queue_begin, uint32_t* __restrict__ tickets, uint32_t* __restrict__ split_done,
    int rows, int n_bins, int item_capacity, int slot_capacity, int n_wg, int grid, int halves) {
  // per number of selected blocks the rows of the die, later those with more blocks | those in front of the workgroup's own << 32;
  // pieces: behind them the items of the rows with more blocks (int32)
  extern __shared__ unsigned long long s_bins[];
  __shared__ int32_t s_blk[SHPLB_MAX_SEQ + 1], s_tok[SHPLB_MAX_SEQ + 1];
  __shared__ uint32_t s_kv[SHPLB_MAX_MAPPED_HEADS / 4];
  __shared__ int32_t s_pre[kPlacePairs];     // listed units: listed rows before its own ...
  __shared__ int32_t s_row[kPlacePairs];     // ... first row ...
  __shared__ int32_t s_nb[kPlacePairs];      // ... blocks (streams on several dies)
  __shared__ int32_t s_listed;               // rows listed | units listed << 20
  __shared__ int32_t s_before, s_slots, s_splits;   // items, slots and split rows on the dies before
  __shared__ int32_t s_total[kXcds], s_halved[kXcds], s_longest, s_wave[2][kPlaceWaves], s_n[kPlaceRows];
  static_assert(SHPLB_MAX_SEQ < kPlaceThreads && SHPLB_MAX_BLOCKS < 1 << 16 && kPlaceCounted < 1 << 20 && kPlacePairs < 1 << 12, "");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // asked for together: the geometry, of which a lane-dependent index is read
  const int my_blk = meta.blk_begin[min(tid, SHPLB_MAX_SEQ)], my_tok = meta.tok_begin[min(tid, SHPLB_MAX_SEQ)];
  const uint32_t my_kv = meta.kv_of[min(tid, SHPLB_MAX_MAPPED_HEADS / 4 - 1)];
  const int64_t first_sel = sel_ptr[0], end_sel = sel_ptr[rows];
  const int n_seq = meta.n_seq, hq = meta.n_q_heads, hkv = meta.n_kv_heads;
  const bool map = meta.kv_map != 0;
  auto scalar = [](int v) { return int(__builtin_amdgcn_readfirstlane(v)); };
  // x / y of non-negative numbers, x below 2^25, quotients below 2^16
  auto quotient = [](int x, int y) {
    const int q = int(float(x) * __builtin_amdgcn_rcpf(float(y))), r = x - q * y;
    return q + (r >= y ? 1 : 0) - (r < 0 ? 1 : 0);
  };
  const int group = map ? 1 : scalar(quotient(hq, hkv));      // heads of a unit, whose K/V is one stream ...
  const int units = map ? hq : hkv, n_units = n_seq * units;  // ... and how many units a sequence has, and all have
  const int n_streams = n_seq * hkv;
  const int mod = n_streams < kXcds ? scalar(quotient(kXcds, n_streams)) : 1;   // dies of a stream: 1, 2, 4 or 8
  const int log_mod = 31 - __builtin_clz(mod);
  const int top_seq = n_seq > 1 ? 1 << (31 - __builtin_clz(n_seq - 1)) : 0;
  if (tid <= SHPLB_MAX_SEQ) {
    s_blk[tid] = my_blk;
    s_tok[tid] = my_tok;
  }
  if (tid < SHPLB_MAX_MAPPED_HEADS / 4) s_kv[tid] = my_kv;
  if (tid < kXcds) s_total[tid] = s_halved[tid] = 0;
  if (tid == 0) s_listed = s_before = s_slots = s_splits = s_longest = 0;
  for (int b = tid; b < n_bins; b += kPlaceThreads) s_bins[b] = 0;
  __syncthreads();
  auto kv_head = [&](int h) { return map ? int(s_kv[h >> 2] >> (8 * (h & 3)) & 0xff) : quotient(h, group); };
  struct Unit { int stream, nb, row; };                       // (row: its first)
  auto unit_of = [&](int u) {
    const int s = quotient(u, units), first = (u - s * units) * group, b0 = s_blk[s], nb = s_blk[s + 1] - b0;
    return Unit{map ? s * hkv + kv_head(first) : u, nb, b0 * hq + first * nb};
  };
  // The die of query block i of a stream is (stream << log_mod) + (i & (mod - 1)), or stream % 8: first_die() + the block's residue.
  auto first_die = [&](int stream) { return mod == 1 ? stream % kXcds : stream << log_mod; };
  // Query blocks of nb with residue r, and with one below r (r: 0 .. mod).
  auto with_residue = [&](int nb, int r) { return (nb + mod - 1 - r) >> log_mod; };
  auto below_residue = [&](int nb, int r) { return (nb >> log_mod) * r + min(nb & (mod - 1), r); };

  // List the units that have rows on `die`, in any order.  Returns a thread's sum of the rows on the dies before.
  auto list_units = [&](int die) {
    int before = 0;
    for (int u0 = 0; u0 < n_units; u0 += kPlaceThreads) {
      const int u = u0 + tid;
      Unit e{0, 0, 0};
      int n = 0;
      if (u < n_units) {
        e = unit_of(u);
        const int r = die - first_die(e.stream);              // the residue that lives on the die, if it is one
        n = r >= 0 && r < mod ? group * with_residue(e.nb, r) : 0;
        before += group * below_residue(e.nb, min(max(r, 0), mod));
      }
      const uint32_t own = n > 0 ? uint32_t(n) | 1u << 20 : 0u;
      const uint32_t to = uint32_t(wave_scan(int(own)));
      uint32_t at = 0;
      if (lane == 63 && to != 0) at = uint32_t(atomicAdd(&s_listed, int(to)));
      at = uint32_t(__builtin_amdgcn_readlane(int(at), 63)) + to - own;
      if (n > 0) {
        s_pre[at >> 20] = int(at & 0xfffff);
        s_row[at >> 20] = e.row;
        if (mod > 1) s_nb[at >> 20] = e.nb;
      }
    }
    return before;
  };
  // f(row, blocks it selects, whether there is a row) for the listed rows, of residue `res`, by whole waves
  auto each_row = [&](int res, auto&& f) {
    const int n_rows = s_listed & 0xfffff, n_list = int(uint32_t(s_listed) >> 20);
    const int top = n_list > 1 ? 1 << (31 - __builtin_clz(n_list - 1)) : 0;
    for (int r0 = 0; r0 < n_rows; r0 += kPlaceInFlight * kPlaceThreads) {
      int row[kPlaceInFlight];
      int64_t begin[kPlaceInFlight], end[kPlaceInFlight];
#pragma unroll
      for (int u = 0; u < kPlaceInFlight; ++u) {
        row[u] = -1;
        if (r0 + u * kPlaceThreads >= n_rows) continue;       // (the same for all)
        const int r = r0 + u * kPlaceThreads + tid;
        int x = 0;
        for (int d = top; d > 0; d >>= 1)
          if (x + d < n_list && s_pre[x + d] <= r) x += d;
        int at = r - s_pre[x];
        if (mod > 1) {
          const int nb = s_nb[x], per_head = with_residue(nb, res), h = quotient(at, per_head);
          at = h * nb + ((at - h * per_head) << log_mod) + res;
        }
        if (r < n_rows) row[u] = s_row[x] + at;
        begin[u] = sel_ptr[max(row[u], 0)];
        end[u] = sel_ptr[max(row[u], 0) + 1];
      }
#pragma unroll
      for (int u = 0; u < kPlaceInFlight; ++u)
        if (r0 + u * kPlaceThreads < n_rows)
          f(row[u], int(min(max(end[u] - begin[u], int64_t(0)), int64_t(n_bins - 1))), row[u] >= 0);
    }
  };
  // f(die, blocks it selects) for every row of the launch for which is_long(blocks) holds.  (Only those are decoded.)
  auto each_long = [&](auto&& is_long, auto&& f) {
    constexpr int kRun = 8;
    for (int r0 = 0; r0 < rows; r0 += kRun * kPlaceThreads) {
      int n[kRun];
      uint32_t found = 0;
#pragma unroll
      for (int u = 0; u < kRun; ++u) {
        const int at = min(r0 + u * kPlaceThreads + tid, rows - 1);
        n[u] = int(min(max(sel_ptr[at + 1] - sel_ptr[at], int64_t(0)), int64_t(n_bins - 1)));
      }
#pragma unroll
      for (int u = 0; u < kRun; ++u) found |= r0 + u * kPlaceThreads + tid < rows && is_long(n[u]) ? 1u << u : 0u;
      for (; found != 0; found &= found - 1) {
        const int u = __builtin_ctz(found), r = r0 + u * kPlaceThreads + tid;
        int n_u = n[0], of = 0;
#pragma unroll
        for (int x = 1; x < kRun; ++x) n_u = u == x ? n[x] : n_u;
        for (int d = top_seq; d > 0; d >>= 1)
          if (of + d < n_seq && s_blk[of + d] * hq <= r) of += d;
        const int nb = s_blk[of + 1] - s_blk[of], local = r - s_blk[of] * hq, h = quotient(local, nb);
        f(first_die(of * hkv + kv_head(h)) + ((local - h * nb) & (mod - 1)), n_u);
      }
    }
  };
  const int len = kPieces ? int(min(split_length(end_sel - first_sel, slot_capacity, n_wg, meta.block), int64_t(1 << 24))) : 0;
  auto pieces_here = [&](int n) { return !kPieces || n <= len ? 1 : min(quotient(n + len - 1, len), kSplitMaxPieces); };   // pieces_of()

  const bool extra = blockIdx.x == gridDim.x - 1;             // writes the queues' beginnings, and has no rows

  // ---- the workgroup's sequence, heads and rows
  auto parts_of = [&](int nb) { return (group * with_residue(nb, 0) + kPlaceRows - 1) / kPlaceRows << log_mod; };   // of a unit: of every residue as many
  int s = 0, part = extra ? 0 : int(blockIdx.x);
  if (n_seq > 1) {
    const int at = min(lane, n_seq - 1), nb = s_blk[at + 1] - s_blk[at];
    const int end = wave_scan(lane < n_seq ? units * parts_of(nb) : 0);
    s = min(int(__builtin_popcountll(__ballot(lane < n_seq && part >= end))), n_seq - 1);
    part -= s > 0 ? __builtin_amdgcn_readlane(end, s - 1) : 0;
  }
  const int b0 = scalar(s_blk[s]), nb = scalar(s_blk[s + 1]) - b0;
  const int parts = parts_of(nb), unit = scalar(quotient(part, parts));
  part -= unit * parts;
  const int res = part & (mod - 1), per_head = with_residue(nb, res), n_unit = group * per_head;   // rows of the unit on the die
  const int first = (part >> log_mod) * kPlaceRows;
  if (!extra && first >= n_unit) return;
  const int kv = map ? scalar(kv_head(unit)) : unit, die = first_die(s * hkv + kv) + res;
  auto head_of = [&](int at) { return quotient(at, per_head); };
  const int first_head = head_of(first), first_row = b0 * hq + (unit * group + first_head) * nb + ((first - first_head * per_head) << log_mod) + res;
  const int slot_row = tid / kPlaceLanes, at = first + slot_row, e8 = tid % kPlaceLanes;
  const bool live = at < n_unit;
  const int head_in = live ? head_of(at) : first_head, i = live ? ((at - head_in * per_head) << log_mod) + res : res;
  const int h = unit * group + head_in, row = b0 * hq + h * nb + i;
  const int64_t begin = sel_ptr[row], end = sel_ptr[row + 1];

  // ---- count
  int before = 0, slots = 0, splits = 0;
  if (!extra) before = list_units(die);
  const int n_sel = int(min(max(end - begin, int64_t(0)), int64_t(kCostBins - 1))), key = min(n_sel, n_bins - 1);
  const int first_j = n_sel > 0 ? sel_idx[begin] : 0, second_j = n_sel > 0 ? sel_idx[begin + min(1, n_sel - 1)] : 0;
  __syncthreads();
  // Pieces: every row is an item and rows of more than `len` blocks are more than one, of which the dies before matter
  if constexpr (kPieces)
    each_long([&](int n) { return n > len; }, [&](int of, int n) {
      const int pieces = pieces_here(n);
      if (extra) {
        atomicAdd(&s_total[of], pieces - 1);
      } else if (of < die) {
        before += pieces - 1;
        slots += pieces;
        splits += 1;
      }
    });
  each_row(res, [&](int r, int n, bool active) {
    // rows of a wave are mostly neighbours of one head: two bins are counted by ballot, the rest lane by lane (see take_places())
    const uint64_t front = __ballot(r < first_row);
#pragma unroll
    for (int round = 0; round < 2; ++round) {
      const uint64_t open = __ballot(active);
      if (open == 0) break;
      const int lead = round == 0 ? 63 - __builtin_clzll(open) : __builtin_ctzll(open);
      const int b = __builtin_amdgcn_readlane(n, lead);
      const uint64_t same = __ballot(active && n == b);
      if (lane == lead)
        atomicAdd(&s_bins[b], (unsigned long long)(__builtin_popcountll(same)) | (unsigned long long)(__builtin_popcountll(same & front)) << 32);
      if (n == b) active = false;
    }
    if (active) atomicAdd(&s_bins[n], r < first_row ? 1ull | 1ull << 32 : 1ull);
  });
  if (extra) {
    if (!kPieces && halves)
      each_long([&](int n) { return in_halves(n, end_sel - first_sel, n_wg); }, [&](int of, int n) {
        atomicAdd(&s_halved[of], 1);
        atomicMax(&s_longest, n);
      });
    for (int u = tid; u < n_units; u += kPlaceThreads) {
      const Unit e = unit_of(u);
      for (int r = 0; r < mod; ++r) atomicAdd(&s_total[first_die(e.stream) + r], group * with_residue(e.nb, r));
    }
    __syncthreads();
    if (!kPieces && halves && tid < kXcds) queue_begin[kHalvedRows + tid] = worth_halves(s_longest, end_sel - first_sel, n_wg) ? s_halved[tid] : 0;
    if (tid <= kXcds) {
      int begin = 0;
      for (int x = 0; x < tid; ++x) begin += s_total[x];
      queue_begin[tid] = begin;
    }
    if (tid < kXcds) tickets[tid * kTicketStride] = uint32_t(grid - tid + kXcds - 1) / kXcds;   // see order_kernel
    return;
  }
  auto add_up = [&](int v, int32_t* sum) {
    v = wave_scan(v);
    if (lane == 63 && v != 0) atomicAdd(sum, v);
  };
  add_up(before, &s_before);
  if constexpr (kPieces) {
    add_up(slots, &s_slots);
    add_up(splits, &s_splits);
  }
  if (e8 == 0) s_n[slot_row] = live ? key : -1;
  __syncthreads();

  // ---- rows (and items) with more blocks, a thread owns a run of bins
  int32_t* const s_items = reinterpret_cast<int32_t*>(s_bins + n_bins);
  const int per = (n_bins + kPlaceThreads - 1) / kPlaceThreads;
  const int k0 = min(tid * per, n_bins), k1 = min(k0 + per, n_bins);
  int more = 0, more_items = 0;
  for (int k = k0; k < k1; ++k) {
    const int c = int(uint32_t(s_bins[n_bins - 1 - k]));
    more += c;
    if constexpr (kPieces) more_items += c * pieces_here(n_bins - 1 - k);
  }
  const int more_inc = wave_scan(more), items_inc = kPieces ? wave_scan(more_items) : 0;
  if (lane == 63) {
    s_wave[0][wave] = more_inc;
    s_wave[1][wave] = items_inc;
  }
  __syncthreads();
  auto waves_before = [&](const int32_t (&sums)[kPlaceWaves]) {
    const int to = wave_scan(lane < kPlaceWaves ? sums[lane] : 0);
    return wave > 0 ? __builtin_amdgcn_readlane(to, wave - 1) : 0;
  };
  more = more_inc - more + waves_before(s_wave[0]);
  if constexpr (kPieces) more_items = items_inc - more_items + waves_before(s_wave[1]);
  for (int k = k0; k < k1; ++k) {
    const int b = n_bins - 1 - k, c = int(uint32_t(s_bins[b]));
    s_bins[b] = (s_bins[b] >> 32 << 32) | uint32_t(more);
    more += c;
    if constexpr (kPieces) {
      s_items[b] = more_items;
      more_items += c * pieces_here(b);
    }
  }
  __syncthreads();

  // ---- the row's place
  int same = 0;                                               // rows of the workgroup in front with as many blocks
#pragma unroll
  for (int x = e8; x < kPlaceRows; x += kPlaceLanes) same += x < slot_row && s_n[x] == key;
  same += __shfl_xor(same, 1);
  same += __shfl_xor(same, 2);
  same += __shfl_xor(same, 4);
  same += int(s_bins[key] >> 32);
  const int rows_above = int(uint32_t(s_bins[key])), items_above = kPieces ? s_items[key] : rows_above;
  const int pieces = pieces_here(key);
  const int place = s_before + items_above + pieces * same;
  if (!live || uint32_t(place) + uint32_t(pieces) > uint32_t(item_capacity)) return;      // (the latter never: keeps stores in bounds)
  if constexpr (kPieces) {
    if (pieces > 1) {
      const int slot = s_slots + items_above + pieces * same, entry = s_splits + rows_above + same;   // split rows are the first of a queue
      if (slot + pieces > slot_capacity || entry >= slot_capacity / 2 + 1) return;        // likewise
      if (e8 == 0) split_done[entry] = 0;
      for (int x = 0; x < pieces; ++x) {
        const int64_t from = piece_begin(n_sel, pieces, x), from_sel = begin + from;
        const int n = int(piece_begin(n_sel, pieces, x + 1) - from);
        int lo = 0, hi = n;
        if (e8 == 1) lo = int(uint32_t(from_sel)), hi = int(from_sel >> 32);
        if (e8 == 2) lo = slot + x, hi = pieces;                        // slot, pieces
        if (e8 == 3) lo = slot, hi = entry;                             // first_slot, split_index
        if (e8 == 4) lo = s_tok[s], hi = s_tok[s + 1];
        if (e8 == 5) lo = h, hi = kv;
        if (e8 == 6) lo = i, hi = nb;
        if (e8 == 7) lo = sel_idx[from_sel], hi = sel_idx[from_sel + min(1, n - 1)];
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
  const bool pieces = w.slot_capacity >= 2;
  if (places_counted(g, pieces)) {
    const int units = m.kv_map ? m.n_q_heads : m.n_kv_heads, group = m.n_q_heads / units, n_streams = m.n_seq * m.n_kv_heads;
    const int mod = n_streams < kXcds ? kXcds / n_streams : 1;          // dies of a stream
    int64_t parts = 0;
    for (int s = 0; s < m.n_seq; ++s) {
      const int64_t per_head = (m.blk_begin[s + 1] - m.blk_begin[s] + mod - 1) / mod;   // rows of a head on a die, at most
      parts += units * mod * ((group * per_head + kPlaceRows - 1) / kPlaceRows);
    }
    hipLaunchKernelGGL(pieces ? place_kernel<true> : place_kernel<false>, dim3(uint32_t(parts + 1)), dim3(kPlaceThreads),
                       (g.max_nb + 1) * (pieces ? 12 : 8), stream, m, sel_ptr, sel_idx, reinterpret_cast<ItemRec*>(workspace + w.items),
                       reinterpret_cast<int32_t*>(workspace + w.queue_begin), reinterpret_cast<uint32_t*>(workspace + w.tickets),
                       reinterpret_cast<uint32_t*>(workspace + w.split_done), int(g.rows), int(g.max_nb + 1), int(w.item_capacity),
                       int(w.slot_capacity), n_wg, grid, int(halves));
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
