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
// One launch of eight workgroups; workgroup x builds the queue of die x with a counting sort
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
// What bounds it: a chain of dependent memory round trips (geometry, row pointer, first
// selected blocks, record) on eight compute units.  A thread works out one (sequence, head)
// pair, a prefix sum over the pairs lies in LDS, and threads then find their rows in it by
// bisection: nothing loops over sequences and no lane is idle when sequences are short.
// 8.1 us at 2080 rows (one 8K prompt, 32 heads), 9.2 us for 3668 rows in 48 sequences, 15.4 us at
// 16384, 26 us at 32768.  Before, one workgroup sorted launches of up to 16384 rows and five dependent
// launches the larger ones, decoding every row (a loop over the sequences and two integer divisions)
// twice: 8.8, 41.8, 37.8 and 38 us.
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
  bool fetched = false;                              // all rows of the die are in the threads' registers
  for (int base = 0; base < n_pairs; base += kBatch) {
    if (base > 0) __syncthreads();
    n_rows = load_batch(base, split, begin);
    fetched = !split && n_pairs <= kBatch && n_rows <= kInFlight * kOrderThreads;
    for (int r0 = tid; r0 - tid < n_rows; r0 += kInFlight * kOrderThreads) {
      fetch(r0, n_rows, fetched);
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
    if (split || n_pairs > kBatch) {                 // else the batch is still laid out
      int unused = 0;
      if (base > 0) __syncthreads();
      n_rows = load_batch(base, false, unused);
    }
    for (int r0 = tid; r0 - tid < n_rows; r0 += kInFlight * kOrderThreads) {
      if (!fetched) fetch(r0, n_rows, true);
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

}  // namespace

int32_t launch_order(const Geometry& g, const int64_t* sel_ptr, const int32_t* sel_idx, const WorkspaceLayout& w,
                     char* workspace, int32_t n_wg, int32_t grid, hipStream_t stream) {
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
