// Internal declarations shared by the translation units of libshplb (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "shplb.h"

namespace shplb {

constexpr int kHeadDim = 128;
constexpr int kCostBins = 4100;       // selected-block counts 0..SHPLB_MAX_BLOCKS, rounded up
constexpr int kXcds = 8;              // accelerator dies (XCDs) of an MI355X, each with its own L2
constexpr int kTicketStride = 16;     // uint32 slots between two queue tickets (one 64-byte line each)
constexpr int kSplitSlotsMax = 1 << 16;   // most partial-result slots a caller may ask for (64 KB + 1 KB each)
constexpr int kSplitMinTiles = 32;    // a piece of a split row covers at least this many 64-key tiles: a piece costs
                                      // about 7 us more than it computes for (write-through stores of its partial
                                      // result, the count) and a merge 12-15 us; 32 tiles are about 50 us of work
constexpr int kSplitShare = 2;        // rows longer than 1/kSplitShare of a workgroup's average share are split
constexpr int64_t kSlotFloatsO = 128 * kHeadDim;   // one partial result: unnormalised O of up to 128 queries ...
constexpr int64_t kSlotFloatsML = 2 * 128;         // ... and their reference exponent and denominator

// Sequence geometry, passed to kernels by value (about 1 KB of kernel arguments).
struct SeqMeta {
  int32_t n_seq;
  int32_t n_q_heads;
  int32_t n_kv_heads;
  int32_t block;
  int32_t tok_begin[SHPLB_MAX_SEQ + 1];   // cu_seqlens
  int32_t blk_begin[SHPLB_MAX_SEQ + 1];   // cumulative block counts
  int64_t score_off[SHPLB_MAX_SEQ + 1];   // float offset of each sequence's score cube
  int32_t kv_map;                         // 1: kv_of[] holds the KV head of every query head
  uint32_t kv_of[SHPLB_MAX_MAPPED_HEADS / 4];   // one byte per query head, four to a word
};

struct Strides {
  int64_t q_t, q_h, kv_t, kv_h;
};

// Validated, host-side view of a shplb_problem.
struct Geometry {
  SeqMeta meta;
  Strides st;
  int64_t total_tokens;
  int64_t total_blocks;
  int64_t rows;
  int32_t max_nb;
  float scale;
};

// Workspace carve-up (byte offsets, each 256-byte aligned).
struct WorkspaceLayout {
  int64_t qbar, kbar;        // pooled blocks as three bf16 planes, each [H][total_blocks][128]
  int64_t items;             // ItemRec [item_capacity]: the work items, one queue per XCD after the other
  int64_t split_done;        // uint32 [slot_capacity / 2 + 1]: pieces finished, per split row
  int64_t part_o;            // float [slot_capacity][128][kHeadDim]: partial results of the pieces
  int64_t part_ml;           // float [slot_capacity][2][128]
  int64_t item_capacity, slot_capacity;   // counts, not offsets
  int64_t queue_begin;       // int32 [kXcds + 1]: queue x is items[queue_begin[x] .. queue_begin[x+1]); from kHalvedRows on [kXcds] more
  int64_t tickets;           // uint32 [kXcds * kTicketStride]
  int64_t total;
};

int32_t make_geometry(const shplb_problem* p, Geometry* g);
// split_slots: partial-result slots for rows split along the keys (0: rows stay whole)
// with_pooled = false leaves out the pooled planes (the attention step alone does not use them)
WorkspaceLayout make_layout(const Geometry& g, int32_t split_slots = 0, bool with_pooled = true);
// Persistent workgroups of an attention launch on the current device: as many as fit at two waves
// per SIMD (two per compute unit with 128-token blocks, four with 64); <0 on HIP error.
int32_t persistent_workgroups(int block = 128);

// Kernel launchers (each returns a SHPLB status).
int32_t launch_pool_scores(const Geometry& g, const void* q, const void* k, float* scores,
                           uint16_t* q_planes, uint16_t* k_planes, int n_compute_units, hipStream_t stream);
int32_t launch_select(const Geometry& g, const float* scores, const int64_t* sel_ptr,
                      int32_t* sel_idx, hipStream_t stream);
int32_t launch_order(const Geometry& g, const int64_t* sel_ptr, const int32_t* sel_idx, const WorkspaceLayout& w,
                     char* workspace, int32_t n_wg, int32_t grid, bool halves, hipStream_t stream);
int32_t launch_mfma_rate(int random_operands, int iters, int n_workgroups, void* scratch, hipStream_t stream);
int32_t launch_block_mass(const Geometry& g, const void* q, const void* k, float* mass, hipStream_t stream);
int32_t launch_token_recovery(const Geometry& g, const void* q, const void* k, const int32_t* budgets,
                              int32_t n_budgets, float* recovery, hipStream_t stream);
// One work item of an attention launch: a row, or one piece of a row that was split along
// its selected key blocks (positions [first, first + n_sel) of the row's selection).  It carries
// everything a workgroup needs to start: sixteen words, one vector load of a word per lane (read_record()).
struct alignas(64) ItemRec {
  int32_t unused;
  int32_t n_sel;        // selected key blocks this item covers
  int64_t sel_begin;    // index of its first one in sel_idx
  int32_t slot;         // partial-result slot it writes, or -1: the item is the whole row and writes the output
  int32_t pieces;       // pieces of its row (1: whole row)
  int32_t first_slot;   // slot of the row's first piece; the row's pieces hold slots first_slot .. + pieces - 1
  int32_t split_index;  // the row's entry in the finished-pieces counters
  int32_t seq_begin, seq_end;         // tokens of the row's sequence
  int32_t head, kv_head, query_block;
  int32_t n_blocks;                   // blocks of the sequence
  int32_t first_block, second_block;  // the item's first two selected blocks (the same one twice if it has one)
};

// Longest item, in key blocks, of a launch whose rows select total_cost blocks in all, run by
// n_wg persistent workgroups, with room for slot_capacity partial results (0: never split).
// Rows longer than this are cut into near-equal pieces, so that no single item is a large
// part of a workgroup's average share (total / n_wg) and a launch of few rows still fills the
// chip.  Three lower bounds: a piece covers at least kSplitMinTiles key tiles (an item's fixed
// cost must stay small beside its work); no longer than needed (1/kSplitShare of the share:
// at long contexts nothing is split); and the pieces must fit the slots: a split row of n
// blocks has ceil(n / len) < 2 n / len pieces, so all split rows together have fewer than
// 2 total / len <= slot_capacity.
__host__ __device__ inline int64_t split_length(int64_t total_cost, int slot_capacity, int n_wg, int block) {
  if (slot_capacity < 2) return int64_t(1) << 40;
  int64_t len = kSplitMinTiles * 64 / block;
  const int64_t fit = (2 * total_cost + slot_capacity - 1) / slot_capacity;
  const int64_t share = (total_cost + int64_t(n_wg) * kSplitShare - 1) / (int64_t(n_wg) * kSplitShare);
  if (fit > len) len = fit;
  if (share > len) len = share;
  return len;
}
constexpr int kSplitMaxPieces = 64;   // pieces of one row (their weights meet in a fixed piece of LDS)
__host__ __device__ inline int pieces_of(int64_t n_sel, int64_t split_len) {
  if (n_sel <= split_len) return 1;
  const int64_t p = (n_sel + split_len - 1) / split_len;
  return int(p < kSplitMaxPieces ? p : kSplitMaxPieces);
}
// piece c of a row of n selected blocks cut into p pieces covers [piece_begin(c), piece_begin(c + 1))
__host__ __device__ inline int64_t piece_begin(int64_t n_sel, int p, int c) { return n_sel * c / p; }

// Launches whose rows count their own places (place_kernel); others are sorted by a workgroup per die (order_kernel).  A die's row
// pointers (with pieces all) are read by each of its workgroups: 57344 rows of four sequences take 26 us, and the sort as long from
// 32768 on; with pieces 4096 rows 9.2 us against 18.
constexpr int kPlacePairs = 2048, kPlaceCounted = 1 << 16, kPlaceCountedCut = 1 << 14;
inline bool places_counted(const Geometry& g, bool pieces) {
  return int64_t(g.meta.n_seq) * g.meta.n_q_heads <= kPlacePairs && g.rows <= (pieces ? kPlaceCountedCut : kPlaceCounted);
}

// A queue's item `at` where the first `halved` rows of the queue, its longest, are worked on in halves: the row's place in the
// queues, with the half (0: whole row, 1, 2) above it.
constexpr int kHalfShift = 28, kPlaceMask = (1 << kHalfShift) - 1;
constexpr int kHalvedRows = 16;       // halved rows of queue x: queue_begin[kHalvedRows + x] (launches with AttentionPlan::halves)
__host__ __device__ inline int queue_place(int begin, int halved, int at) {
  return at < 2 * halved ? (begin + (at >> 1)) | ((at & 1) + 1) << kHalfShift : begin + at - halved;
}
// Whether a row is worked on in halves, given what all rows select together and the persistent workgroups: from 1.2 times the average share on.
// A half takes some 0.65 of the row's time (its waves have half of the products and exponentials but all of the copies), so halves pay where
// a row is longer than a workgroup's average share and the launch waits for it: 28/4 heads x 5971 with two dense ones 142 -> 112 us,
// 8/2 x 16903 with one 332 -> 255, 32/8 x 3000 82 -> 70.  From 1.0 times the share on 16/4 x 12000 with two dense
// ones takes 292 us for 276 (in whole rows 293), from 0.8 on 28/4 x (3107, 2525, 392) 129 for 119; with rows of 10 to 16
// blocks in halves too 40/8 x 2155 takes 72 us for 69.
__host__ __device__ inline bool in_halves(int64_t n_sel, int64_t total_cost, int n_wg) {
  return n_sel > 16 && n_sel * 5 * n_wg > total_cost * 6;
}
// ... and whether any are: where the longest row of the launch is less than 5/3 of the share, all stay whole.  Halves are more work in all, and they
// come before whole rows that take longer than they.  Attention calls in whole rows and in halves, longest row against the share: 32/8 heads x
// 5000 1.39 times 71 -> 82 us, 32/8 x 8231 with four dense ones 1.40 times 196 -> 220, 32/8 x 12000 with one 1.42 times 272 -> 291, 40/8 x
// 6000 with four 1.66 times 136 -> 153; of 33 calls from 5/3 on 31 are 6 to 25% faster and two 2% slower.  In between some
// gain and lose this: 28/4 x 8231 with four dense ones 1.47 times 194 -> 182, 32/8 x 8231 with two 1.64 times 184 -> 169.
__host__ __device__ inline bool worth_halves(int64_t longest, int64_t total_cost, int n_wg) {
  return in_halves(longest, total_cost, n_wg) && longest * 3 * n_wg >= total_cost * 5;
}

// The per-XCD work queues the ordering kernel builds (device pointers into the workspace).
struct WorkQueues {
  const ItemRec* items;        // items, queue after queue, each by descending row cost
  const int32_t* queue_begin;  // [kXcds + 1]
  uint32_t* tickets;           // [kXcds * kTicketStride]: items taken, set by the ordering kernel to those that
                               // the attention launch's workgroups start with (see order_kernel)
};

// Where the pieces of split rows leave their results, and the per-row counts of finished pieces.
struct SplitBuffers {
  float* part_o;
  float* part_ml;
  uint32_t* done;              // [slot_capacity / 2 + 1], zeroed by the ordering kernel
  int32_t slot_capacity;
};

// How an attention launch is laid out.
struct AttentionPlan {
  int32_t groups;       // groups of waves of a workgroup that share a row: of 64 tokens by its keys, of 128 by its queries
  int32_t grid;         // workgroups
  int32_t compute_units;
  bool ordered;         // items come from queues; else every row has a workgroup
  bool halves;          // of which the longest may be halves of rows, see queue_place()
};
AttentionPlan plan_attention(const Geometry& g, int32_t n_wg, int64_t slot_capacity);
int32_t launch_attention(const Geometry& g, const AttentionPlan& plan, const void* q, const void* k, const void* v,
                         const int64_t* sel_ptr, const int32_t* sel_idx, void* out, float* lse,
                         shplb_wg_stats* stats, WorkQueues wq, SplitBuffers sb, int32_t n_wg, hipStream_t stream);

// KV head that query head h reads: the caller's map, or equal groups of consecutive heads.
__device__ __forceinline__ int kv_head_of(const SeqMeta& m, int h) {
  return m.kv_map ? int(m.kv_of[h >> 2] >> (8 * (h & 3)) & 0xff) : h / (m.n_q_heads / m.n_kv_heads);
}

// x / y, the same in all lanes, of non-negative numbers; quotients below 2^20 (the approximate one is then off by one at most).
__device__ __forceinline__ int small_quotient(int x, int y) {
  const int q = __builtin_amdgcn_readfirstlane(int(float(x) * __builtin_amdgcn_rcpf(float(y)))), r = x - q * y;
  return q + (r >= y ? 1 : 0) - (r < 0 ? 1 : 0);
}

// Row -> (sequence, head, query block), blocks of the sequence and offset of its scores.  Rows of one sequence are
// contiguous.  Of several sequences a lane looks at one (all 64 of them active); what is wanted of the row's comes from
// that lane, not by another load.  (A load that waits for another one costs some 0.3 us at the start of a launch.  With the
// geometry, the row's entry in sel_ptr and its scores asked for as early as they can be, here and in the kernels, the whole path takes 24.2
// us for 25.3 at 777 tokens x 32/8 heads, 28.9 for 30.3 at 2048 x 8/8 with 64-token blocks, 139.2 for 140.5 for 48 sequences.)
__device__ __forceinline__ void decode_row(const SeqMeta& m, int32_t row, int& s, int& h, int& i, int& nb, int64_t& score_off) {
  static_assert(SHPLB_MAX_SEQ == 64, "a lane per sequence");
  s = 0;
  nb = m.blk_begin[1];
  score_off = 0;
  if (m.n_seq > 1) {
    const int lane = threadIdx.x & 63, end = m.blk_begin[lane + 1];
    const int64_t off = m.score_off[lane];
    s = __builtin_popcountll(__ballot(lane < m.n_seq - 1 && row >= end * m.n_q_heads));
    const int first = s > 0 ? __builtin_amdgcn_readlane(end, s - 1) : 0;
    nb = __builtin_amdgcn_readlane(end, s) - first;
    row -= first * m.n_q_heads;
    score_off = int64_t(uint32_t(__builtin_amdgcn_readlane(int(off), s))) | int64_t(__builtin_amdgcn_readlane(int(off >> 32), s)) << 32;
  }
  h = small_quotient(row, nb);
  i = row - h * nb;
}

// An item from another die's queue for a persistent workgroup whose own is empty (called by one whole
// wave).  Every item comes from the queue that has the most items left at that moment (ties: the first
// one from home on): helpers so spread over the dies that still have work in proportion to what is left
// there, and no queue is left for last with its heavy items still in it.  Counts are read with device-scope
// loads, a lane per queue, and may be a little old: that only affects which queue is tried, the ticket decides.
// A queue whose ticket came back past its end is never tried again (*empty_mask), so the loop ends after at
// most kXcds misses.  Returns the item's place in the queues, or -1 when every queue is empty.
// (Now two memory round trips; with one thread going through the queues, load after load, it was ten: 48 sequences
// x 28 heads, whose dies hold unequal work, 172 -> 165 us for the whole path, an 8K prompt 189 -> 187 us.  Asked
// for behind the item's last steps they cost the tile loop registers, and 2% at 32K and 128K.)
template <bool kHalves>
__device__ __attribute__((noinline)) int help_item(const int32_t* queue_begin, uint32_t* tickets, int home, int* empty_mask) {
  static_assert(kXcds == 8, "the largest of eight lanes in three exchanges");
  int empty = *empty_mask;
  const int lane = threadIdx.x & 63, x = (home + lane) % kXcds;
  const int begin = queue_begin[x], halved = kHalves ? queue_begin[kHalvedRows + x] : 0, size = queue_begin[x + 1] - begin + halved;
  for (;;) {
    const uint32_t taken = __hip_atomic_load(tickets + x * kTicketStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int left = taken < uint32_t(size) && !(empty >> x & 1) ? size - int(taken) : 0;
    // items left and, below them, the order from home on: the largest of lanes 0 .. 7
    int best = left > 0 ? left << 3 | (kXcds - 1 - (lane & 7)) : 0;
#pragma unroll
    for (int d = 1; d < kXcds; d <<= 1) best = max(best, __shfl_xor(best, d));
    best = __builtin_amdgcn_readfirstlane(best);
    if (best == 0) break;
    const int pick = kXcds - 1 - (best & 7);             // the lane of the queue
    uint32_t t = 0;
    if (lane == pick) t = atomicAdd(tickets + x * kTicketStride, 1u);
    t = __builtin_amdgcn_readlane(t, pick);
    if (t < uint32_t(__builtin_amdgcn_readlane(size, pick))) {
      *empty_mask = empty;
      return queue_place(__builtin_amdgcn_readlane(begin, pick), kHalves ? __builtin_amdgcn_readlane(halved, pick) : 0, int(t));
    }
    empty |= 1 << __builtin_amdgcn_readlane(x, pick);
  }
  *empty_mask = empty;
  return -1;
}

__device__ __forceinline__ int my_xcd() {
  return int(__builtin_amdgcn_s_getreg((4 - 1) << 11 | 0 << 6 | 20) & 0xf) % kXcds;   // XCC_ID[3:0]
}

}  // namespace shplb
