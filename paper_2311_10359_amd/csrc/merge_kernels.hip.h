// Merging the profile of further runs into the profile of the runs so far (Section 3.2: the statistics
// run over all T measured runs of a task; a run of N kernels has N - 1 idle times, so profiles taken run
// by run and merged leave the idle time between runs out).
#pragma once

#include "common.hip.h"

namespace fikit {

constexpr int MERGE_THREADS = 256;
// IDs of a task and input kept in LDS for the searches.  A workgroup goes from one wait for memory to the next, so what
// counts is how many of them a compute unit holds: three with the larger tables, seven with the smaller ones (writing the rows
// of 20,000 tasks of 90 + 90 rows: 269 us with three, 182 us with seven; 146 us, 4.7 TB/s, since a lane moves 16 bytes and rows
// that go nowhere are not read).  Tables beyond the larger number are searched in memory.
constexpr uint32_t MERGE_IDS = 3072, MERGE_IDS_SMALL = 1024;
constexpr uint32_t MERGE_LARGE_WORKGROUPS = 3 * 256;   // of the larger tables: as many as the chip holds

template <uint32_t IDS>
struct MergeSmem {
  uint64_t ida[IDS];
  uint64_t idb[IDS];
  uint32_t aux[8];
  uint32_t partner[MERGE_THREADS];   // per row of the round: its row in the other table, or MERGE_NONE
  uint32_t place[MERGE_THREADS];     // where it goes in the task's output, or MERGE_NONE: nowhere
};
constexpr uint32_t MERGE_NONE = 0xffffffffu;

// Number of rows of `rows[0..n)` (ordered by ID) whose ID is below `id`; *found: one of them equals it.
// `ids` is the LDS copy of the IDs, or null.
__device__ __forceinline__ uint32_t ids_below(const fikit_row* __restrict__ rows, const uint64_t* ids, uint32_t n, uint64_t id,
                                              bool* found) {
  uint32_t lo = 0, hi = n;
  while (lo < hi) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    const uint64_t v = ids ? ids[mid] : rows[mid].kernel_id;
    if (v < id) lo = mid + 1; else hi = mid;
  }
  *found = lo < n && (ids ? ids[lo] : rows[lo].kernel_id) == id;
  return lo;
}

// One 8-byte field of a merged row.  f: the field's number in the row (0 ID, 1 task, 2..7 the execution
// times' count, sum, min, max, p50, p95, 8..13 the same of the idle times, 14..15 reserved); x, y: the field
// in the two rows; cx, cy: the sample counts of the field's block in the two rows.
__device__ __forceinline__ uint64_t merge_field(uint32_t f, uint64_t x, uint64_t y, uint64_t cx, uint64_t cy) {
  if (f < 2 || f >= 14) return x;
  if (cx == 0) return y;
  if (cy == 0) return x;
  const uint32_t kind = (f - 2) % 6;
  const int64_t sx = static_cast<int64_t>(x), sy = static_cast<int64_t>(y);
  if (kind <= 1) return x + y;                                            // count, sum (modulo 2^64)
  if (kind == 2) return static_cast<uint64_t>(sx < sy ? sx : sy);         // min
  if (kind == 3) return static_cast<uint64_t>(sx > sy ? sx : sy);         // max
  return cy > cx ? y : x;   // the percentiles of the union are not known: those of the input with more samples stand in
}

// Writes the planned rows of a round (sm.place / sm.partner, `rows` of them, taken from src[first ..]): eight
// lanes per row, two 8-byte fields each, so that a wave reads and writes whole rows side by side.  Rows that go nowhere
// (they went out with their partner) are not read.  Neither is needed again, and the caches keep what the next tasks' searches
// read: 20,000 tasks of 90 + 90 rows, call 262 us with ordinary reads and writes, 242 with the hint on the writes, 231 with it on
// both.
template <uint32_t IDS>
__device__ __forceinline__ void merge_write_round(const MergeSmem<IDS>& sm, const fikit_row* __restrict__ src, uint32_t first,
                                                  uint32_t rows, const fikit_row* __restrict__ other, fikit_row* __restrict__ out) {
  const uint32_t tid = threadIdx.x, f = tid & 7u;
  const int count_lane = static_cast<int>(lane_id() - f + (f < 4 ? 1 : 4));   // (fields 2 and 8)
  for (uint32_t r = tid >> 3; r < rows; r += MERGE_THREADS / 8) {      // (the eight lanes of a row stay together)
    const uint32_t place = sm.place[r], partner = sm.partner[r];
    if (place == MERGE_NONE) continue;
    ulonglong2 v = load_once(reinterpret_cast<const ulonglong2*>(src + first + r) + f);
    ulonglong2 y = make_ulonglong2(0, 0);
    if (partner != MERGE_NONE) y = load_once(reinterpret_cast<const ulonglong2*>(other + partner) + f);
    const uint64_t cx = shfl_u64(v.x, count_lane), cy = shfl_u64(y.x, count_lane);
    if (partner != MERGE_NONE) v = make_ulonglong2(merge_field(2 * f, v.x, y.x, cx, cy), merge_field(2 * f + 1, v.y, y.y, cx, cy));
    store_once(reinterpret_cast<ulonglong2*>(out + place) + f, v);
  }
}

// The control block, and what the host would have to wait for before anything runs (20,000 tasks of 90 + 90 rows, call 271 us
// with that wait, 262 us without): whether there are more rows than can be merged (`most` or more of both together), and which
// tables take the tasks (Ctrl::wide).  With MERGE_IDS_SMALL rows in both tables of a task together on average, most fit the small
// ones, and the few that do not are listed; beyond it the list would hold too many, and the larger tables take all tasks (us with
// the list / without: 1000 tasks of 2000 + 2000 rows 484 / 460, 3000 of 1100 + 1100 664 / 594; 3000 of 700 + 700 368 / 376, 7945
// of 349 + 349 427 / 449, the last two and the ones without the list with the host's wait, 8 us).
__global__ void k_merge_begin(const uint64_t* __restrict__ n_a, const uint64_t* __restrict__ n_b, uint32_t n_tasks, uint64_t most, Ctrl* ctrl) {
  const uint64_t a = *n_a, b = *n_b;
  const uint32_t i = threadIdx.x;
  Ctrl c{};
  c.status = a >= most || b >= most || a + b >= most ? ERR_TOO_MANY : 0u;
  c.wide = (a + b) / n_tasks > MERGE_IDS_SMALL ? 1u : 0u;
  if (i == 0) *ctrl = c;
}

// MODE 0: checks both inputs of a task (task field, IDs strictly ascending) and counts the rows of the
// union into dcount[t].  MODE 1: writes the union's rows at row_off[t].. in ID order.
// One workgroup per task; rank of an ID in the union = IDs below it in a + IDs below it in b - IDs below
// it that are in both (a running count of the matched rows seen so far).
// LARGE: with larger tables, either the tasks of list[0 .. ctrl->n_class[MODE]) or all (Ctrl::wide).  Otherwise all tasks or
// none; those with more than IDS rows in a table are put on the list instead.
// The large kernel's workgroups stay and count the tasks they take in ctrl->n_class[2 + MODE]: in fixed turns, tasks that are
// long at the pace of the turns meet in few workgroups, and ragged ones leave some workgroups behind (us per call, four
// workgroups for each that the chip holds in fixed turns / as many as it holds, counted: 20,000 tasks of 100 and 1800 rows in
// turn 4374 / 2882, 6144 of 200 rows, of which 200 in a row have 12,000 at two places, 3590 / 2370, 20,000 lognormal ones of 830
// rows on average 5300 / 4660, 20,000 of 700 2055 / 1975, 4000 of 700 467 / 457, 3072 of 700 371 / 376).
template <int MODE, uint32_t IDS, bool LARGE>
__global__ void __launch_bounds__(MERGE_THREADS, IDS == MERGE_IDS_SMALL ? 7 : 3)
k_merge(const fikit_row* __restrict__ a, const uint64_t* __restrict__ a_off, const fikit_row* __restrict__ b,
        const uint64_t* __restrict__ b_off, uint32_t n_tasks, uint32_t* dcount,
        const uint64_t* row_off, fikit_row* __restrict__ out, uint64_t capacity, uint32_t* list, Ctrl* ctrl) {
  __shared__ MergeSmem<IDS> sm;
  // (MODE 0: only the bit of k_merge_begin: the others are set by workgroups of this launch)
  if (MODE == 0 ? (ctrl->status & ERR_TOO_MANY) != 0 : (ctrl->status || ctrl->n_rows > capacity)) return;   // (enqueued before the host knows)
  const bool all = ctrl->wide != 0;
  if (MODE == 0 && !LARGE && blockIdx.x == 0 && threadIdx.x == 0) dcount[n_tasks] = 0;   // (the scan leaves the total here)
  if (!LARGE && all) return;
  const uint64_t n_a = a_off[n_tasks], n_b = b_off[n_tasks];
  const uint32_t tid = threadIdx.x;
  const uint32_t items = LARGE && !all ? ctrl->n_class[MODE] : n_tasks;
  auto following = [&](uint32_t item) -> uint32_t {   // (called by all threads once a task is done)
    if constexpr (!LARGE) return item + gridDim.x;
    __syncthreads();   // (all have read the word that is written now, and the task's searches are over)
    if (tid == 0) sm.aux[0] = atomicAdd(&ctrl->n_class[2 + MODE], 1u);
    __syncthreads();
    return gridDim.x + sm.aux[0];
  };
  for (uint32_t item = blockIdx.x; item < items; item = following(item)) {
    // (the rows are written from the last task to the first: what the counting pass read last is still in the cache)
    const uint32_t t = LARGE && !all ? list[item] : MODE == 1 ? items - 1 - item : item;
    const uint64_t a0 = a_off[t], a1 = a_off[t + 1], b0 = b_off[t], b1 = b_off[t + 1];
    // (n_a, n_b: the rows there are; with this every row read is in bounds, whatever the other offsets say)
    if (a1 < a0 || b1 < b0 || a1 > n_a || b1 > n_b || a1 - a0 >= (1ull << 32) || b1 - b0 >= (1ull << 32) || (t == 0 && (a0 != 0 || b0 != 0))) {
      if (tid == 0) { atomicOr(&ctrl->status, ERR_OFFSETS); if (MODE == 0) dcount[t] = 0; }
      continue;    // (the same for all threads)
    }
    const uint32_t na = static_cast<uint32_t>(a1 - a0), nb = static_cast<uint32_t>(b1 - b0);
    const fikit_row* ra = a + a0;
    const fikit_row* rb = b + b0;
    const bool in_lds = na <= IDS && nb <= IDS;
    if (!LARGE && !in_lds) {   // (the same for all threads)
      if (tid == 0) list[atomicAdd(&ctrl->n_class[MODE], 1u)] = t;
      continue;
    }
    __syncthreads();   // (the previous task's searches are over)
    bool bad = false;
    if (in_lds) {   // (ID and task are the first 16 bytes of a row: its line is touched once here)
      auto take = [&](const fikit_row* r, uint64_t* ids, uint32_t i) {
        const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(r + i);
        ids[i] = v.x;
        bad |= static_cast<uint32_t>(v.y) != t;
      };
      for (uint32_t i = tid; i < na; i += MERGE_THREADS) take(ra, sm.ida, i);
      for (uint32_t i = tid; i < nb; i += MERGE_THREADS) take(rb, sm.idb, i);
    }
    __syncthreads();
    const uint64_t* ida = in_lds ? sm.ida : nullptr;
    const uint64_t* idb = in_lds ? sm.idb : nullptr;
    uint32_t carry = 0;      // matched rows of a before this round
    for (uint32_t i0 = 0; i0 < na; i0 += MERGE_THREADS) {
      const uint32_t i = i0 + tid;
      bool found = false;
      uint32_t below = 0;
      uint64_t id = 0;
      if (i < na) {
        id = ida ? ida[i] : ra[i].kernel_id;
        below = ids_below(rb, idb, nb, id, &found);
        if (MODE == 0) bad |= (!ida && ra[i].task != t) || (i > 0 && (ida ? ida[i - 1] : ra[i - 1].kernel_id) >= id);
      }
      uint32_t total;
      const uint32_t before = block_excl_scan_256(found ? 1u : 0u, sm.aux, total);
      if (MODE == 1) {
        sm.partner[tid] = found ? below : MERGE_NONE;
        sm.place[tid] = i < na ? i + below - (carry + before) : MERGE_NONE;
        __syncthreads();
        merge_write_round(sm, ra, i0, na - i0 < MERGE_THREADS ? na - i0 : MERGE_THREADS, rb, out + row_off[t]);
        __syncthreads();
      }
      carry += total;
    }
    const uint32_t matched = carry;
    carry = 0;               // matched rows of b before this round
    for (uint32_t k0 = 0; k0 < nb; k0 += MERGE_THREADS) {
      const uint32_t k = k0 + tid;
      bool found = false;
      uint32_t below = 0;
      if (k < nb) {
        const uint64_t id = idb ? idb[k] : rb[k].kernel_id;
        if (MODE == 1) below = ids_below(ra, ida, na, id, &found);
        if (MODE == 0) bad |= (!idb && rb[k].task != t) || (k > 0 && (idb ? idb[k - 1] : rb[k - 1].kernel_id) >= id);
      }
      if (MODE == 1) {
        uint32_t total;
        const uint32_t before = block_excl_scan_256(found ? 1u : 0u, sm.aux, total);
        sm.partner[tid] = MERGE_NONE;
        sm.place[tid] = (k < nb && !found) ? k + below - (carry + before) : MERGE_NONE;    // (matched rows went out with a's)
        __syncthreads();
        merge_write_round(sm, rb, k0, nb - k0 < MERGE_THREADS ? nb - k0 : MERGE_THREADS, ra, out + row_off[t]);
        __syncthreads();
        carry += total;
      }
    }
    if (MODE == 0) {
      if (bad) atomicOr(&ctrl->status, ERR_ROWS);
      if (tid == 0) dcount[t] = na + nb - matched;
    }
  }
}

}  // namespace fikit
