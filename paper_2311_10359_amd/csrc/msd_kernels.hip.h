// Long tasks (more launches than one workgroup can hold): one pass over the launch records splits
// every tile of a task by the top bits of the Kernel ID, and one workgroup each then works on
// units of consecutive ID buckets, gathering each unit's launches from the tiles.  Because the ID is a
// hash, the buckets are of similar size unless a few IDs dominate the task; a bucket larger than a
// workgroup can hold is streamed by one (k_unit_large) if its task is long enough, otherwise the task
// keeps the general sort-based path.  In a task of more tiles than a unit's run table lists
// (UNIT_RUNS_MAX) every bucket is streamed, however small.
//
//   k_plan_msd        which tasks are long, how many tiles each has
//   k_tile_partition  one tile per workgroup: Kernel ID / execution time / idle time of every launch
//                     (Section 3.2); the IDs leave in launch order (an output of the call), and the tile's
//                     launches leave again as (ID, execution time, idle time) triples ordered by bucket
//                     inside the tile's own index range, with the tile's table of bucket boundaries.
//                     Nothing depends on another tile: no counters, no waiting, one read of the records.
//   k_msd_units       bucket sizes of a task (summed over its tiles) -> units of at most FUSE_MID_MAX
//                     launches (FUSE_SMALL_MAX in shorter tasks; or one larger bucket)
//   k_unit_sorted     (unit_kernels.hip.h) reads a unit's launches as one run per tile and makes its rows
//   k_unit_large      (stream_kernels.hip.h) the same for units of more than FUSE_MID_MAX launches, and the streamed ones
//   k_msd_task_rows / k_gather_units   row counts and final placement of the units' rows
//   k_long_general_values   per-launch values of long tasks that had to be left to the general path
#pragma once

#include "common.hip.h"
#include "profile_kernels.hip.h"
#include "sort_kernels.hip.h"
#include "task_kernels.hip.h"

namespace fikit {

// Top ID bits that name a launch's bucket.  All tasks use as many: neighbouring buckets are packed into one unit anyway, and
// the finer the buckets, the fewer IDs share one with a frequent ID (unit_streamed).
constexpr uint32_t MSD_BITS = 8;
constexpr uint32_t MSD_SLOTS = 1u << MSD_BITS;       // buckets, and unit slots reserved per long task
constexpr uint32_t PT_TILE = 4096;                   // launches per tile of the partition pass
constexpr int PT_THREADS = 512, PT_WAVES = PT_THREADS / WAVE, PT_KPT = PT_TILE / PT_THREADS;
constexpr int PT_LB = 2;                             // rounds of record loads in flight per lane
// A bucket of more than FUSE_MAX launches (one frequent ID) is streamed (unit_streamed) if its task has at least this
// many launches; otherwise the task is sorted.  fikit_profile, one ID with 90 / 50 / 35 % of the launches beside 300 others, in
// ms sorted / streamed (the line moved down for it):
//   64 tasks of 24,000 launches: 0.53 / 0.31 (90 %), 0.53 / 0.28 (70 %)   64 of 40,000: 0.65 / 0.38, 0.76 / 0.28 (50 %)
//   64 of 65,536: 0.82 / 0.43, 0.94 / 0.33, 0.91 / 0.31   256 of 131,072: 3.90 / 1.15, 4.53 / 1.07, 4.47 / 1.03
//   256 of 262,143: 8.29 / 2.16, 7.91 / 2.00, 7.76 / 1.97
// Streaming is ahead in all of these, and the tasks below the line are sorted all the same: it was drawn when streaming still
// lost at 24,000 and 40,000 launches, and has not been moved since.  A task may also be tried in vain, as a unit of the other IDs
// holds more of them than its table; that costs little (sorted / tried and sorted, one ID with half of the launches beside 20,000
// others: 64 tasks of 40,000 1.23 / 1.28, 64 of 65,536 1.55 / 1.59, 256 of 131,072 8.24 / 8.45, 256 of 262,143 12.6 / 13.0).
constexpr uint64_t STREAM_MIN = 1u << 18;
// Tasks of up to this many launches are cut into units of at most FUSE_SMALL_MAX launches, longer ones (whose buckets alone may
// be longer) of FUSE_MID_MAX.  fikit_profile, uniform over 300 IDs, in ms with the smaller / the larger units:
//   1024 tasks of 65,536 launches: 1.88 / 1.98   1000 of 100,000: 2.62 / 2.71   50 of 131,072: 0.260 / 0.288
//   256 of 262,144: 1.92 / 1.82   16 of 1,048,576: 0.60 / 0.60
constexpr uint64_t UNIT_SMALL_TASK = 1u << 17;
constexpr uint32_t STREAM_HUGE = 1u << 16;           // streamed units beyond this are started first
constexpr uint32_t STREAM_LONGEST = 1u << 17;        // and counted beyond this (see k_unit_large)
constexpr uint32_t PT_ROWS = MSD_SLOTS + 1;          // rows of a task's boundary table: bucket 0 .. 256 (= the tile's end)
static_assert(PT_TILE <= 0xffffu, "bucket boundaries inside a tile are stored in 16 bits");
static_assert(MSD_SLOTS == 256, "the scans over a task's slots are those of a 256-thread block");
static_assert(MSD_SLOTS * FUSE_MAX / PT_TILE <= UNIT_RUNS_MAX, "a unit's run table holds one run per tile of its task");

// is_long[t] = 1 for tasks that take this path, mtiles[t] = their number of tiles; both arrays have
// n_tasks + 1 entries (last 0) and are turned into prefix sums by the caller.
__global__ void k_plan_msd(const uint64_t* __restrict__ off, uint32_t n_tasks, const uint32_t* __restrict__ gflag,
                           uint32_t* __restrict__ is_long, uint32_t* __restrict__ mtiles, uint32_t* __restrict__ wflag) {
  const uint64_t t = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t > n_tasks) return;
  uint32_t l = 0, tiles = 0;
  if (t < n_tasks) {
    const uint64_t len = off[t + 1] - off[t];
    if (gflag[t] && len > FUSE_MAX) { l = 1; tiles = static_cast<uint32_t>((len + PT_TILE - 1) / PT_TILE); }
    wflag[t] = 0;
  }
  is_long[t] = l;
  mtiles[t] = tiles;
}

// What the partition pass adds up, and the work lists' lengths (which are reused for units).
__global__ void k_msd_clear(uint32_t* __restrict__ bucket_size, uint64_t count, Ctrl* ctrl) {
  const uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < count) bucket_size[i] = 0;
  if (i < 6) ctrl->n_class[i] = 0;
  if (i == 6) ctrl->taken = 0;
}

struct PartSmem {
  uint64_t stage[PT_TILE];   // the tile's IDs in bucket order, then its values
  uint32_t cnt[PT_WAVES][256];
  uint32_t aux[8];
};

// One tile (PT_TILE launches of one long task) per workgroup, its launches dealt to the waves in turns of 64, so that a round of
// the workgroup's reads is one piece of memory.  What bounds it is the memory that reads and writes by turns: 256 tasks of
// 1,048,576 launches, 23.6 GB, 4.62 ms with a stretch of 512 launches per wave and ordinary stores, 4.45 ms with either the turns
// or stores that are not kept in the caches, 4.27 ms = 5.5 TB/s with both (the units then gather 4 % slower, 2.04 against 1.95
// ms; only the IDs stored so: no change; the reads hinted the same way: no change).  The boundary table of a task is stored
// bucket-major, tile-minor (bound[(first tile of the task) * PT_ROWS + bucket * tiles + tile]) so that a unit reads the two
// boundaries it needs of all tiles as two contiguous vectors.  Execution and idle times travel as 32-bit numbers (idle time
// NONE32 = the task's last launch has none); a task with a value that does not fit is flagged and left to the general path.
__global__ void __launch_bounds__(PT_THREADS)
k_tile_partition(const fikit_launch* __restrict__ rec, const uint64_t* __restrict__ off, uint32_t n_tasks,
                 const uint32_t* __restrict__ tile_prefix, const uint32_t* __restrict__ long_prefix,
                 uint64_t* __restrict__ ids, uint64_t* __restrict__ part_id, uint2* __restrict__ part_kg,
                 uint16_t* __restrict__ bound, uint32_t* __restrict__ bucket_size, uint32_t* __restrict__ wflag, Ctrl* ctrl) {
  extern __shared__ __align__(16) unsigned char part_raw[];
  PartSmem& sm = *reinterpret_cast<PartSmem*>(part_raw);
  const uint32_t j = blockIdx.x;
  const uint32_t t = task_of_tile(tile_prefix, n_tasks, j);
  const uint32_t tp = tile_prefix[t];
  const uint32_t tiles_t = tile_prefix[t + 1] - tp;
  const uint32_t jl = j - tp;
  const uint64_t task_start = off[t], task_end = off[t + 1];
  const uint64_t start = task_start + static_cast<uint64_t>(jl) * PT_TILE;
  const uint32_t m = static_cast<uint32_t>(task_end - start < PT_TILE ? task_end - start : PT_TILE);
  constexpr int shift = 64 - static_cast<int>(MSD_BITS);
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  for (uint32_t d = lane; d < 256; d += WAVE) sm.cnt[w][d] = 0;
  __builtin_amdgcn_wave_barrier();

  uint64_t idr[PT_KPT];
  uint2 kgr[PT_KPT];
  bool bad = false, wide = false;
#pragma unroll
  for (int r0 = 0; r0 < PT_KPT; r0 += PT_LB) {
    uint4 qa[PT_LB], qb[PT_LB], qc[PT_LB];
    int64_t qn[PT_LB];
    uint32_t qrun[PT_LB], qnrun[PT_LB];
#pragma unroll
    for (int u = 0; u < PT_LB; ++u) {
      const uint32_t pos = (r0 + u) * PT_THREADS + tid;
      qa[u] = qb[u] = qc[u] = make_uint4(0, 0, 0, 0);
      qn[u] = 0;
      qrun[u] = 0; qnrun[u] = 1;
      if (pos < m) {
        const uint64_t i = start + pos;
        const uint4* p = reinterpret_cast<const uint4*>(rec + i);
        qa[u] = p[0]; qb[u] = p[1]; qc[u] = p[2];
        qrun[u] = rec[i].run;
        // the next launch is the next lane's; only the wave's last lane has to read it
        if (lane == WAVE - 1 && i + 1 < task_end) { qn[u] = rec[i + 1].start_ns; qnrun[u] = rec[i + 1].run; }
      }
    }
#pragma unroll
    for (int u = 0; u < PT_LB; ++u) {
      const int r = r0 + u;
      const uint32_t pos = r * PT_THREADS + tid;
      const uint32_t nx_lo = from_next_lane(qc[u].x), nx_hi = from_next_lane(qc[u].y), nx_run = from_next_lane(qrun[u]);
      if (lane != WAVE - 1) { qn[u] = static_cast<int64_t>((static_cast<uint64_t>(nx_hi) << 32) | nx_lo); qnrun[u] = nx_run; }
      idr[r] = 0;
      kgr[r] = make_uint2(0, 0);
      if (pos < m) {
        const uint64_t i = start + pos;
        const uint4 a = qa[u], b = qb[u], c = qc[u];
        const uint32_t wd[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        const uint64_t id = kernel_id_of(wd);
        const int64_t st = static_cast<int64_t>((static_cast<uint64_t>(c.y) << 32) | c.x);
        const int64_t en = static_cast<int64_t>((static_cast<uint64_t>(c.w) << 32) | c.z);
        bad |= (en < st);
        const uint64_t e64 = static_cast<uint64_t>(en - st);
        wide |= (e64 >= NONE32);
        uint32_t g32 = NONE32;
        if (i + 1 < task_end && qnrun[u] == qrun[u]) {   // an idle time follows: same task, same run
          const int64_t g = qn[u] - en;
          const uint64_t g64 = static_cast<uint64_t>(g < 0 ? 0 : g);
          wide |= (g64 >= NONE32);
          g32 = static_cast<uint32_t>(g64);
        }
        store_once(ids + i, id);
        idr[r] = id;
        kgr[r] = make_uint2(static_cast<uint32_t>(e64), g32);
      }
    }
  }
  if (bad) atomicOr(&ctrl->status, ERR_BAD_RECORD);
  if (ballot(wide) && lane == 0) atomicOr(&wflag[t], 1u);

  uint32_t rk[PT_KPT];
#pragma unroll
  for (int r = 0; r < PT_KPT; ++r) {
    const uint32_t pos = r * PT_THREADS + tid;
    rk[r] = wave_rank_digit(static_cast<uint32_t>(idr[r] >> shift), pos < m, sm.cnt[w]);
  }
  tile_digit_offsets<PT_WAVES>(sm.cnt, sm.aux, nullptr);
  // where each bucket starts inside the tile, and the
  // tile's share of the task's bucket sizes (integer adds: the totals do not depend on the order of the tiles)
  if (tid < 256) {
    const uint32_t first = sm.cnt[0][tid], next = tid < 255 ? sm.cnt[0][tid + 1] : m;
    bound[static_cast<uint64_t>(tp) * PT_ROWS + static_cast<uint64_t>(tid) * tiles_t + jl] = static_cast<uint16_t>(first);
    if (next > first) atomicAdd(&bucket_size[static_cast<uint64_t>(long_prefix[t]) * MSD_SLOTS + tid], next - first);
  }
  if (tid == 256) bound[static_cast<uint64_t>(tp) * PT_ROWS + static_cast<uint64_t>(MSD_SLOTS) * tiles_t + jl] = static_cast<uint16_t>(m);
  uint32_t at[PT_KPT];
#pragma unroll
  for (int r = 0; r < PT_KPT; ++r) {
    const uint32_t pos = r * PT_THREADS + tid;
    at[r] = sm.cnt[w][static_cast<uint32_t>(idr[r] >> shift)] + rk[r];
    if (pos < m) sm.stage[at[r]] = idr[r];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PT_KPT; ++r) {
    const uint32_t i = tid + r * PT_THREADS;
    if (i < m) store_once(part_id + start + i, sm.stage[i]);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PT_KPT; ++r) {
    const uint32_t pos = r * PT_THREADS + tid;
    if (pos < m) sm.stage[at[r]] = (static_cast<uint64_t>(kgr[r].y) << 32) | kgr[r].x;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PT_KPT; ++r) {
    const uint32_t i = tid + r * PT_THREADS;
    if (i < m) store_once(reinterpret_cast<uint64_t*>(part_kg) + start + i, sm.stage[i]);   // (execution time in the lower half)
  }
}

// One workgroup per task: packs a long task's ID buckets into units (a bucket of more than FUSE_MAX launches is a
// unit of its own).  A task with such a bucket and fewer than STREAM_MIN launches, or with an execution or idle time
// that does not fit 32 bits, keeps the general path (mflag 0); otherwise mflag 1 and gflag cleared.  Every thread finds where a
// unit that starts at its bucket would end and the next one start, one thread follows these from unit to unit, and all threads
// together write the unit slots and the work lists.  bucket_size: the task's bucket sizes as the tiles added them up.
__global__ void __launch_bounds__(MSD_SLOTS)
k_msd_units(const uint64_t* __restrict__ off, uint32_t n_tasks, const uint32_t* __restrict__ long_prefix,
            const uint32_t* __restrict__ tile_prefix, const uint32_t* bucket_size, uint32_t* ustage, const uint32_t* __restrict__ wflag,
            uint32_t* __restrict__ ustart, uint32_t* __restrict__ ulen, uint32_t* __restrict__ utask,
            uint32_t* __restrict__ udcount, uint32_t* __restrict__ ubuckets, uint32_t* __restrict__ mflag,
            uint32_t* __restrict__ gflag, uint32_t* __restrict__ lists, uint32_t list_stride, Ctrl* ctrl) {
  __shared__ uint32_t bstart[MSD_SLOTS + 1];   // where each bucket starts inside the task (in bucket order)
  __shared__ uint32_t after[MSD_SLOTS], follows[MSD_SLOTS + 1], ufirst[MSD_SLOTS];
  __shared__ uint32_t aux[8];
  __shared__ uint32_t n_used, too_large;
  const uint32_t t = blockIdx.x, d = threadIdx.x;
  if (t >= n_tasks) return;
  if (d == 0) mflag[t] = 0;
  if (long_prefix[t + 1] == long_prefix[t]) return;   // not a long task
  const uint32_t o = long_prefix[t];
  const uint64_t task_start = off[t], len = off[t + 1] - task_start;
  const uint32_t tiles_t = tile_prefix[t + 1] - tile_prefix[t];
  const uint32_t size = bucket_size[static_cast<uint64_t>(o) * MSD_SLOTS + d];
  uint32_t total;
  const uint32_t before = block_excl_scan_256(size, aux, total);
  bstart[d] = before;
  if (d == 0) { bstart[MSD_SLOTS] = total; too_large = 0; follows[MSD_SLOTS] = MSD_SLOTS; }
  __syncthreads();
  const bool may_stream = len >= STREAM_MIN;
  const uint32_t unit_max = len <= UNIT_SMALL_TASK ? FUSE_SMALL_MAX : FUSE_MID_MAX;
  const bool single = tiles_t > UNIT_RUNS_MAX;   // more runs than a unit's table holds: every bucket is streamed
  if (size > FUSE_MAX && !may_stream) too_large = 1;
  // first index in (lo, MSD_SLOTS] at which the buckets before it hold more than `most` launches, or MSD_SLOTS + 1
  auto passes = [&](uint32_t lo, uint32_t most) {
    uint32_t hi = MSD_SLOTS + 1;
    while (hi - lo > 1) { const uint32_t mid = (lo + hi) >> 1; if (bstart[mid] > most) hi = mid; else lo = mid; }
    return hi;
  };
  // A unit that starts at bucket d ends before the bucket that makes it longer than unit_max, but holds one bucket at least.
  {
    const uint32_t end = single ? d + 1 : passes(d, before + unit_max) - 1;
    after[d] = end > d ? end : d + 1;
  }
  __syncthreads();
  {   // the next unit starts at the first bucket from there on that is not empty
    const uint32_t e = after[d];
    follows[d] = e < MSD_SLOTS ? passes(e, bstart[e]) - 1 : MSD_SLOTS;
  }
  __syncthreads();
  if (d == 0) {
    uint32_t u = 0;
    for (uint32_t f = passes(0, 0) - 1; f < MSD_SLOTS; f = follows[f]) ufirst[u++] = f;
    const bool ok = total == len && (!single || may_stream) && wflag[t] == 0 && !too_large;
    n_used = ok ? u : 0;
    if (ok) {
      mflag[t] = 1;
      gflag[t] = 0;
      atomicAdd(reinterpret_cast<unsigned long long*>(&ctrl->n_general), ~0ull);   // one general task fewer
    }
  }
  __syncthreads();
  const uint32_t used = n_used;
  const uint32_t u = o * MSD_SLOTS + d;
  utask[u] = t;
  udcount[u] = 0;
  ustage[u] = ~0u;   // (SU_UNPLACED; in the place of this thread's own bucket size)
  const bool live = d < used;
  const uint32_t first = live ? ufirst[d] : 0u, past = live ? after[first] : 0u;
  const uint32_t l = live ? bstart[past] - bstart[first] : 0u;
  ustart[u] = live ? static_cast<uint32_t>(task_start) + bstart[first] : 0u;
  ulen[u] = l;
  ubuckets[u] = live ? first | (past << 16) : 0u;
  // work lists of units by size class (see k_classify): one reservation per task and class (a counter that every
  // unit bumped on its own would serialise the whole launch on one address)
  // (list 3: streamed units, huge ones from its front and the others from its back)
  const bool streamed = live && (l > FUSE_MAX || tiles_t > UNIT_RUNS_MAX);
  if (streamed && l > STREAM_LONGEST) atomicAdd(&ctrl->n_class[5], 1u);
  const uint32_t c = !live ? 5u : streamed ? (l > STREAM_HUGE ? 3u : 4u) : (l <= FUSE_SMALL_MAX ? 0u : (l <= FUSE_MID_MAX ? 1u : 2u));
  const uint32_t in_large = wave_sum_u32(c >= 2 && c <= 4 ? l : 0u);   // (k_unit_large's part of the launches, of which there are fewer than 2^32)
  if (in_large && lane_id() == 0) atomicAdd(&ctrl->n_large, in_large);
  __syncthreads();   // (aux is reused)
  for (uint32_t k = 0; k < 5; ++k) {
    uint32_t total;
    const uint32_t at = block_excl_scan_256(c == k ? 1u : 0u, aux, total);
    __shared__ uint32_t list_base;
    if (d == 0) list_base = total ? atomicAdd(&ctrl->n_class[k], total) : 0u;
    __syncthreads();
    if (c == k) lists[k < 4 ? static_cast<uint64_t>(k) * list_stride + list_base + at : 4ull * list_stride - 1 - (list_base + at)] = u;
    __syncthreads();
  }
}

// Long tasks that the general path has to take after all (a bucket too large for a workgroup, too many
// distinct IDs in a unit, a value beyond 32 bits): the general path wants (ID, execution time, idle time)
// of every launch of the task, in any order, as 64-bit arrays.  They are unpacked from the tile-ordered
// triples; only a task with a value beyond 32 bits is measured again from its records.
__global__ void __launch_bounds__(256)
k_long_general_values(const fikit_launch* __restrict__ rec, const uint64_t* __restrict__ off, uint32_t n_tasks,
                      const uint32_t* __restrict__ tile_prefix, const uint32_t* __restrict__ gflag,
                      const uint32_t* __restrict__ wflag, const uint64_t* __restrict__ ids, uint64_t* __restrict__ key,
                      const uint2* __restrict__ part_kg, int64_t* __restrict__ e0, int64_t* __restrict__ g0) {
  const uint32_t j = blockIdx.x;
  const uint32_t t = task_of_tile(tile_prefix, n_tasks, j);
  if (!gflag[t]) return;
  const uint32_t jl = j - tile_prefix[t];
  const uint64_t task_end = off[t + 1];
  const uint64_t start = off[t] + static_cast<uint64_t>(jl) * PT_TILE;
  const uint32_t m = static_cast<uint32_t>(task_end - start < PT_TILE ? task_end - start : PT_TILE);
  const bool from_records = wflag[t] != 0;
  for (uint32_t x = threadIdx.x; x < m; x += 256) {
    const uint64_t i = start + x;
    if (from_records) {
      const int64_t en = rec[i].end_ns;
      int64_t gap = GAP_NONE;
      if (i + 1 < task_end && rec[i + 1].run == rec[i].run) { gap = rec[i + 1].start_ns - en; gap = gap < 0 ? 0 : gap; }
      key[i] = ids[i];
      e0[i] = en - rec[i].start_ns;
      g0[i] = gap;
    } else {
      const uint2 kg = part_kg[i];
      e0[i] = static_cast<int64_t>(kg.x);
      g0[i] = kg.y == NONE32 ? GAP_NONE : static_cast<int64_t>(kg.y);
    }
  }
}

// Row count of every long task that went through units, and each unit's first row inside its task.  One workgroup per task.
__global__ void __launch_bounds__(MSD_SLOTS)
k_msd_task_rows(uint32_t n_tasks, const uint32_t* __restrict__ long_prefix, const uint32_t* __restrict__ mflag,
                const uint32_t* __restrict__ udcount, uint32_t* __restrict__ urow, uint32_t* __restrict__ dcount) {
  __shared__ uint32_t aux[8];
  const uint32_t t = blockIdx.x;
  if (t >= n_tasks || long_prefix[t + 1] == long_prefix[t] || !mflag[t]) return;   // (the same for all threads)
  const uint32_t u = long_prefix[t] * MSD_SLOTS + threadIdx.x;
  uint32_t total;
  urow[u] = block_excl_scan_256(udcount[u], aux, total);
  if (threadIdx.x == 0) dcount[t] = total;
}

// Moves a unit's staged rows to their final place.
__global__ void __launch_bounds__(256)
k_gather_units(const uint64_t* __restrict__ off, const uint32_t* __restrict__ ulen, const uint32_t* __restrict__ utask,
               const uint32_t* __restrict__ udcount, const uint32_t* __restrict__ urow, const uint32_t* __restrict__ ustage,
               const uint32_t* __restrict__ mflag,
               const uint64_t* __restrict__ row_off, const int64_t* __restrict__ stage_a, const int64_t* __restrict__ stage_b,
               uint32_t n_units, fikit_row* __restrict__ rows, uint64_t capacity, uint64_t general_done, const Ctrl* ctrl) {
  if (!rows_final(ctrl, capacity, general_done)) return;
  const uint32_t u = xcd_item(blockIdx.x, n_units);
  if (u >= n_units) return;
  if (ulen[u] == 0) return;
  const uint32_t t = utask[u];
  if (!mflag[t]) return;
  const uint32_t D = udcount[u];
  uint64_t* out = reinterpret_cast<uint64_t*>(rows + row_off[t] + urow[u]);
  const uint64_t base = off[t];
  const uint32_t m = static_cast<uint32_t>(off[t + 1] - base), row0 = ustage[u];
  for (uint32_t x = threadIdx.x; x < D * 16; x += 256) {
    const uint32_t j = x >> 4, f = x & 15;
    out[x] = staged_row(const_cast<int64_t*>(stage_a), const_cast<int64_t*>(stage_b), base, m, row0 + j)[f];
  }
}

}  // namespace fikit
