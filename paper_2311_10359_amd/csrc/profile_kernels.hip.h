// Kernel ID hashing and per-launch measurement (Section 3.2, "Identifying each kernel" and
// "Measuring the execution and idle time of kernel"), plus small bookkeeping kernels.
#pragma once

#include "common.hip.h"

namespace fikit {

__global__ void k_clear_ctrl(Ctrl* ctrl) {
  if (threadIdx.x < sizeof(Ctrl) / 4) reinterpret_cast<uint32_t*>(ctrl)[threadIdx.x] = 0;
}

// Words for the host: stored in its memory, and behind them, once they are there, the number that it waits for.  One wave.
constexpr int REPORT_READS = 4;
struct Report {
  const uint32_t* from[REPORT_READS];
  uint32_t* to[REPORT_READS];
  uint32_t words[REPORT_READS];
};
__global__ void __launch_bounds__(WAVE)
k_report(const Report r, uint32_t* seen, uint32_t number) {
#pragma unroll
  for (int i = 0; i < REPORT_READS; ++i)
    if (threadIdx.x < r.words[i]) r.to[i][threadIdx.x] = r.from[i][threadIdx.x];
  __threadfence_system();
  if (threadIdx.x == 0) __hip_atomic_store(seen, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Fills `count` 32-bit words with `value` (used instead of memset so that a caller may capture
// the stream into a graph).
__global__ void k_fill_u32(uint32_t* __restrict__ p, uint64_t count, uint32_t value) {
  uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const uint64_t stride = static_cast<uint64_t>(gridDim.x) * blockDim.x;
  for (; i < count; i += stride) p[i] = value;
}

// Checks the CSR task offsets: first 0, non-decreasing, last == n.
__global__ void k_validate_offsets(const uint64_t* __restrict__ off, uint32_t n_tasks, uint64_t n, Ctrl* ctrl) {
  const uint64_t t = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  bool bad = false;
  if (t < n_tasks) {
    const uint64_t a = off[t], b = off[t + 1];
    bad = (a > b) || (b > n);
    if (t == 0 && a != 0) bad = true;
    if (t == n_tasks - 1 && b != n) bad = true;
  } else if (t == 0 && n_tasks == 0) {
    bad = (off[0] != 0) || (n != 0);
  }
  if (bad) atomicOr(&ctrl->status, ERR_OFFSETS);
}

// Sorts tasks into work lists by length: lists[c * n_tasks ...] for c = 0 (up to len_small launches),
// 1 (up to len_mid), 2 (up to len_max); longer tasks start on the long-task path (gflag 1).  A kernel
// that handles one class is launched over that class's list, so that every workgroup it starts has
// work of similar size (workgroups are handed to compute units in turn: a launch in which busy and
// idle workgroups alternate would keep only some of the units busy).  Order inside a list is arbitrary.
__global__ void k_classify(const uint64_t* __restrict__ off, uint32_t n_tasks, uint32_t len_small, uint32_t len_mid,
                           uint32_t len_max, uint32_t* __restrict__ gflag, uint32_t* __restrict__ dcount,
                           uint32_t* __restrict__ lists, Ctrl* ctrl) {
  if (ctrl->status & ERR_OFFSETS) return;
  const uint64_t t = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  uint32_t c = 3;   // 0, 1, 2: work list; 3: none
  bool is_long = false;
  if (t <= n_tasks) dcount[t] = 0;
  if (t < n_tasks) {
    const uint64_t len = off[t + 1] - off[t];
    is_long = len > len_max;
    gflag[t] = is_long ? 1u : 0u;
    if (!is_long && len > 0) c = len <= len_small ? 0u : (len <= len_mid ? 1u : 2u);
  }
  for (uint32_t k = 0; k < 3; ++k) {
    const uint32_t pos = wave_append(&ctrl->n_class[k], c == k);
    if (c == k) lists[static_cast<uint64_t>(k) * n_tasks + pos] = static_cast<uint32_t>(t);
  }
  const uint64_t longs = ballot(is_long);
  if (longs && lane_id() == 0) {
    atomicAdd(reinterpret_cast<unsigned long long*>(&ctrl->n_general), static_cast<unsigned long long>(__popcll(longs)));
    atomicAdd(reinterpret_cast<unsigned long long*>(&ctrl->n_long), static_cast<unsigned long long>(__popcll(longs)));
  }
}

// Everything that precedes the launches' own kernels, for up to BEGIN_TASKS tasks in one workgroup: what k_clear_ctrl,
// k_validate_offsets, k_classify and (for the long tasks) k_plan_msd and its two prefix sums do.  With few tasks all of
// these only wait for each other: a kernel that depends on the one before it costs 4.5 us however little it does (three
// launches, ten with long tasks; this one takes 2.7 us for 2 tasks and 4.2 us for 256), and the number of the long tasks'
// tiles is known a host round trip earlier.  With more tasks the calls are so long that it no longer matters.
constexpr uint32_t BEGIN_TASKS = 2048;
constexpr int BEGIN_THREADS = 1024;
struct ProfileBegin {
  uint64_t n;
  uint32_t len_small, len_mid, len_max, tile;
  uint32_t *gflag, *dcount, *lists, *long_prefix, *tile_prefix, *wflag;
  Ctrl* ctrl;
};
// (off: the task offsets, in LDS)
__device__ __forceinline__ void profile_begin(const uint64_t* off, uint32_t n_tasks, const ProfileBegin& a) {
  const uint64_t n = a.n;
  const uint32_t len_small = a.len_small, len_mid = a.len_mid, len_max = a.len_max, tile = a.tile;
  uint32_t* __restrict__ gflag = a.gflag;
  uint32_t* __restrict__ dcount = a.dcount;
  uint32_t* __restrict__ lists = a.lists;
  uint32_t* __restrict__ long_prefix = a.long_prefix;
  uint32_t* __restrict__ tile_prefix = a.tile_prefix;
  uint32_t* __restrict__ wflag = a.wflag;
  Ctrl* ctrl = a.ctrl;
  __shared__ uint32_t lds[16], listed[3], bad;
  const uint32_t tid = threadIdx.x;
  if (tid < 3) listed[tid] = 0;
  if (tid == 3) bad = 0;
  __syncthreads();
  bool wrong = n_tasks == 0 && tid == 0 && (off[0] != 0 || n != 0);
  for (uint32_t t = tid; t < n_tasks; t += BEGIN_THREADS) {
    const uint64_t a = off[t], b = off[t + 1];
    wrong |= a > b || b > n || (t == 0 && a != 0) || (t + 1 == n_tasks && b != n);
  }
  if (wrong) bad = 1;
  __syncthreads();
  uint32_t longs = 0, tiles = 0;
  for (uint32_t t0 = 0; !bad && t0 <= n_tasks; t0 += BEGIN_THREADS) {   // (one entry more than tasks)
    const uint32_t t = t0 + tid;
    uint32_t c = 3, is_long = 0, my_tiles = 0;
    if (t < n_tasks) {
      const uint64_t len = off[t + 1] - off[t];
      is_long = len > len_max ? 1u : 0u;
      my_tiles = is_long ? static_cast<uint32_t>((len + tile - 1) / tile) : 0u;
      gflag[t] = is_long;
      wflag[t] = 0;
      if (!is_long && len > 0) c = len <= len_small ? 0u : (len <= len_mid ? 1u : 2u);
    }
    for (uint32_t k = 0; k < 3; ++k) {
      const uint32_t pos = wave_append(&listed[k], c == k);
      if (c == k) lists[static_cast<uint64_t>(k) * n_tasks + pos] = t;
    }
    uint32_t more_longs, more_tiles;
    const uint32_t l = block_excl_scan_1024(is_long, lds, more_longs), x = block_excl_scan_1024(my_tiles, lds, more_tiles);
    if (t <= n_tasks) {
      dcount[t] = 0;
      long_prefix[t] = longs + l;
      tile_prefix[t] = tiles + x;
    }
    longs += more_longs;
    tiles += more_tiles;
  }
  __syncthreads();
  if (tid == 0) {
    Ctrl c{};
    c.status = bad ? ERR_OFFSETS : 0u;
    c.n_big_tiles = tiles;
    c.n_general = c.n_long = longs;
    for (int k = 0; k < 3; ++k) c.n_class[k] = listed[k];
    *ctrl = c;
  }
}
// Execution time and idle time of every launch as they stand in the trace (Section 3.2, "Measuring the
// execution and idle time of kernel"); task boundaries are put right by k_measure_task_ends afterwards.
// Bound by HBM, which reads 64 bytes and writes 16 by turns.  A lane reads its own launch's times as 16 bytes and its run; the next
// launch's are the next lane's, the wave's last lane has its neighbour's read by all as one place.  24,000,000 launches:
// 399 us with the next launch read by every lane, 361 so, 341 us = 5.6 TB/s with the hint that neither what is read nor what is
// written will be used again (only the writes 347, only the reads 361; two launches per lane 370 with both hints; 378 without,
// four 383).
__global__ void __launch_bounds__(256)
k_measure(const fikit_launch* __restrict__ rec, uint64_t n, int64_t* __restrict__ exec_ns, int64_t* __restrict__ gap_ns,
          Ctrl* ctrl) {
  if (ctrl->status & ERR_OFFSETS) return;
  const uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const uint64_t wave = i & ~static_cast<uint64_t>(WAVE - 1);
  if (wave >= n) return;
  const fikit_launch *mine = rec + (i < n ? i : n - 1), *behind = rec + (wave + WAVE < n ? wave + WAVE : n - 1);
  // (records lie on 16 bytes, see fikit_launch; a caller's are only asked to lie on 8)
  const u64x2_native t = __builtin_nontemporal_load(reinterpret_cast<const u64x2_native*>(&mine->start_ns));
  const uint32_t run = mine->run;
  const int64_t behind_start = behind->start_ns;
  const uint32_t behind_run = behind->run;
  const int64_t start = static_cast<int64_t>(t.x), end = static_cast<int64_t>(t.y);
  const uint32_t lo = from_next_lane(static_cast<uint32_t>(t.x)), hi = from_next_lane(static_cast<uint32_t>(t.x >> 32)), next_run = from_next_lane(run);
  const bool last = lane_id() == WAVE - 1;
  const int64_t next = last ? behind_start : static_cast<int64_t>(static_cast<uint64_t>(hi) << 32 | lo);
  if (i >= n) return;
  if (end < start) atomicOr(&ctrl->status, ERR_BAD_RECORD);
  int64_t g = GAP_NONE;
  if (i + 1 < n && (last ? behind_run : next_run) == run) { g = next - end; g = g < 0 ? 0 : g; }   // (same run)
  store_once(exec_ns + i, end - start);
  store_once(gap_ns + i, g);
}

// The last launch of every task has no idle time after it (whatever run the next task's first launch names).
__global__ void k_measure_task_ends(const uint64_t* __restrict__ off, uint32_t n_tasks, int64_t* __restrict__ gap_ns,
                                    const Ctrl* ctrl) {
  if (ctrl->status & ERR_OFFSETS) return;
  const uint64_t t = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t < n_tasks && off[t + 1] > off[t]) gap_ns[off[t + 1] - 1] = GAP_NONE;
}

// FNV-1a, 64 bit, over the eight little-endian 32-bit words that hold a launch's identity
// (name id, grid x y z, block x y z, dynamic shared-memory bytes): for each byte in memory
// order, xor it into the hash, then multiply by the FNV prime 2^40 + 0x1b3 modulo 2^64.
__device__ __forceinline__ uint64_t kernel_id_of(const uint32_t (&w)[8]) {
  uint32_t lo = 0x84222325u, hi = 0xcbf29ce4u;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      lo ^= (w[k] >> (8 * b)) & 0xffu;
      // (hi:lo) * (2^40 + 0x1b3): the 2^40 term only reaches the high word as lo << 8.
      const uint32_t hi_part = hi * 0x1b3u + (lo << 8);
      const uint64_t prod = static_cast<uint64_t>(lo) * 0x1b3u + (static_cast<uint64_t>(hi_part) << 32);
      lo = static_cast<uint32_t>(prod);
      hi = static_cast<uint32_t>(prod >> 32);
    }
  }
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

}  // namespace fikit
