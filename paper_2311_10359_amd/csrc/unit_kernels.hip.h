// Units of long tasks: groups of consecutive ID buckets, gathered from the tiles that k_tile_partition ordered, one workgroup each.
//
//   1. The unit's launches are read, one run per tile, into registers.  Their IDs are entered in an LDS table, and a count per
//      slot gives every launch its place among those of its ID.
//   2. The slots' counts are summed up, the IDs are ranked (rows leave in ascending ID order), and execution and idle times go to
//      LDS grouped by ID.
//   3. An ID with more than twice a wave's share of the launches is worked on by all waves, each on its share of them: the steps of
//      pick_group with a barrier between them.  The other IDs are taken by a wave each.  Rows are staged.
//
// What bounds it: half of the time is the gather (runs of a few hundred bytes), the other half vector instructions, about sixty
// per sample pair in step 3; a workgroup's LDS (8 bytes per launch) decides how many units a compute unit overlaps.  Steps 1 and
// 2 as before with registers instead of LDS and a barrier after each of some forty short steps took 1.1 to 2.2 times as long:
// fikit_profile, us, before / now: 256 tasks of 1,048,576 launches, uniform over 1000 IDs 7840 / 6945 (its units 3240 / 2410);
// 64 of them, Zipf over 4096 IDs 3580 / 2410 (1440 / 685 for the units, the rest from the streamed ones); 16 of 1,000,000, 1000
// IDs, times that hardly vary 1208 / 542; 64 of 131,072, 30 IDs, times in steps of 500 ns 809 / 375; 256 of 50,000 in passes over
// 300 IDs 574 / 434; 64 of 20,000, 20 IDs 141 / 132.  The share from which on all waves work on an ID: with one wave for every ID
// the skewed units take 1770 us, with all waves from one share on those of the 1000 IDs 2790 us.
#pragma once

#include <type_traits>

#include "common.hip.h"
#include "select_kernels.hip.h"
#include "task_kernels.hip.h"

namespace fikit {

constexpr int UNIT_DMAX = 256;      // IDs of a unit of up to FUSE_MID_MAX launches
constexpr int UNIT_DMAX_LARGE = 512;   // of a larger one
constexpr uint32_t UNIT_SHARE_MIN = 256;   // an ID of up to this many launches is a wave's

template <int NT, int KPT, int DMAX>
struct UnitSmem {
  static constexpr uint32_t HT = 2 * DMAX, CAP = NT * KPT, NW = NT / WAVE;
  union {
    struct { uint32_t at[UNIT_RUNS_MAX], before[UNIT_RUNS_MAX + 4]; uint16_t of[CAP]; } runs;   // step 1
    uint32_t val[2][CAP];      // from step 2: execution times, idle times
  } u;
  union {
    uint64_t ht_key[HT];       // ID table (open addressing), until the IDs are ranked
    uint32_t hist[NW][PICK_HIST];
  } v;
  uint32_t ht_cnt[HT];         // by slot: launches
  uint16_t first[HT];          //          where they start in val
  uint64_t key[DMAX];          // the IDs in the order in which they were met
  uint16_t slot[DMAX], rank[DMAX];
  uint16_t order[DMAX];        // the IDs that all waves work on, then the others
  struct { Tally t; Range r50, r95; } shared[NW][2];   // by place in order and array
  uint32_t aux[NW];
  uint32_t ndist, fallback, first_row, given_up, n_shared, shared_launches, more;
};

template <int NT, int KPT, int DMAX>
__device__ __forceinline__ void unit_sorted(const FusedArgs& A, uint32_t unit, UnitSmem<NT, KPT, DMAX>& sm) {
  using Smem = UnitSmem<NT, KPT, DMAX>;
  constexpr uint32_t HT = Smem::HT, CAP = Smem::CAP, NW = Smem::NW;
  constexpr int PLACE_AT = 10;   // a launch's slot and place in one word
  static_assert(HT <= 1u << PLACE_AT && CAP <= PICK_SAMPLES && CAP <= 1u << (32 - PLACE_AT), "slot and place of a launch");
  static_assert(UNIT_RUNS_MAX <= 0x10000, "runs are numbered in 16 bits");
  Ctrl* ctrl = A.ctrl;
  const uint32_t t = A.utask[unit], m = A.ulen[unit];
  if (m == 0 || m > CAP) return;   // (cannot happen for a listed unit)
  const uint64_t base = A.off[t];
  const uint32_t task_len = static_cast<uint32_t>(A.off[t + 1] - base);
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t w = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(tid / WAVE)));

  for (uint32_t i = tid; i < HT; i += NT) { sm.v.ht_key[i] = HT_EMPTY; sm.ht_cnt[i] = 0; }
  if (tid == 0) { sm.ndist = 0; sm.fallback = 0; }

  // ---- 1. read ---------------------------------------------------------------------------------
  // The unit's launches lie in one run per tile of its task: between the boundaries of its first bucket and of the bucket
  // after its last.  Where each run starts, and how many of the unit's launches precede it:
  {
    const uint32_t ub = A.ubuckets[unit], d0 = ub & 0xffffu, d1 = ub >> 16;
    const uint32_t tp = A.tile_prefix[t], tiles_t = A.tile_prefix[t + 1] - tp;
    // (another unit may have given the task up; looked at when the run table stands, so that nothing waits for it)
    const uint32_t alive = tid == 0 ? __hip_atomic_load(&A.mflag[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 1u;
    const uint16_t* b_lo = A.bound + static_cast<uint64_t>(tp) * (256 + 1) + static_cast<uint64_t>(d0) * tiles_t;
    const uint16_t* b_hi = A.bound + static_cast<uint64_t>(tp) * (256 + 1) + static_cast<uint64_t>(d1) * tiles_t;
    uint32_t carry = 0;
    for (uint32_t j0 = 0; j0 < tiles_t; j0 += NT) {   // (trip count is the same for every thread)
      const uint32_t j = j0 + tid;
      uint32_t lo = 0, c = 0;
      if (j < tiles_t) { lo = b_lo[j]; c = static_cast<uint32_t>(b_hi[j]) - lo; }
      uint32_t total;
      const uint32_t ex = block_excl_scan<NT>(c, sm.aux, total);
      if (j < tiles_t) {
        sm.u.runs.at[j] = static_cast<uint32_t>(base) + j * A.tile_len + lo;
        sm.u.runs.before[j] = carry + ex;
      }
      carry += total;
    }
    if (tid == 0) { sm.u.runs.before[tiles_t] = carry; sm.given_up = alive ? 0u : 1u; }
    __syncthreads();
    if (sm.given_up) return;   // (the same for all threads: nothing else writes the word)
    if (carry != m) {   // (cannot happen: the unit's length is the sum of these runs)
      if (tid == 0) atomicOr(&ctrl->status, ERR_OFFSETS);
      return;
    }
    // every run writes its number over the launches it holds, so that a launch finds its run with one look
    for (uint32_t j = tid; j < tiles_t; j += NT) {
      const uint32_t hi = sm.u.runs.before[j + 1];
      for (uint32_t i = sm.u.runs.before[j]; i < hi; ++i) sm.u.runs.of[i] = static_cast<uint16_t>(j);
    }
    __syncthreads();
  }
  uint32_t ev[KPT], gv[KPT], at[KPT];   // execution time, idle time (NONE32 for a run's last launch); slot and place
  {
    // all of a thread's launches are located first and then read together, so that their loads are in flight at once
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
      const uint32_t i = min_u32(r * NT + tid, m - 1);
      const uint32_t j = sm.u.runs.of[i];
      at[r] = sm.u.runs.at[j] + (i - sm.u.runs.before[j]);
    }
    uint64_t id[KPT];
#pragma unroll
    for (int r = 0; r < KPT; ++r) id[r] = A.part_id[at[r]];
#pragma unroll
    for (int r = 0; r < KPT; ++r) { const uint2 kg = A.part_kg[at[r]]; ev[r] = kg.x; gv[r] = kg.y; }
    bool full = false;
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
      uint32_t h = (static_cast<uint32_t>(id[r] >> 32) ^ static_cast<uint32_t>(id[r])) & (HT - 1);
      if (r * NT + tid < m) {
        bool placed = false;
        if (id[r] != HT_EMPTY) {
          for (uint32_t probe = 0; probe < HT; ++probe) {
            const uint64_t k = __hip_atomic_load(&sm.v.ht_key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (k == id[r]) { placed = true; break; }
            if (k == HT_EMPTY) {
              const uint64_t old = atomicCAS(reinterpret_cast<unsigned long long*>(&sm.v.ht_key[h]), HT_EMPTY, id[r]);
              if (old == HT_EMPTY) {
                const uint32_t d = atomicAdd(&sm.ndist, 1u);
                if (d < DMAX) { sm.key[d] = id[r]; sm.slot[d] = static_cast<uint16_t>(h); }
                placed = true;
                break;
              }
              if (old == id[r]) { placed = true; break; }
            }
            h = (h + 1) & (HT - 1);
            // (a table that already holds too many is not searched to its end: a unit that fails costs what its reads do)
            if ((probe & 7) == 7 && __hip_atomic_load(&sm.ndist, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > DMAX) break;
          }
        }
        full |= !placed;
      }
      at[r] = h;
    }
    if (full) atomicOr(&sm.fallback, 1u);
  }
#pragma unroll
  for (int r = 0; r < KPT; ++r)
    if (r * NT + tid < m) at[r] |= atomicAdd(&sm.ht_cnt[at[r]], 1u) << PLACE_AT;
  __syncthreads();
  const uint32_t D = sm.ndist;
  if (sm.fallback || D > DMAX) {
    if (tid == 0) unit_to_general(A, t);
    return;
  }
  // Units take the room for their rows from their task's, not from that of their own launches: a bucket of rarely launched
  // kernels has more rows than its launches would leave room for.
  // (for an address that is the same in the whole wave the compiler reads the answer of the atomic into a scalar at once, and
  // the workgroup waits for it at the next barrier)
  uint32_t rows_before = 0;
  if (tid == 0) {
    uint32_t which = t;
    asm volatile("" : "+v"(which));
    rows_before = atomicAdd(&A.staged[which], D);
  }

  // ---- 2. group by ID --------------------------------------------------------------------------
  const uint32_t share = max_u32(2 * m / NW, UNIT_SHARE_MIN);   // (fewer than NW IDs have more launches)
  if (w == 0) {
    uint32_t launches = 0, ids = 0;
    for (uint32_t part = 0; part < 2; ++part) {
      for (uint32_t j0 = 0; j0 < D; j0 += WAVE) {
        const uint32_t j = j0 + lane, s = j < D ? sm.slot[j] : 0u, c = j < D ? sm.ht_cnt[s] : 0u;
        const bool here = j < D && (c > share) == (part == 0);
        const uint32_t incl = wave_incl_scan_u32(here ? c : 0u);
        const uint64_t all = ballot(here);
        if (here) {
          sm.first[s] = static_cast<uint16_t>(launches + incl - c);
          sm.order[ids + popc_below(all)] = static_cast<uint16_t>(j);
        }
        launches += read_lane_u32(incl, WAVE - 1);
        ids += popc64(all);
      }
      if (part == 0 && lane == 0) { sm.n_shared = ids; sm.shared_launches = launches; }
    }
  } else if (w == 1 && lane < 2 * NW) {
    auto& h = sm.shared[lane / 2][lane & 1u];
    h.t = Tally{0, NONE32, 0, 0};
    if (lane == 0) sm.more = 0;
  }
  {   // rank of every ID: eight lanes count the smaller ones
    constexpr uint32_t RL = 8;
    for (uint32_t j0 = 0; j0 < D; j0 += NT / RL) {   // (trip count is the same for every thread)
      const uint32_t j = j0 + tid / RL;
      const uint64_t k = sm.key[j < D ? j : 0u];
      uint32_t below = 0;
      for (uint32_t i = tid % RL; i < D; i += RL) below += sm.key[i] < k ? 1u : 0u;
      below += dpp_move<0xB1>(below);
      below += dpp_move<0x4E>(below);
      below += dpp_move<0x141>(below);
      if (j < D && tid % RL == 0) sm.rank[j] = static_cast<uint16_t>(below);
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    if (r * NT + tid < m) {
      const uint32_t to = sm.first[at[r] & (HT - 1)] + (at[r] >> PLACE_AT);
      sm.u.val[0][to] = ev[r];
      sm.u.val[1][to] = gv[r];
    }
  }
  if (tid == 0) { sm.first_row = rows_before; A.ustage[unit] = rows_before; }
  __syncthreads();
  const uint32_t row0 = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(sm.first_row)));
  if (row0 + D > stage_room(task_len)) {
    if (tid == 0) unit_to_general(A, t);
    return;
  }

  // ---- 3. rows ---------------------------------------------------------------------------------
  const uint32_t n_shared = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(sm.n_shared)));
  auto stage = [&](uint32_t j, uint32_t array, const Picked& p) {   // (one lane)
    uint64_t* row = staged_row(A.stage_a, A.stage_b, base, task_len, row0 + sm.rank[j]);
    uint64_t* half = row + (array ? 8 : 2);
    half[0] = p.count; half[1] = p.sum; half[2] = p.min; half[3] = p.max; half[4] = p.p50; half[5] = p.p95;
    row += array ? 14 : 0;
    row[0] = array ? 0 : sm.key[j];
    row[1] = array ? 0 : t;
  };
  if (n_shared) {
    // Half a wave for the execution times, half for the idle times.  Wave w takes launches [begin, end) of the shared IDs'.
    constexpr uint32_t GW = 32;
    const uint32_t array = lane / GW, g = lane & (GW - 1);
    const uint32_t launches = sm.shared_launches, each = (launches + NW - 1) / NW;
    const uint32_t begin = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(min_u32(w * each, launches))));
    const uint32_t end = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(min_u32(w * each + each, launches))));
    auto parts = [&](auto use) {   // use(place in order, the group's samples, how many)
      uint32_t at = begin, before = 0;
      for (uint32_t h = 0; h < n_shared && at < end; ++h) {
        const uint32_t past = before + static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(sm.ht_cnt[sm.slot[sm.order[h]]])));
        if (at < past) {
          const uint32_t to = min_u32(end, past);
          use(h, sm.u.val[array] + at, to - at);
          at = to;
        }
        before = past;
      }
    };
    if (w < n_shared) clear_hist(sm.v.hist[w]);
    parts([&](uint32_t h, const uint32_t* v, uint32_t n) {
      LaneTally lane_tally;
      each_sample<GW>(v, n, n, n, [&](uint32_t x) { lane_tally.add(x); });
      const Tally x = lane_tally.of_group<GW>();
      if (g == 0) {
        Tally& q = sm.shared[h][array].t;
        atomicAdd(&q.count, x.count);
        atomicMin(&q.min, x.min);
        atomicMax(&q.max1, x.max1);
        atomicAdd(reinterpret_cast<unsigned long long*>(&q.sum), static_cast<unsigned long long>(x.sum));
      }
    });
    __syncthreads();
    parts([&](uint32_t h, const uint32_t* v, uint32_t n) {
      add_first(window_of<GW>(sm.shared[h][array].t), v, n, n, n, sm.v.hist[h] + array * (PICK_HIST / 2));
    });
    __syncthreads();
    auto& own = sm.shared[w < n_shared ? w : 0u][array];
    Range r50, r95;
    if (w < n_shared) first_ranges(window_of<GW>(own.t), sm.v.hist[w], own.t.count, r50, r95);
    for (uint32_t round = 1;; ++round) {
      if (w < n_shared) {
        if (g == 0) { own.r50 = r50; own.r95 = r95; }
        const bool wide = ballot(r50.wide(GW) || r95.wide(GW)) != 0;
        if (wide && lane == 0) sm.more = round;
        if (wide) clear_hist(sm.v.hist[w]); else clear_lists<GW>(sm.v.hist[w]);
      }
      __syncthreads();
      if (sm.more != round) break;   // (the same for all threads: written before the barrier, and not before the next one)
      parts([&](uint32_t h, const uint32_t* v, uint32_t n) {
        const auto& q = sm.shared[h][array];
        const Range q50 = q.r50, q95 = q.r95;
        if (ballot(q50.wide(GW) || q95.wide(GW))) add_cut<GW>(q50, q95, v, n, n, n, sm.v.hist[h] + array * (PICK_HIST / 2));
      });
      __syncthreads();
      if (w < n_shared) narrow<GW>(sm.v.hist[w], r50, r95);
    }
    parts([&](uint32_t h, const uint32_t* v, uint32_t n) {
      const auto& q = sm.shared[h][array];
      const Range q50 = q.r50, q95 = q.r95;
      if (ballot(q50.width || q95.width)) add_lists<GW>(q50, q95, v, n, n, n, sm.v.hist[h] + array * (PICK_HIST / 2));
    });
    __syncthreads();
    if (w < n_shared) {
      uint32_t v50, v95;
      rank_lists<GW>(sm.v.hist[w] + array * (PICK_HIST / 2), r50, r95, v50, v95);
      const bool some = own.t.count != 0;
      const Picked p{own.t.count, some ? own.t.min : 0u, some ? own.t.max1 - 1 : 0u, r50.width ? v50 : r50.lo, r95.width ? v95 : r95.lo, own.t.sum};
      if (g == 0) stage(sm.order[w], array, p);
    }
  }
  auto rows = [&](auto width) {
    constexpr uint32_t GW = decltype(width)::value, IDS = WAVE / (2 * GW);
    const uint32_t array = (lane / GW) & 1u;
    for (uint32_t i0 = n_shared + w * IDS; i0 < D; i0 += NW * IDS) {
      const uint32_t i = i0 + lane / (2 * GW);
      const bool live = i < D;
      const uint32_t j = sm.order[live ? i : i0], s = sm.slot[j], n = live ? sm.ht_cnt[s] : 0u;
      const uint32_t n0 = read_lane_u32(n, 0), n1 = IDS == 2 ? read_lane_u32(n, 2 * GW) : n0;
      static_assert(IDS <= 2, "IDs that a wave takes at a time");
      const Picked p = pick_group<GW>(sm.u.val[array] + sm.first[s], n, min_u32(n0, n1), max_u32(n0, n1), sm.v.hist[w]);
      if (live && (lane & (GW - 1)) == 0) stage(j, array, p);
    }
  };
  if (m - sm.shared_launches >= (D - n_shared) * 128) rows(std::integral_constant<uint32_t, 32>{});
  else rows(std::integral_constant<uint32_t, 16>{});
  if (tid == 0) A.dcount[unit] = D;
}

template <int NT, int KPT, int DMAX, int WPE>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE, 8)))
k_unit_sorted(const FusedArgs A) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if (A.ctrl->status & ERR_OFFSETS) return;
  // (neighbours in the list, whose runs lie next to each other in every tile, run on the same die and share its L2: with lists of
  // the percentile step made cheaper as well, 2184 -> 1891 us for the units of 8192 launches of 256 tasks of 1,048,576)
  const uint32_t units = *A.count;
  if (blockIdx.x >= xcd_grid(units)) return;
  const uint32_t item = xcd_item(blockIdx.x, units);
  if (item >= units) return;
  unit_sorted(A, A.list[item], *reinterpret_cast<UnitSmem<NT, KPT, DMAX>*>(smem_raw));
}

}  // namespace fikit
