// Units that k_unit_sorted does not take: an ID bucket of a long task that a few frequent Kernel IDs fill with more launches
// than a workgroup's registers hold (skewed traces: some kernel is launched over and over), and every bucket of a task of more
// than UNIT_RUNS_MAX tiles, down to buckets of a single launch.  One workgroup streams the bucket's launches as often as it
// needs; nothing is sorted.
//
//   1. The bucket's runs (one per tile) are read once: IDs are found in an LDS table, count / sum / min / max per ID (Section
//      3.2: sum / count = SK_j, SG_j) are gathered, and the launches are written back packed: (execution time, idle time) and
//      the ID's table slot, 10 bytes each.
//   2. Nearest-rank p50 / p95 (statistics of the same samples): a histogram per (ID, array) over the ID's own value range, on
//      the scale of pick_group and with as many bins as the ID has samples, gives the bin of each wanted rank.  The samples of
//      that bin only are then listed and ranked if they are few, else counted by their offset in the bin, again if a bin of that
//      is still more than one value wide.  Two passes over the packed launches as a rule.
//
// What bounds it: a compute unit's share of memory (the largest bucket is one workgroup's), and in the first pass the
// same-address LDS atomics that one frequent ID causes: every wave therefore keeps the sums of the ID it meets most in
// registers.  A bucket of 227,000 launches of which one ID has nearly all takes 250 us in step 1 and 150 us in each pass of step 2.
// (The launches of other IDs taken from all of a wave's runs together, or once there are 64 of them: no change.)  With bins shared
// out evenly and no lists three or four passes were needed: the streamed units of 64 tasks of 1,048,576 launches, Zipf over 4096
// IDs, 975 us, now 690; 16 tasks of 1,000,000 with equal execution times (nothing to search then) 2020 -> 1152 us for the call.
#pragma once

#include "common.hip.h"
#include "select_kernels.hip.h"
#include "task_kernels.hip.h"
#include "unit_kernels.hip.h"

namespace fikit {

constexpr int SU_THREADS = 1024, SU_WAVES = SU_THREADS / WAVE;
constexpr uint32_t SU_DMAX = 256, SU_HT = 2 * SU_DMAX;   // IDs of a bucket, slots of its ID table
constexpr uint32_t SU_HIST = 24576;                      // words of the histograms (96 KB of the 160 KB)
constexpr uint32_t SU_RUNS = 8;                          // runs a wave reads at a time: 16 loads in flight per lane
constexpr uint32_t SU_KPT = 4;                           // packed launches a lane reads at a time
constexpr uint32_t SU_BITS_MAX = 11;

struct StreamSmem {
  uint64_t ht_key[SU_HT], esum[SU_HT], gsum[SU_HT];
  uint32_t cnt[SU_HT], gcnt[SU_HT], emin[SU_HT], emax[SU_HT], gmin[SU_HT], gmax[SU_HT];
  uint4 sel[2][SU_HT];          // by array and slot: low end of the ID's window (a value or on the scale), how it is cut and the rank (su_bin), the bins of p50 and p95
  uint16_t room[2][SU_HT];      // by array and slot: first word of its histogram
  uint32_t base[4][SU_DMAX];    // by 2 * array + percentile and rank: where the bin searched next begins (a value) ...
  uint32_t rest[4][SU_DMAX];    // ... the wanted rank among the samples from there on ...
  uint32_t width[4][SU_DMAX];   // ... how many values further it ends ...
  uint32_t has[4][SU_DMAX];     // ... its samples ...
  uint8_t fine[4][SU_DMAX];     // ... the shift that cuts it into bins, or SU_LISTED ...
  uint16_t part[4][SU_DMAX];    // ... first word of those bins or of the list (its length is the word before it) ...
  uint8_t log2n[4][SU_DMAX];    // ... and log2 of the bins
  uint16_t slot_of[SU_DMAX];    // rank -> slot
  uint32_t aux[SU_WAVES];
  uint32_t ndist, fallback, filled, again, first_row, given_up;
  union {
    uint32_t hist[SU_HIST];
    struct { uint64_t ckey[SU_DMAX]; uint16_t cslot[SU_DMAX]; } tmp;
  } u;
};
static_assert(sizeof(StreamSmem) <= 160 * 1024, "fits a compute unit's LDS");
using LargeSmem = UnitSmem<SU_THREADS, FUSE_MAX / SU_THREADS, UNIT_DMAX_LARGE>;
constexpr size_t UNIT_LARGE_LDS = sizeof(StreamSmem) > sizeof(LargeSmem) ? sizeof(StreamSmem) : sizeof(LargeSmem);
static_assert(UNIT_LARGE_LDS + 16 <= 160 * 1024, "fits a compute unit's LDS, with the ticket");
constexpr uint32_t SU_NO_BIN = ~0u;
constexpr uint32_t SU_LIST = 31, SU_LISTED = 0xffu;      // samples of a bin that are listed and ranked, not counted again
static_assert(SU_HIST <= 0xffffu && 4 * SU_DMAX * (SU_LIST + 1) > SU_HIST, "places in the histograms fit 16 bits; lists may have to be shorter");

__device__ __forceinline__ uint32_t su_log2_above(uint32_t v) { return v > 1 ? 32u - static_cast<uint32_t>(__builtin_clz(v - 1)) : 0u; }   // 2^this >= v

// Shares the histogram space among items, thread i's being 2^want words unless that is more than the space holds: then the
// largest are cut, all to the same size.  Every thread calls, with SU_NONE for no item; gives the first word and the log2 granted.
constexpr uint32_t SU_NONE = 32;
__device__ __forceinline__ uint32_t su_share(uint32_t want, uint32_t* aux, uint32_t& granted) {
  for (uint32_t most = SU_BITS_MAX;; --most) {
    granted = want < most ? want : most;
    uint32_t total;
    const uint32_t at = block_excl_scan<SU_THREADS>(want == SU_NONE ? 0u : 1u << granted, aux, total);
    if (total <= SU_HIST || most == 0) return at;   // (at most SU_THREADS items: one word each always fits)
  }
}
static_assert(4 * SU_DMAX <= SU_THREADS && SU_THREADS <= SU_HIST, "a thread per item");

// The bin of hist[0 .. bins) that holds the rank k (0-based; the bins' counts sum to more than k), the rank inside it and its
// samples.  Called by whole waves with the same arguments; the results are in all lanes.
__device__ __forceinline__ void su_find(const uint32_t* hist, uint32_t bins, uint32_t k, uint32_t& bin, uint32_t& inside, uint32_t& count) {
  const uint32_t lane = lane_id();
  const uint32_t per = bins > WAVE ? bins / WAVE : 1u;   // (bins is a power of two)
  uint32_t mine = 0;
  if (lane * per < bins)
    for (uint32_t b = 0; b < per; ++b) mine += hist[lane * per + b];
  const uint32_t incl = wave_incl_scan_u32(mine);
  const uint64_t holds = ballot(k < incl);
  const int leader = holds ? __builtin_ctzll(holds) : WAVE - 1;
  uint32_t at = 0, in = 0, has = 0;
  if (static_cast<int>(lane) == leader) {
    uint32_t cum = incl - mine;
    for (uint32_t b = 0; b < per; ++b) {
      const uint32_t c = hist[lane * per + b];
      if (k < cum + c) { at = lane * per + b; in = k - cum; has = c; break; }
      cum += c;
    }
  }
  bin = __shfl(at, leader, WAVE);
  inside = __shfl(in, leader, WAVE);
  count = __shfl(has, leader, WAVE);
}

__device__ __forceinline__ uint32_t su_scale(uint32_t v) { return pick_scale(__uint2float_rn(v)); }
// The bin of a value by its ID's window (StreamSmem::sel), whose word y is shift | linear << 7 | rank << 8.
constexpr uint32_t SU_LINEAR = 0x80u;
__device__ __forceinline__ uint32_t su_bin(const uint4& window, uint32_t v) {
  return ((window.y & SU_LINEAR ? v : su_scale(v)) - window.x) >> (window.y & 31u);
}

// Slot of an ID in the table (entered if it is new), or SU_HT if the table holds too many.
__device__ __forceinline__ uint32_t su_slot(StreamSmem& sm, uint64_t id) {
  uint32_t h = (static_cast<uint32_t>(id >> 32) ^ static_cast<uint32_t>(id)) & (SU_HT - 1);
  if (id == HT_EMPTY) return SU_HT;
  for (uint32_t probe = 0; probe < SU_HT; ++probe) {
    const uint64_t k = __hip_atomic_load(&sm.ht_key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (k == id) return h;
    if (k == HT_EMPTY) {
      const uint64_t old = atomicCAS(reinterpret_cast<unsigned long long*>(&sm.ht_key[h]), HT_EMPTY, id);
      if (old == HT_EMPTY) return atomicAdd(&sm.ndist, 1u) < SU_DMAX ? h : SU_HT;
      if (old == id) return h;
    }
    h = (h + 1) & (SU_HT - 1);
    if ((probe & 7) == 7 && __hip_atomic_load(&sm.ndist, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > SU_DMAX) break;
  }
  return SU_HT;
}

// pack_kg, pack_slot: two 8-byte arrays that only the sort would use.  A unit writes the slices of both that belong to its own
// launches (ustart, ulen) and nothing else: other tasks may have handed their values over to the sort there already.
// Another unit may give the task up to the sort at any time (the launches of smaller units have run, but units of more than
// FUSE_MID_MAX launches and other streamed ones run beside it): the task's flag is looked at along the way, and the unit leaves.
// fikit_profile, us, flag looked at at the start only / along the way, with 600 IDs in a bucket of 12,000 launches beside one ID
// with most of the others: a task of 300,000 launches 1500 / 1185, 16 of them 1830 / 1520, 64 of 1,000,000 11,150 / 9550;
// profiles of which no task is given up are the same.
// PART: what of the launches is looked at.
enum : int { SU_BOTH = 0, SU_EXEC = 1, SU_IDLE = 2 };
constexpr uint32_t SU_UNPLACED = ~0u;
template <int PART>
__device__ __forceinline__ void unit_streamed(const FusedArgs& A, uint32_t unit, uint2* __restrict__ pack_kg_all,
                                              int64_t* __restrict__ pack_slot_all, StreamSmem& sm) {
  constexpr bool EXEC = PART != SU_IDLE, IDLE = PART != SU_EXEC;
  const uint32_t m = A.ulen[unit], t = A.utask[unit];
  const uint64_t base = A.ustart[unit];
  // (the two parts of a unit pack for themselves, into a half of its slices each)
  uint2* __restrict__ pack_kg = pack_kg_all + base;
  uint32_t* __restrict__ pack_v = reinterpret_cast<uint32_t*>(pack_kg) + (PART == SU_IDLE ? m : 0u);
  uint16_t* __restrict__ pack_slot = reinterpret_cast<uint16_t*>(pack_slot_all + base) + (PART == SU_IDLE ? 2 * static_cast<uint64_t>(m) : 0u);
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t w = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(tid / WAVE)));

  for (uint32_t s = tid; s < SU_HT; s += SU_THREADS) {
    sm.ht_key[s] = HT_EMPTY; sm.esum[s] = 0; sm.gsum[s] = 0; sm.cnt[s] = 0; sm.gcnt[s] = 0;
    sm.emin[s] = ~0u; sm.emax[s] = 0; sm.gmin[s] = ~0u; sm.gmax[s] = 0;
  }
  auto given_up = [&]() -> uint32_t {   // (nothing waits for the answer where it is asked)
    return __hip_atomic_load(&A.mflag[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 0u : 1u;
  };
  if (tid == 0) { sm.ndist = 0; sm.filled = 0; sm.fallback = given_up(); }
  __syncthreads();

  // ---- 1. gather the bucket's runs --------------------------------------------------------------------------------
  {
    const uint32_t ub = A.ubuckets[unit], d0 = ub & 0xffffu, d1 = ub >> 16;
    const uint32_t tp = A.tile_prefix[t], tiles_t = A.tile_prefix[t + 1] - tp;
    const uint32_t task_start = static_cast<uint32_t>(A.off[t]);
    const uint16_t* b_lo = A.bound + static_cast<uint64_t>(tp) * (256 + 1) + static_cast<uint64_t>(d0) * tiles_t;
    const uint16_t* b_hi = A.bound + static_cast<uint64_t>(tp) * (256 + 1) + static_cast<uint64_t>(d1) * tiles_t;
    uint64_t dom_id = HT_EMPTY, dom_es = 0, dom_gs = 0;   // the ID this wave met most at the start, and its sums so far
    uint32_t dom_slot = SU_HT, dom_c = 0, dom_gc = 0, dom_en = ~0u, dom_ex = 0, dom_gn = ~0u, dom_gx = 0;
    for (uint32_t j0 = w * SU_RUNS; j0 < tiles_t; j0 += SU_WAVES * SU_RUNS) {
      if (__hip_atomic_load(&sm.fallback, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
      uint32_t lo = 0, c = 0;
      const uint32_t j = j0 + lane;
      if (lane < SU_RUNS && j < tiles_t) { lo = b_lo[j]; c = static_cast<uint32_t>(b_hi[j]) - lo; }
      const uint32_t incl = wave_incl_scan_u32(c);   // (lanes from SU_RUNS on add nothing)
      const uint32_t total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), WAVE - 1));
      uint32_t place = 0;
      if (lane == 0) place = atomicAdd(&sm.filled, total);
      place = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(place)));
      uint32_t rc[SU_RUNS], rat[SU_RUNS], rto[SU_RUNS], longest = 0;
#pragma unroll
      for (uint32_t r = 0; r < SU_RUNS; ++r) {
        rc[r] = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(c), static_cast<int>(r)));
        rat[r] = task_start + (j0 + r) * A.tile_len + static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(lo), static_cast<int>(r)));
        rto[r] = place + static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), static_cast<int>(r))) - rc[r];
        longest = rc[r] > longest ? rc[r] : longest;
      }
      for (uint32_t x0 = 0; x0 < longest; x0 += WAVE) {
        if (__hip_atomic_load(&sm.fallback, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
        const uint32_t leave = tid == 0 ? given_up() : 0u;
        const uint32_t x = x0 + lane;
        uint64_t id[SU_RUNS];
        uint2 kg[SU_RUNS];
#pragma unroll
        for (uint32_t r = 0; r < SU_RUNS; ++r) {
          id[r] = HT_EMPTY;
          kg[r] = make_uint2(0, NONE32);
          if (x < rc[r]) { id[r] = A.part_id[rat[r] + x]; kg[r] = A.part_kg[rat[r] + x]; }
        }
        if (dom_slot == SU_HT) {
          // the most frequent among four of the first 64 launches (a guess that costs nothing if it is wrong)
          uint32_t most = 0;
          for (uint32_t q = 0; q < WAVE; q += WAVE / 4) {
            const uint64_t cand = read_lane_u64(id[0], q);
            const uint32_t have = cand == HT_EMPTY ? 0u : static_cast<uint32_t>(__popcll(ballot(id[0] == cand)));
            if (have > most) { most = have; dom_id = cand; }
          }
          if (most > 0) dom_slot = su_slot(sm, dom_id);
          if (ballot(dom_slot == SU_HT)) dom_slot = SU_HT;   // (the lane that entered one too many knows; the same for the wave)
        }
#pragma unroll
        for (uint32_t r = 0; r < SU_RUNS; ++r) {
          if (x < rc[r]) {
            const uint32_t e = kg[r].x, g = kg[r].y;
            uint32_t s = dom_slot;
            if (id[r] == dom_id && dom_slot != SU_HT) {
              if (EXEC) {
                ++dom_c; dom_es += e;
                dom_en = e < dom_en ? e : dom_en; dom_ex = e > dom_ex ? e : dom_ex;
              }
              if (IDLE && g != NONE32) {
                ++dom_gc; dom_gs += g;
                dom_gn = g < dom_gn ? g : dom_gn; dom_gx = g > dom_gx ? g : dom_gx;
              }
            } else {
              s = su_slot(sm, id[r]);
              if (s == SU_HT) { atomicOr(&sm.fallback, 1u); s = 0; }
              if (EXEC) {
                atomicAdd(&sm.cnt[s], 1u);
                atomicAdd(reinterpret_cast<unsigned long long*>(&sm.esum[s]), static_cast<unsigned long long>(e));
                atomicMin(&sm.emin[s], e); atomicMax(&sm.emax[s], e);
              }
              if (IDLE && g != NONE32) {
                atomicAdd(&sm.gcnt[s], 1u);
                atomicAdd(reinterpret_cast<unsigned long long*>(&sm.gsum[s]), static_cast<unsigned long long>(g));
                atomicMin(&sm.gmin[s], g); atomicMax(&sm.gmax[s], g);
              }
            }
            if (rto[r] + x < m) {   // (always: the unit's length is the sum of its runs)
              if (PART == SU_BOTH) pack_kg[rto[r] + x] = kg[r]; else pack_v[rto[r] + x] = EXEC ? e : g;
              pack_slot[rto[r] + x] = static_cast<uint16_t>(s);
            }
          }
        }
        if (leave) atomicOr(&sm.fallback, 1u);
      }
    }
    if (dom_slot != SU_HT) {   // (the same in the whole wave)
      const uint32_t c = wave_sum_u32(dom_c), gc = wave_sum_u32(dom_gc);
      const uint64_t es = wave_sum_u64(dom_es), gs = wave_sum_u64(dom_gs);
      const uint32_t ex = wave_max_u32(dom_ex), gx = wave_max_u32(dom_gx), en = ~wave_max_u32(~dom_en), gn = ~wave_max_u32(~dom_gn);
      if (EXEC && lane == 0 && c) {
        atomicAdd(&sm.cnt[dom_slot], c);
        atomicAdd(reinterpret_cast<unsigned long long*>(&sm.esum[dom_slot]), static_cast<unsigned long long>(es));
        atomicMin(&sm.emin[dom_slot], en); atomicMax(&sm.emax[dom_slot], ex);
      }
      if (IDLE && lane == 0 && gc) {
        atomicAdd(&sm.gcnt[dom_slot], gc);
        atomicAdd(reinterpret_cast<unsigned long long*>(&sm.gsum[dom_slot]), static_cast<unsigned long long>(gs));
        atomicMin(&sm.gmin[dom_slot], gn); atomicMax(&sm.gmax[dom_slot], gx);
      }
    }
  }
  __syncthreads();
  const uint32_t D = sm.ndist;
  const uint64_t task_start = A.off[t];
  const uint32_t task_len = static_cast<uint32_t>(A.off[t + 1] - task_start);
  const bool fits = !sm.fallback && D <= SU_DMAX && sm.filled == m;
  if (tid == 0) {
    sm.given_up = given_up();
    if (PART == SU_BOTH) {
      sm.first_row = fits ? atomicAdd(&A.staged[t], D) : 0u;
      A.ustage[unit] = sm.first_row;
    } else {   // the rows are where the part that came first has put them (if both come at once, the other's room is left empty)
      uint32_t at = __hip_atomic_load(&A.ustage[unit], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (at == SU_UNPLACED && fits) {
        const uint32_t room = atomicAdd(&A.staged[t], D), held = atomicCAS(&A.ustage[unit], SU_UNPLACED, room);
        at = held == SU_UNPLACED ? room : held;
      }
      sm.first_row = fits ? at : 0u;
    }
  }
  __syncthreads();
  if (sm.given_up) return;   // (the same for all threads)
  const uint32_t row0 = sm.first_row;
  if (!fits || row0 + D > stage_room(task_len)) {
    if (tid == 0) unit_to_general(A, t);
    return;
  }

  // ---- rank the distinct IDs; where each value range is searched --------------------------------------------------
  {
    uint32_t total;
    const bool used = tid < SU_HT && sm.ht_key[tid < SU_HT ? tid : 0] != HT_EMPTY;
    const uint32_t at = block_excl_scan<SU_THREADS>(used ? 1u : 0u, sm.aux, total);
    if (used) { sm.u.tmp.ckey[at] = sm.ht_key[tid]; sm.u.tmp.cslot[at] = static_cast<uint16_t>(tid); }
    __syncthreads();
    if (tid < D) {
      const uint64_t k = sm.u.tmp.ckey[tid];
      uint32_t rank = 0;
      for (uint32_t i = 0; i < D; ++i) rank += sm.u.tmp.ckey[i] < k;
      sm.slot_of[rank] = sm.u.tmp.cslot[tid];
    }
    __syncthreads();
  }
  {
    const bool mine = tid < (PART == SU_BOTH ? 2 * D : D);
    const uint32_t second = mine && tid >= D ? 1u : 0u, arr = PART == SU_BOTH ? second : PART == SU_EXEC ? 0u : 1u;
    const uint32_t j = mine ? tid - second * D : 0u, s = sm.slot_of[j];
    const uint32_t n = arr ? sm.gcnt[s] : sm.cnt[s];
    uint32_t bins_log2;
    const uint32_t at = su_share(mine ? su_log2_above(n) : SU_NONE, sm.aux, bins_log2);
    if (mine) {
      // (equal steps of the value where the range is narrow, as in pick_group)
      const uint32_t lo = n ? (arr ? sm.gmin[s] : sm.emin[s]) : 0u, by_value = n ? (arr ? sm.gmax[s] : sm.emax[s]) - lo : 0u;
      const uint32_t by_scale = su_scale(lo + by_value) - su_scale(lo);
      const bool linear = (by_value >> bins_log2) == 0 || (by_scale >> bins_log2) == 0;
      sm.sel[arr][s] = make_uint4(linear ? lo : su_scale(lo), cut_shift(linear ? by_value : by_scale, bins_log2) | (linear ? SU_LINEAR : 0u) | (j << 8),
                                  SU_NO_BIN, SU_NO_BIN);
      sm.room[arr][s] = static_cast<uint16_t>(at);
      sm.log2n[arr][j] = static_cast<uint8_t>(bins_log2);
    }
  }
  for (uint32_t i = tid; i < SU_HIST; i += SU_THREADS) sm.u.hist[i] = 0;
  if (tid == 0) sm.again = 0;
  __syncthreads();

  // ---- 2. nearest-rank percentiles -------------------------------------------------------------------------------
  const uint32_t leave = tid == 0 ? given_up() : 0u;
  for (uint32_t i0 = 0; i0 < m; i0 += SU_KPT * SU_THREADS) {
    uint2 kg[SU_KPT];
    uint32_t sl[SU_KPT];
#pragma unroll
    for (uint32_t u = 0; u < SU_KPT; ++u) {
      const uint32_t i = i0 + u * SU_THREADS + tid;
      kg[u] = make_uint2(0, NONE32); sl[u] = 0;
      if (i < m) {
        if (PART == SU_BOTH) kg[u] = pack_kg[i]; else (EXEC ? kg[u].x : kg[u].y) = pack_v[i];
        sl[u] = pack_slot[i];
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < SU_KPT; ++u) {
      if (i0 + u * SU_THREADS + tid < m) {
        if (EXEC) {
          const uint4 se = sm.sel[0][sl[u]];
          atomicAdd(&sm.u.hist[sm.room[0][sl[u]] + su_bin(se, kg[u].x)], 1u);
        }
        if (IDLE && kg[u].y != NONE32) {
          const uint4 sg = sm.sel[1][sl[u]];
          atomicAdd(&sm.u.hist[sm.room[1][sl[u]] + su_bin(sg, kg[u].y)], 1u);
        }
      }
    }
  }
  if (leave) sm.given_up = 1;
  __syncthreads();
  if (sm.given_up) return;
  const uint32_t q_first = EXEC ? 0u : 2 * D, q_past = IDLE ? 4 * D : 2 * D;
  for (uint32_t q = q_first + w; q < q_past; q += SU_WAVES) {   // (2 * array + percentile, rank); a wave each
    const uint32_t ap = q / D, j = q - ap * D, arr = ap >> 1, s = sm.slot_of[j];
    const uint32_t n = arr ? sm.gcnt[s] : sm.cnt[s];
    if (n == 0) {
      if (lane == 0) sm.base[ap][j] = 0;
      continue;
    }
    const uint32_t k = static_cast<uint32_t>(rank_index(ap & 1u ? 95 : 50, n));
    uint32_t bin, inside, has;
    su_find(sm.u.hist + sm.room[arr][s], 1u << sm.log2n[arr][j], k, bin, inside, has);
    if (lane == 0) {
      const uint4 sel = sm.sel[arr][s];
      const uint32_t sh = sel.y & 31u, mn = arr ? sm.gmin[s] : sm.emin[s], mx = arr ? sm.gmax[s] : sm.emax[s], t = sel.x + (bin << sh);
      // the values of the bin, both ends included
      const bool linear = (sel.y & SU_LINEAR) != 0;
      const uint32_t first = linear ? t : max_u32(pick_scale_low(t), mn);
      const uint32_t last = linear ? (mx - t < 1u << sh ? mx : t + (1u << sh) - 1) : min_u32(pick_scale_low(t + (1u << sh)) - 1, mx);
      sm.base[ap][j] = first;
      sm.rest[ap][j] = inside;
      sm.width[ap][j] = last - first;
      sm.has[ap][j] = has;
      if (last != first) {   // (else found)
        (ap & 1u ? sm.sel[arr][s].w : sm.sel[arr][s].z) = bin;
        atomicOr(&sm.again, 1u);
      }
    }
  }
  __syncthreads();
  while (sm.again) {   // (the same for all threads: changed behind the barriers of su_share and in front of the loop's last)
    // Room for every bin that is searched: a list if its samples are few, bins one value wide if there are so many words, fewer
    // and wider ones if not.
    {
      const uint32_t ap = tid / SU_DMAX, j = tid % SU_DMAX, arr = ap >> 1, s = j < D ? sm.slot_of[j] : 0u;
      const bool searched = j < D && (arr ? IDLE : EXEC) && (ap & 1u ? sm.sel[arr][s].w : sm.sel[arr][s].z) != SU_NO_BIN;
      const uint32_t width = searched ? sm.width[ap][j] : 0u, has = searched ? sm.has[ap][j] : 0u;
      const bool list = searched && has <= SU_LIST && width != 0;
      uint32_t granted;
      const uint32_t at = su_share(!searched ? SU_NONE : list ? su_log2_above(has + 1) : width < 1u << SU_BITS_MAX ? su_log2_above(width + 1) : SU_BITS_MAX,
                                   sm.aux, granted);
      if (searched) {
        sm.part[ap][j] = static_cast<uint16_t>(at);
        sm.log2n[ap][j] = static_cast<uint8_t>(granted);
        sm.fine[ap][j] = static_cast<uint8_t>(list && has < 1u << granted ? SU_LISTED : cut_shift(width, granted));
      }
    }
    for (uint32_t i = tid; i < SU_HIST; i += SU_THREADS) sm.u.hist[i] = 0;
    if (tid == 0) sm.again = 0;
    __syncthreads();
    // a sample of a bin that is searched: listed, or counted by its offset from where the search has got to
    auto count = [&](uint32_t arr, uint32_t v, uint32_t slot) {
      const uint4 sel = sm.sel[arr][slot];
      const uint32_t bin = su_bin(sel, v), j = sel.y >> 8;
#pragma unroll
      for (uint32_t p = 0; p < 2; ++p) {
        if (bin == (p ? sel.w : sel.z)) {
          const uint32_t ap = 2 * arr + p, past = v - sm.base[ap][j], sh = sm.fine[ap][j];
          uint32_t* mine = sm.u.hist + sm.part[ap][j];
          if (past <= sm.width[ap][j]) {
            if (sh == SU_LISTED) mine[1 + (atomicAdd(&mine[0], 1u) & SU_LIST)] = v;
            else atomicAdd(&mine[past >> sh], 1u);
          }
        }
      }
    };
    for (uint32_t i0 = 0; i0 < m; i0 += SU_KPT * SU_THREADS) {
      uint2 kg[SU_KPT];
      uint32_t sl[SU_KPT];
#pragma unroll
      for (uint32_t u = 0; u < SU_KPT; ++u) {
        const uint32_t i = i0 + u * SU_THREADS + tid;
        kg[u] = make_uint2(0, NONE32); sl[u] = 0;
        if (i < m) {
          if (PART == SU_BOTH) kg[u] = pack_kg[i]; else (EXEC ? kg[u].x : kg[u].y) = pack_v[i];
          sl[u] = pack_slot[i];
        }
      }
#pragma unroll
      for (uint32_t u = 0; u < SU_KPT; ++u) {
        if (i0 + u * SU_THREADS + tid < m) {
          if (EXEC) count(0, kg[u].x, sl[u]);
          if (IDLE && kg[u].y != NONE32) count(1, kg[u].y, sl[u]);
        }
      }
    }
    __syncthreads();
    for (uint32_t q = q_first + w; q < q_past; q += SU_WAVES) {
      const uint32_t ap = q / D, j = q - ap * D, arr = ap >> 1, s = sm.slot_of[j];
      const uint32_t searched = ap & 1u ? sm.sel[arr][s].w : sm.sel[arr][s].z;
      if (searched == SU_NO_BIN) continue;
      const uint32_t* mine = sm.u.hist + sm.part[ap][j];
      const uint32_t sh = sm.fine[ap][j];
      uint32_t bin = 0, inside = 0, has = 0;
      if (sh == SU_LISTED) {   // a lane per sample counts the smaller ones; the wanted one is the largest with at most `rest` of them
        const uint32_t n = mine[0], v = lane < n ? mine[1 + lane] : 0u;
        uint32_t smaller = 0;
        for (uint32_t i = 0; i < n; ++i) smaller += mine[1 + i] < v ? 1u : 0u;
        bin = wave_max_u32(lane < n && smaller <= sm.rest[ap][j] ? v : 0u) - sm.base[ap][j];
      } else {
        su_find(mine, 1u << sm.log2n[ap][j], sm.rest[ap][j], bin, inside, has);
        bin <<= sh;
      }
      if (lane == 0) {
        sm.base[ap][j] += bin;
        if (sh == 0 || sh == SU_LISTED) {   // found
          (ap & 1u ? sm.sel[arr][s].w : sm.sel[arr][s].z) = SU_NO_BIN;
        } else {
          sm.rest[ap][j] = inside;
          sm.width[ap][j] = min_u32(sm.width[ap][j] - bin, (1u << sh) - 1);
          sm.has[ap][j] = has;
          atomicOr(&sm.again, 1u);
        }
      }
    }
    __syncthreads();
  }

  if (tid < D) {
    const uint32_t s = sm.slot_of[tid];
    uint64_t* row = staged_row(A.stage_a, A.stage_b, task_start, task_len, row0 + tid);
    if (EXEC) {
      row[0] = sm.ht_key[s]; row[1] = t;
      row[2] = sm.cnt[s]; row[3] = sm.esum[s]; row[4] = sm.emin[s]; row[5] = sm.emax[s];
      row[6] = sm.base[0][tid]; row[7] = sm.base[1][tid];
      row[14] = 0; row[15] = 0;
    }
    if (IDLE) {
      const uint32_t gc = sm.gcnt[s];
      row[8] = gc; row[9] = sm.gsum[s]; row[10] = gc ? sm.gmin[s] : 0; row[11] = gc ? sm.gmax[s] : 0;
      row[12] = sm.base[2][tid]; row[13] = sm.base[3][tid];
    }
  }
  if (tid == 0) A.dcount[unit] = D;
}

// The streamed units and, beside them, the units of more than FUSE_MID_MAX launches: both need a compute unit's whole LDS, and the
// longest streamed units leave most of the chip to the others (64 tasks of 1,048,576 launches, Zipf over 4096 IDs: 915 us
// in a launch each, 726 us together; workgroups that stay also save the 30 us that 33,000 without a unit take to come and go).
// Workgroups stay, one per compute unit, and take units in order from a counter: streamed ones from the front of their list (the
// largest first), then from its back, then the others.
//
// One of the front's is taken by two workgroups, one for the execution times and one for the idle times, where that leaves a
// compute unit to each: all of them, or only those of more than STREAM_LONGEST launches, or none.  What a unit of 227,000
// launches takes decides the launch then, and the memory of one compute unit decides that; both workgroups find and rank the
// IDs, and nothing is waited for, but all of it together is a third more work.  Where a quarter of the launches and more is in
// units that are not streamed, these fill the chip behind the streamed ones, and none of those is taken so that is not longer,
// by a quarter, than what there is for each workgroup to do: the third more is all that would come of it.
// This launch in us, whole / in parts: 4 tasks of 1,048,576 launches, Zipf over 4096 IDs, 678 / 423, 64 of them 757 / 631 (only the
// longest), 96 of them 1001 / 1005; 16 tasks of 300,000 over 50 IDs 218 / 178, 30 of 1,000,000 649 / 517; one of 4,300,000 1700 /
// 1391; 60 of 400,000, two IDs with 0.3 of the launches each and 30 others 273 / 242; 30 of 1,000,000 over 20 IDs alike 458 / 380,
// 20 of 2,000,000 over 30 (all streamed, the others' order decides) 932 / 675.  Left whole for what else there is: 100 tasks of
// 300,000, one ID with 0.3 of the launches and 20 others 373 / 418, 128 of 1,000,000, one with 0.1 and 300 others 656 / 724, 40 of
// 2,000,000, two IDs with 0.1 each and 200 others 655 / 747.
constexpr uint64_t UNIT_LARGE_WORKGROUPS = 256;
constexpr uint32_t SU_SPLIT_PARTS = 192, SU_FILL_PART = 4;
constexpr uint32_t LARGE_TYPICAL = (FUSE_MID_MAX + FUSE_MAX) / 2;   // launches of a unit that is not streamed
__global__ void __launch_bounds__(SU_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_unit_large(const FusedArgs A, const uint32_t* __restrict__ streamed, uint32_t streamed_end, uint2* __restrict__ pack_kg_all,
             int64_t* __restrict__ pack_slot_all) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ uint32_t ticket;
  if (A.ctrl->status & ERR_OFFSETS) return;
  const uint32_t large = A.ctrl->n_class[2], front = A.ctrl->n_class[3], back = A.ctrl->n_class[4];
  const uint32_t longest = A.ctrl->n_class[5];   // units of more than STREAM_LONGEST
  const uint32_t launches = A.ctrl->n_large, for_each = launches / static_cast<uint32_t>(UNIT_LARGE_WORKGROUPS);
  const bool filled = static_cast<uint64_t>(large) * LARGE_TYPICAL >= launches / SU_FILL_PART;
  const uint32_t split_above = max_u32(2 * front <= UNIT_LARGE_WORKGROUPS ? 0u : 2 * longest <= SU_SPLIT_PARTS ? STREAM_LONGEST : ~0u,
                                       filled ? for_each + for_each / 4 : 0u);
  for (;;) {
    if (threadIdx.x == 0) ticket = atomicAdd(&A.ctrl->taken, 1u);
    __syncthreads();
    const uint32_t at = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(ticket)));
    StreamSmem& stream = *reinterpret_cast<StreamSmem*>(smem_raw);
    if (at < 2 * front) {   // (two places for each of the front's units)
      const uint32_t unit = streamed[at / 2];
      if (A.ulen[unit] > split_above) {
        if (at & 1) unit_streamed<SU_IDLE>(A, unit, pack_kg_all, pack_slot_all, stream);
        else unit_streamed<SU_EXEC>(A, unit, pack_kg_all, pack_slot_all, stream);
      } else if (!(at & 1)) {
        unit_streamed<SU_BOTH>(A, unit, pack_kg_all, pack_slot_all, stream);
      }
    } else {
      const uint32_t next = at - 2 * front;
      if (next >= back + large) return;
      if (next < back) unit_streamed<SU_BOTH>(A, streamed[streamed_end - 1 - next], pack_kg_all, pack_slot_all, stream);
      else unit_sorted<SU_THREADS, FUSE_MAX / SU_THREADS, UNIT_DMAX_LARGE>(A, A.list[next - back], *reinterpret_cast<LargeSmem*>(smem_raw));
    }
    __syncthreads();   // (the next unit's tables take the place of this one's)
  }
}

}  // namespace fikit
