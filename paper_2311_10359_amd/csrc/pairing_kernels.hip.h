// The best low-priority partner of every high-priority task among evaluated combinations (the paper's
// discussion section, "What Tasks are Suitable for Sharing a GPU").
#pragma once

#include "common.hip.h"

namespace fikit {

constexpr int PAIR_THREADS = 256;
constexpr uint64_t PAIR_MOST_GAPS = (1ull << 32) - (1ull << 24);   // a call with as many or more is refused

// The control block and start values per task (no memset: the stream may be under graph capture): the values of a task that heads
// no scenario.  The number of gaps is looked at here and not by the host, which would have to wait for it.
__global__ void k_pair_init(uint32_t n_tasks, const uint64_t* __restrict__ n_gaps, long long* __restrict__ top_filled,
                            unsigned long long* __restrict__ best_scenario, uint32_t* __restrict__ best_lp,
                            int64_t* __restrict__ best_filled, Ctrl* ctrl) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  const bool refused = n_gaps && *n_gaps >= PAIR_MOST_GAPS;
  if (t < sizeof(Ctrl) / 4) reinterpret_cast<uint32_t*>(ctrl)[t] = t == 0 && refused ? ERR_GAP_OFFSETS : 0u;
  if (t >= n_tasks || refused) return;
  top_filled[t] = INT64_MIN;
  best_scenario[t] = ~0ull;
  best_lp[t] = ~0u;
  best_filled[t] = 0;
}

// G lanes per scenario (a workgroup or a wave), which take every so-manieth one: they check the scenario, sum the time filled in
// its gaps (8 B read per gap) and raise the largest filled time seen for its high-priority task.  Bound by HBM once enough bytes
// are in flight: a lane has up to eight 16-byte reads out at a time.  From PAIR_WAVES scenarios on a wave takes one: as many
// waves as there are places for stay and look the next scenario up while they read, so that nothing but the reads themselves is
// waited for, and no barrier is met on the way (16,384 scenarios of 2047 gaps: a workgroup each 62 us = 4.3 TB/s, call 84.3 us;
// waves 57 us = 4.7 TB/s, call 79.6 us; twice as many workgroups 83.3, half as many 81.6, sixteen reads at a time 81.1, reads
// that are not to be kept 83.5). Below it, a workgroup's reads come back sooner than a wave's (40 scenarios of 4772 gaps: call
// 26.6 against 27.3 us).  Where the gaps are no more than the lanes, each reads one of them: eight guarded reads are then most
// of the instructions (200,000 scenarios of 3 gaps, call 273 us with them, 227 us without; of 30 gaps 253 and 225 us, both with
// a workgroup each). The atomic returns nothing, so nothing waits for it; looking at the word first does wait, at a word that
// all scenarios of a task share (158 us).
//
// A scenario of many more gaps than the others (PAIR_LONG times the average and more than PAIR_LONG_LEAST) is left to the end by
// its wave, and the workgroup's waves sum it up together: a wave alone decided the call.  us per call, a workgroup per
// scenario / waves alone / now: 8192 scenarios of 1000 gaps, one of 100,000 65 / 78 / 60, one of 1,000,000 202 / 364 / 191, eight
// of 1,000,000 212 / 388 / 207; 8192 of 100, 64 of 200,000 84 / 112 / 79; 20,000 of 500, one of 4,000,000 668 / 1356 / 645; 8192
// of 20,000 282 / 268 / 262.
constexpr uint64_t PAIR_WAVES = 8192, PAIR_STAY = 2048;   // (PAIR_STAY workgroups of four waves fill the chip)
constexpr uint64_t PAIR_LONG = 8, PAIR_LONG_LEAST = 8192;
constexpr uint32_t PAIR_LONGS = 256;   // of a workgroup; what is beyond stays with its wave
template <int G>
__device__ __forceinline__ uint64_t pair_lane_sum(const uint64_t* __restrict__ f, uint64_t g0, uint64_t g1, uint32_t at) {
  constexpr int READS = 8;
  uint64_t acc[2] = {0, 0};      // (sums wrap like the oracle's additions)
  if (g1 - g0 <= G) {   // few gaps: one read per lane, and few instructions
    if (at < g1 - g0) acc[0] = f[g0 + at];
  } else {
    // pairs from the first gap on that lies on a 16-byte address; the gap before them and the one behind by one lane
    const uint64_t p0 = (reinterpret_cast<uintptr_t>(f + g0) & 15) ? g0 + 1 : g0;
    const uint32_t pairs = static_cast<uint32_t>((g1 - p0) / 2);
    const ulonglong2* v = reinterpret_cast<const ulonglong2*>(f + p0);
    uint32_t i = at;
    for (; i + (READS - 1) * G < pairs; i += READS * G) {
      ulonglong2 x[READS];
#pragma unroll
      for (int k = 0; k < READS; ++k) x[k] = v[i + k * G];
#pragma unroll
      for (int k = 0; k < READS; ++k) { acc[0] += x[k].x; acc[1] += x[k].y; }
    }
    {
      ulonglong2 x[READS];
#pragma unroll
      for (int k = 0; k < READS; ++k) {
        x[k] = make_ulonglong2(0, 0);
        if (i + k * G < pairs) x[k] = v[i + k * G];
      }
#pragma unroll
      for (int k = 0; k < READS; ++k) { acc[0] += x[k].x; acc[1] += x[k].y; }
    }
    if (at == 0) {
      if (p0 > g0) acc[0] += f[g0];
      if (p0 + 2 * static_cast<uint64_t>(pairs) < g1) acc[1] += f[g1 - 1];
    }
  }
  return acc[0] + acc[1];
}
template <int G>
__global__ void __launch_bounds__(PAIR_THREADS)
k_pair_sum(const uint32_t* __restrict__ hp_task, const uint32_t* __restrict__ lp_task, uint32_t n_scen, uint32_t n_tasks,
           const uint64_t* __restrict__ gap_off, const int64_t* __restrict__ filled_ns, int64_t* __restrict__ scen_filled,
           long long* __restrict__ top_filled, Ctrl* ctrl) {
  static_assert(G == WAVE || G == PAIR_THREADS, "a wave or a workgroup");
  __shared__ uint64_t part[PAIR_THREADS / WAVE];
  __shared__ uint32_t n_longs, longs[G == WAVE ? PAIR_LONGS : 1];
  const uint32_t at = threadIdx.x % G, groups = gridDim.x * (PAIR_THREADS / G);
  uint32_t s = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x * (PAIR_THREADS / G) + threadIdx.x / G)));
  const uint64_t n_gaps = gap_off[n_scen];
  if (n_gaps >= PAIR_MOST_GAPS) return;   // (k_pair_init has seen the number too)
  const uint64_t* f = reinterpret_cast<const uint64_t*>(filled_ns);
  // the workgroup's sum over its threads' (the words are free again behind the caller's next barrier)
  auto all_of = [&](uint64_t mine) {
    uint64_t total = wave_sum_u64(mine);
    if (lane_id() == 0) part[threadIdx.x / WAVE] = total;
    __syncthreads();
    total = 0;
#pragma unroll
    for (int w = 0; w < PAIR_THREADS / WAVE; ++w) total += part[w];
    return total;
  };
  if (G == WAVE) {
    if (threadIdx.x == 0) n_longs = 0;
    __syncthreads();
  }
  if (s < n_scen) {   // (the same in the whole group)
    const uint64_t average = n_gaps / n_scen, long_above = average * PAIR_LONG > PAIR_LONG_LEAST ? average * PAIR_LONG : PAIR_LONG_LEAST;
    uint32_t hp = hp_task[s], lp = lp_task[s];
    uint64_t g0 = gap_off[s], g1 = gap_off[s + 1];
    // scenarios of one task that follow each other share an exchange (100,000 of 64 tasks in turn: sums 240 us with a workgroup
    // each, 325 by waves that exchange every one, 37 so)
    long long top = INT64_MIN;   // (what a task starts with)
    for (;;) {
      const uint32_t s_next = n_scen - s > groups ? s + groups : s;   // (the last one is looked up again)
      const uint32_t hp_next = hp_task[s_next], lp_next = lp_task[s_next];
      const uint64_t g0_next = gap_off[s_next], g1_next = gap_off[s_next + 1];
      if (hp >= n_tasks || lp >= n_tasks) {   // (these are the same in all of the group's lanes)
        if (at == 0) atomicOr(&ctrl->status, ERR_TASK_INDEX);
      } else if (g1 < g0 || g1 > n_gaps || (s == 0 && g0 != 0)) {
        if (at == 0) atomicOr(&ctrl->status, ERR_GAP_OFFSETS);
      } else {
        uint32_t place = PAIR_LONGS;
        if (G == WAVE && g1 - g0 > long_above) {
          if (at == 0) place = atomicAdd(&n_longs, 1u);
          place = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(place)));
        }
        if (place < PAIR_LONGS) {
          if (at == 0) longs[place] = s;
        } else {
          const uint64_t mine = pair_lane_sum<G>(f, g0, g1, at), total = G == WAVE ? wave_sum_u64(mine) : all_of(mine);
          if (at == 0) scen_filled[s] = static_cast<int64_t>(total);
          top = static_cast<long long>(total) > top ? static_cast<long long>(total) : top;
        }
        if (hp_next != hp || s_next == s) {
          if (at == 0 && top != INT64_MIN) atomicMax(&top_filled[hp], top);
          top = INT64_MIN;
        }
      }
      if (G != WAVE || s_next == s) break;   // (one scenario per workgroup)
      s = s_next; hp = hp_next; lp = lp_next; g0 = g0_next; g1 = g1_next;
    }
  }
  if (G != WAVE) return;
  __syncthreads();
  for (uint32_t i = 0; i < min_u32(n_longs, PAIR_LONGS); ++i) {
    const uint32_t scenario = longs[i];
    const uint64_t total = all_of(pair_lane_sum<PAIR_THREADS>(f, gap_off[scenario], gap_off[scenario + 1], threadIdx.x));
    if (threadIdx.x == 0) {
      scen_filled[scenario] = static_cast<int64_t>(total);
      atomicMax(&top_filled[hp_task[scenario]], static_cast<long long>(total));
    }
    __syncthreads();
  }
}

// The partner and the filled time of the scenario that was picked.
__device__ __forceinline__ void pair_result(uint32_t t, const uint32_t* __restrict__ lp_task, const int64_t* __restrict__ scen_filled,
                                            unsigned long long* best_scenario, uint32_t* __restrict__ best_lp, int64_t* __restrict__ best_filled) {
  const unsigned long long b = __hip_atomic_load(&best_scenario[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (b == ~0ull) return;
  best_lp[t] = lp_task[b];
  best_filled[t] = scen_filled[b];
}

// Among the scenarios of a task with the largest filled time the one whose partner completes earliest, and among those the
// first.  A scenario takes the task's place from the one that holds it if it comes before that one; both are compared by the
// call's inputs, so the word that changes hands is all that workgroups tell each other.  Few scenarios reach the largest filled
// time as a rule, and few try.  Where nothing fits into any gap all of them do: with more than PAIR_FEW in a workgroup, its best
// one of each task is found in LDS first, and only that one tries (pick in us, all try / so, and two rounds of atomic minima:
// 16,384 scenarios of one task that all fill nothing, completions falling 315 / 10, 195, rising 175 / 10, 194; 100,000 of 64
// tasks, falling 100 / 59, 38). With up to PAIR_LAST_TASKS tasks the last workgroup to get here writes the results; with more,
// k_pair_finish does (one workgroup takes 256 of them at a time, 1.5 us each).  Two launches for what took three (16,384
// scenarios of 128 tasks: call 89.0 us with three).
constexpr uint32_t PAIR_LAST_TASKS = 512;
constexpr uint32_t PAIR_FEW = 8, PAIR_SLOTS = 512, PAIR_PROBES = 8;
constexpr uint32_t PAIR_NONE = ~0u;
__global__ void __launch_bounds__(PAIR_THREADS)
k_pair_pick(const uint32_t* __restrict__ hp_task, const uint32_t* __restrict__ lp_task, uint64_t n_scen, uint32_t n_tasks,
            const int64_t* __restrict__ scen_filled, const int64_t* __restrict__ completion, const long long* __restrict__ top_filled,
            unsigned long long* best_scenario, uint32_t* __restrict__ best_lp, int64_t* __restrict__ best_filled, Ctrl* ctrl) {
  __shared__ uint32_t last;
  __shared__ long long soonest[PAIR_SLOTS];
  __shared__ uint32_t owner[PAIR_SLOTS], first[PAIR_SLOTS];   // (scenarios and tasks number fewer than 2^32 - 1)
  if (ctrl->status) return;
  const unsigned long long s = static_cast<unsigned long long>(blockIdx.x) * PAIR_THREADS + threadIdx.x;
  uint32_t hp = 0;
  bool tries = false;
  if (s < n_scen) {
    hp = hp_task[s];
    tries = scen_filled[s] == top_filled[hp];
  }
  const int64_t done = tries ? completion[s] : 0;
  if (__syncthreads_count(tries) > static_cast<int>(PAIR_FEW)) {
    for (uint32_t i = threadIdx.x; i < PAIR_SLOTS; i += PAIR_THREADS) { soonest[i] = INT64_MAX; owner[i] = PAIR_NONE; first[i] = PAIR_NONE; }
    __syncthreads();
    uint32_t slot = PAIR_NONE;   // (a task that finds none goes on without)
    if (tries) {
      for (uint32_t p = 0; p < PAIR_PROBES && slot == PAIR_NONE; ++p) {
        const uint32_t h = (hp + p) % PAIR_SLOTS, held = atomicCAS(&owner[h], PAIR_NONE, hp);
        if (held == PAIR_NONE || held == hp) slot = h;
      }
      if (slot != PAIR_NONE) atomicMin(&soonest[slot], static_cast<long long>(done));
    }
    __syncthreads();
    tries = tries && (slot == PAIR_NONE || soonest[slot] == done);
    if (tries && slot != PAIR_NONE) atomicMin(&first[slot], static_cast<uint32_t>(s));
    __syncthreads();
    tries = tries && (slot == PAIR_NONE || first[slot] == static_cast<uint32_t>(s));
  }
  if (tries) {
    unsigned long long held = __hip_atomic_load(&best_scenario[hp], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
      if (held != ~0ull) {
        const int64_t then = completion[held];
        if (then < done || (then == done && held < s)) break;
      }
      const unsigned long long old = atomicCAS(&best_scenario[hp], held, s);
      if (old == held) break;
      held = old;
    }
  }
  if (n_tasks > PAIR_LAST_TASKS) return;
  __syncthreads();   // (every exchange of this workgroup has been answered)
  if (threadIdx.x == 0) last = atomicAdd(&ctrl->taken, 1u) + 1 == gridDim.x ? 1u : 0u;
  __syncthreads();
  if (!last) return;
  for (uint32_t t = threadIdx.x; t < n_tasks; t += PAIR_THREADS) pair_result(t, lp_task, scen_filled, best_scenario, best_lp, best_filled);
}

__global__ void __launch_bounds__(PAIR_THREADS)
k_pair_finish(uint32_t n_tasks, const uint32_t* __restrict__ lp_task, const int64_t* __restrict__ scen_filled,
              unsigned long long* best_scenario, uint32_t* __restrict__ best_lp, int64_t* __restrict__ best_filled, const Ctrl* ctrl) {
  if (ctrl->status) return;
  const uint32_t t = blockIdx.x * PAIR_THREADS + threadIdx.x;
  if (t < n_tasks) pair_result(t, lp_task, scen_filled, best_scenario, best_lp, best_filled);
}

}  // namespace fikit
