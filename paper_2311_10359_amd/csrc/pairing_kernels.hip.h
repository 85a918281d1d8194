// The best low-priority partner of every high-priority task among evaluated combinations (the paper's
// discussion section, "What Tasks are Suitable for Sharing a GPU").
#pragma once

#include "common.hip.h"

namespace fikit {

constexpr int PAIR_THREADS = 256;
constexpr uint64_t PAIR_MOST_GAPS = (1ull << 32) - (1ull << 24);   // a call with as many or more is refused

// The control block and start values per task (no memset: the stream may be under graph capture).  The number of gaps is looked
// at here and not by the host, which would have to wait for it (16,384 scenarios of
// 2047 gaps: 109 us with that wait, 95 us without).
__global__ void k_pair_init(uint32_t n_tasks, const uint64_t* __restrict__ n_gaps, long long* __restrict__ top_filled,
                            long long* __restrict__ soonest, unsigned long long* __restrict__ best_scenario, Ctrl* ctrl) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  const bool refused = n_gaps && *n_gaps >= PAIR_MOST_GAPS;
  if (t < sizeof(Ctrl) / 4) reinterpret_cast<uint32_t*>(ctrl)[t] = t == 0 && refused ? ERR_GAP_OFFSETS : 0u;
  if (t >= n_tasks || refused) return;
  top_filled[t] = INT64_MIN;
  soonest[t] = INT64_MAX;
  best_scenario[t] = ~0ull;
}

// One workgroup per scenario: checks the scenario, sums the time filled in its gaps (8 B read per gap) and raises the largest
// filled time seen for its high-priority task.  Bound by HBM once enough bytes are in flight: a lane has up to eight 16-byte
// reads out at a time.  16,384 scenarios of 2047 gaps: 62 us = 4.3 TB/s (four 8-byte reads at a time: 75 us).  A wave per
// scenario is no faster (call 99 us against 97 us; 16,384 of 127 gaps 76 us against 77 us).  Up to 256 gaps a lane reads one of
// them: eight guarded reads are then most of the instructions (200,000 scenarios of 3 gaps, call 273 us with them, 227 us without;
// of 30 gaps 253 and 225 us).  The atomic returns nothing, so
// nothing waits for it; looking at the word first does wait, at a word that all scenarios of a task share (158 us).
__global__ void __launch_bounds__(PAIR_THREADS)
k_pair_sum(const uint32_t* __restrict__ hp_task, const uint32_t* __restrict__ lp_task, uint64_t n_scen, uint32_t n_tasks,
           const uint64_t* __restrict__ gap_off, const int64_t* __restrict__ filled_ns, int64_t* __restrict__ scen_filled,
           long long* __restrict__ top_filled, Ctrl* ctrl) {
  __shared__ uint64_t part[PAIR_THREADS / WAVE];
  const uint32_t tid = threadIdx.x;
  const uint64_t s = blockIdx.x;
  const uint32_t hp = hp_task[s], lp = lp_task[s];
  const uint64_t g0 = gap_off[s], g1 = gap_off[s + 1], n_gaps = gap_off[n_scen];
  if (n_gaps >= PAIR_MOST_GAPS) return;   // (k_pair_init has seen it too)
  if (hp >= n_tasks || lp >= n_tasks) {
    if (tid == 0) atomicOr(&ctrl->status, ERR_TASK_INDEX);
    return;
  }
  if (g1 < g0 || g1 > n_gaps || (s == 0 && g0 != 0)) {
    if (tid == 0) atomicOr(&ctrl->status, ERR_GAP_OFFSETS);
    return;
  }
  constexpr int READS = 8;
  uint64_t acc[2] = {0, 0};      // (sums wrap like the oracle's additions)
  const uint64_t* f = reinterpret_cast<const uint64_t*>(filled_ns);
  if (g1 - g0 <= PAIR_THREADS) {   // few gaps: one read per lane, and few instructions
    if (tid < g1 - g0) acc[0] = f[g0 + tid];
  } else {
    // pairs from the first gap on that lies on a 16-byte address; the gap before them and the one behind by one lane
    const uint64_t p0 = (reinterpret_cast<uintptr_t>(f + g0) & 15) ? g0 + 1 : g0;
    const uint64_t pairs = (g1 - p0) / 2;
    const ulonglong2* v = reinterpret_cast<const ulonglong2*>(f + p0);
    uint64_t i = tid;
    for (; i + (READS - 1) * PAIR_THREADS < pairs; i += READS * PAIR_THREADS) {
      ulonglong2 x[READS];
#pragma unroll
      for (int k = 0; k < READS; ++k) x[k] = v[i + k * PAIR_THREADS];
#pragma unroll
      for (int k = 0; k < READS; ++k) { acc[0] += x[k].x; acc[1] += x[k].y; }
    }
    {
      ulonglong2 x[READS];
#pragma unroll
      for (int k = 0; k < READS; ++k) {
        x[k] = make_ulonglong2(0, 0);
        if (i + k * PAIR_THREADS < pairs) x[k] = v[i + k * PAIR_THREADS];
      }
#pragma unroll
      for (int k = 0; k < READS; ++k) { acc[0] += x[k].x; acc[1] += x[k].y; }
    }
    if (tid == 0) {
      if (p0 > g0) acc[0] += f[g0];
      if (p0 + 2 * pairs < g1) acc[1] += f[g1 - 1];
    }
  }
  uint64_t total = wave_sum_u64(acc[0] + acc[1]);
  if (lane_id() == 0) part[tid >> 6] = total;
  __syncthreads();
  if (tid == 0) {
    total = 0;
#pragma unroll
    for (int w = 0; w < PAIR_THREADS / WAVE; ++w) total += part[w];
    scen_filled[s] = static_cast<int64_t>(total);
    atomicMax(&top_filled[hp], static_cast<long long>(total));
  }
}

// Among the scenarios of a task with the largest filled time: the earliest completion of the partner.
__global__ void k_pair_soonest(const uint32_t* __restrict__ hp_task, uint64_t n_scen, const int64_t* __restrict__ scen_filled,
                               const int64_t* __restrict__ completion, const long long* __restrict__ top_filled,
                               long long* __restrict__ soonest, const Ctrl* ctrl) {
  if (ctrl->status) return;
  const uint64_t s = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= n_scen) return;
  const uint32_t hp = hp_task[s];
  if (scen_filled[s] == top_filled[hp]) atomicMin(&soonest[hp], static_cast<long long>(completion[s]));
}

// Among those: the first scenario.
__global__ void k_pair_first(const uint32_t* __restrict__ hp_task, uint64_t n_scen, const int64_t* __restrict__ scen_filled,
                             const int64_t* __restrict__ completion, const long long* __restrict__ top_filled,
                             const long long* __restrict__ soonest, unsigned long long* __restrict__ best_scenario,
                             const Ctrl* ctrl) {
  if (ctrl->status) return;
  const uint64_t s = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= n_scen) return;
  const uint32_t hp = hp_task[s];
  if (scen_filled[s] == top_filled[hp] && completion[s] == soonest[hp]) atomicMin(&best_scenario[hp], static_cast<unsigned long long>(s));
}

// The partner and the filled time of the scenario that was picked; a task that heads no scenario gets
// the "none" values.
__global__ void k_pair_finish(uint32_t n_tasks, const uint32_t* __restrict__ lp_task, const unsigned long long* __restrict__ best_scenario,
                              uint32_t* __restrict__ best_lp, long long* __restrict__ top_filled, const Ctrl* ctrl) {
  if (ctrl->status) return;
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_tasks) return;
  const unsigned long long b = best_scenario[t];
  best_lp[t] = b == ~0ull ? ~0u : lp_task[b];
  if (b == ~0ull) top_filled[t] = 0;
}

}  // namespace fikit
