// Gap filling (Algorithm 1, FIKIT procedure; Algorithm 2, BestPrioFit, with a single waiting
// request): per scenario, walk the high-priority trace and issue the low-priority task's next
// kernels into each predicted idle gap for as long as they fit.
//
// Because predicted durations are >= 0, "keep issuing the head of the queue while it fits into
// what is left" is the same as "advance the queue pointer to the last position whose running sum
// of durations does not exceed (consumed so far) + (gap - margin)".  Predictions are looked up once per
// launch (k_gf_predict32) and are 32-bit numbers of nanoseconds; calls with a prediction that does not fit take
// the 64-bit kernels (k_gf_predict, k_gf_walk; k_gf_wide where both are one launch).
#pragma once

#include "common.hip.h"

namespace fikit {

// Scenarios in the order in which the walks' waves take them, the longest traces first: buckets of half an octave of the
// high-priority trace's length (bucket 0 the longest), in no order inside.  With several waves per SIMD, what a SIMD has to do is
// the sum of the traces it happens to get, and the longest may start last: 6000 traces of 1 to 2800 launches needed 93 cycles of
// a SIMD per gap, even ones 53.  The kernel that checks the scenarios fills the lists, which costs it 1 to 4 us; scenarios of one
// bucket are taken as they are numbered.  Calls in us as numbered / longest first: gap fill of these 6000 431 / 397, of 20,000 of
// up to 1200 launches 437 / 392, of 2100 of up to 1000 151 / 150; replay of 3000 traces of up to 4000 launches 491 / 463;
// priority queues, 4096 traces of up to 1600 launches and three queues each 1249 / 1088; even lengths, 2100 scenarios 117 / 119,
// 6000 350 / 351, 30,000 407 / 411.  The longest buckets' waves at a higher priority on their SIMD: 397, 392, 150, 464 and 1079
// us for the ragged ones; not worth standing before other streams' waves.
struct GfOrder {
  uint32_t* count;    // [GF_BUCKETS] scenarios of each bucket, in the words behind the control block (which k_gf_clear clears too);
                      // null: as they are numbered
  uint16_t* list;     // [GF_BUCKETS][n_scen]
};
constexpr uint32_t GF_BUCKETS = 32;
constexpr uint32_t GF_BLOCK_WORDS = 64;   // the control block and the words behind it
static_assert(sizeof(Ctrl) + GF_BUCKETS * 4 <= GF_BLOCK_WORDS * 4, "the buckets' counts lie behind the control block");
__device__ __forceinline__ uint32_t gf_bucket(uint64_t launches) {
  // exponent and first bit of the fraction; 16 launches and fewer are the last bucket, 2^19.5 and more the first
  const uint32_t octaves = __float_as_uint(static_cast<float>(launches)) >> 22, least = (127 + 4) * 2;
  const uint32_t k = octaves > least ? octaves - least : 0u;
  return GF_BUCKETS - 1 - (k < GF_BUCKETS - 1 ? k : GF_BUCKETS - 1);
}
// Puts scenario s on its list (called by all threads of a workgroup; cnt: LDS).  One reservation per workgroup and bucket.
__device__ __forceinline__ void gf_order(const GfOrder& order, uint64_t n_scen, uint64_t s, bool valid, uint64_t launches, uint32_t* cnt) {
  const uint32_t tid = threadIdx.x;
  __syncthreads();
  if (tid < GF_BUCKETS) cnt[tid] = 0;
  __syncthreads();
  const uint32_t b = valid ? gf_bucket(launches) : 0u;
  uint32_t at = 0;
  if (valid) at = atomicAdd(&cnt[b], 1u);
  __syncthreads();
  if (tid < GF_BUCKETS && cnt[tid]) cnt[tid] = atomicAdd(&order.count[tid], cnt[tid]);
  __syncthreads();
  if (valid) order.list[b * n_scen + cnt[b] + at] = static_cast<uint16_t>(s);
}

// Start values of a call: the control block, and per task no role, no queue total and (done may be null) no predictions.
__global__ void k_gf_clear(Ctrl* ctrl, uint32_t* __restrict__ role, uint64_t* __restrict__ lp_total, uint32_t* __restrict__ done,
                           uint32_t n_tasks) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < GF_BLOCK_WORDS) reinterpret_cast<uint32_t*>(ctrl)[t] = 0;
  if (t >= n_tasks) return;
  role[t] = 0;
  lp_total[t] = 0;
  if (done) done[t] = 0;
}

// Checks the task offsets (first 0, non-decreasing, last == n_ids) and the scenario arguments (n_gaps: the number of
// per-gap output slots the host sized its buffers for, ANY_GAPS if it does not look at it), and records in role[t] how each
// task is used.  One thread per task and per scenario; nothing is looked up at an offset here, so the two checks need not
// wait for each other.  Returns what is wrong.
constexpr uint64_t ANY_GAPS = ~0ull;
template <typename Mark>
__device__ __forceinline__ uint32_t gf_check_item(const uint64_t* __restrict__ off, uint32_t n_tasks, uint64_t n_ids, uint32_t hp, uint32_t lp,
                                                  uint64_t n_scen, uint64_t g0, uint64_t g1, uint64_t n_gaps, uint64_t s, Mark mark) {
  uint32_t wrong = 0;
  if (s < n_tasks) {
    const uint64_t a = off[s], b = off[s + 1];
    if (a > b || b > n_ids || (s == 0 && a != 0) || (s + 1 == n_tasks && b != n_ids)) wrong |= ERR_OFFSETS;
  }
  if (s >= n_scen) return wrong;
  if (s + 1 == n_scen && n_gaps != ANY_GAPS && g1 != n_gaps) wrong |= ERR_GAP_OFFSETS;
  if (hp >= n_tasks || lp >= n_tasks) return wrong | ERR_TASK_INDEX;
  const uint64_t H = off[hp + 1] - off[hp];
  const uint64_t want = H > 0 ? H - 1 : 0;
  if (g1 < g0 || g1 - g0 != want || (s == 0 && g0 != 0)) wrong |= ERR_GAP_OFFSETS;
  mark(hp, ROLE_HP);
  mark(lp, ROLE_LP);
  return wrong;
}
__global__ void k_gf_check(const uint64_t* __restrict__ off, uint32_t n_tasks, uint64_t n_ids, const uint32_t* __restrict__ hp_task,
                           const uint32_t* __restrict__ lp_task, uint64_t n_scen, const uint64_t* __restrict__ gap_off,
                           uint64_t n_gaps, uint32_t* __restrict__ role, const GfOrder order, Ctrl* ctrl) {
  __shared__ uint32_t cnt[GF_BUCKETS];
  const uint64_t s = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const uint64_t at = s < n_scen ? s : 0u;
  // (a task heads or serves many scenarios: the word is only touched while a bit is still missing)
  const uint32_t wrong = gf_check_item(off, n_tasks, n_ids, hp_task[at], lp_task[at], n_scen, gap_off[at], gap_off[at + 1], n_gaps, s,
                                       [&](uint32_t t, uint32_t bit) {
    if (!(__hip_atomic_load(&role[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)) atomicOr(&role[t], bit);
  });
  if (wrong) atomicOr(&ctrl->status, wrong);
  if (order.count) {
    const bool valid = !wrong && s < n_scen;   // (with an error nothing is walked)
    const uint32_t hp = valid ? hp_task[s] : 0u;
    gf_order(order, n_scen, s, valid, off[hp + 1] - off[hp], cnt);
  }
}

// Both of the above in one workgroup, for so few tasks and scenarios that a second launch costs more (4.5 us) than the
// chip's other units save.  What it does takes no time; what it waits for does: everything is asked for at once (GfFirst,
// BeginOffsets), and the roles are gathered in LDS.  (The offsets read where they are needed and the roles in memory, behind a
// fence / now: 64 scenarios of 16 tasks, call 74.2 / 69.3 us; the first launch of a step of one scenario 11.4 / 7.0 us between
// events.)
constexpr uint32_t GF_BEGIN_ITEMS = 2048;
constexpr int GF_BEGIN_THREADS = 1024;
struct GfBegin {
  const uint32_t *hp_task, *lp_task;
  uint32_t n_scen;
  const uint64_t* gap_off;
  uint64_t n_gaps;
  uint32_t* role;
  uint64_t* lp_total;
  uint32_t* done;
  Ctrl* ctrl;
};
// What a thread looks at of the scenarios, asked for before anything is waited for.
struct GfFirst {
  static constexpr uint32_t ITEMS = GF_BEGIN_ITEMS / GF_BEGIN_THREADS;
  uint32_t hp[ITEMS], lp[ITEMS];
  uint64_t g0[ITEMS], g1[ITEMS];
  __device__ __forceinline__ explicit GfFirst(const GfBegin& a) {
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
      const uint32_t s = threadIdx.x + k * GF_BEGIN_THREADS, at = s < a.n_scen ? s : 0u;   // (there is one at least)
      hp[k] = a.hp_task[at]; lp[k] = a.lp_task[at];
      g0[k] = a.gap_off[at]; g1[k] = a.gap_off[at + 1];
    }
  }
};
// The task offsets in LDS, of up to GF_BEGIN_ITEMS tasks.  Ends with a barrier.
struct BeginOffsets { uint64_t off[GF_BEGIN_ITEMS + 1]; };
__device__ __forceinline__ void begin_offsets(BeginOffsets& sm, const uint64_t* __restrict__ off, uint32_t n_tasks) {
  constexpr uint32_t ROUNDS = GF_BEGIN_ITEMS / GF_BEGIN_THREADS + 1;
  uint64_t v[ROUNDS];
#pragma unroll
  for (uint32_t k = 0; k < ROUNDS; ++k) v[k] = off[min_u32(threadIdx.x + k * GF_BEGIN_THREADS, n_tasks)];
#pragma unroll
  for (uint32_t k = 0; k < ROUNDS; ++k)
    if (threadIdx.x + k * GF_BEGIN_THREADS <= n_tasks) sm.off[threadIdx.x + k * GF_BEGIN_THREADS] = v[k];
  __syncthreads();
}
__device__ __forceinline__ void gf_begin(const BeginOffsets& sm, uint32_t n_tasks, uint64_t n_ids, const GfBegin& a, const GfFirst& first) {
  __shared__ uint32_t role[GF_BEGIN_ITEMS], status;
  const uint32_t tid = threadIdx.x;
  if (tid == 0) status = 0;
  for (uint32_t t = tid; t < n_tasks; t += GF_BEGIN_THREADS) role[t] = 0;
  __syncthreads();
  uint32_t wrong = 0;
#pragma unroll
  for (uint32_t k = 0; k < GfFirst::ITEMS; ++k)
    wrong |= gf_check_item(sm.off, n_tasks, n_ids, first.hp[k], first.lp[k], a.n_scen, first.g0[k], first.g1[k], a.n_gaps, tid + k * GF_BEGIN_THREADS,
                           [&](uint32_t t, uint32_t bit) { atomicOr(&role[t], bit); });
  if (wrong) atomicOr(&status, wrong);
  __syncthreads();
  for (uint32_t t = tid; t < n_tasks; t += GF_BEGIN_THREADS) {
    a.role[t] = role[t];
    a.lp_total[t] = 0;
    if (a.done) a.done[t] = 0;
  }
  if (tid < sizeof(Ctrl) / 4) reinterpret_cast<uint32_t*>(a.ctrl)[tid] = tid == 0 ? status : 0u;
}

__global__ void __launch_bounds__(GF_BEGIN_THREADS)
k_gf_begin(const uint64_t* __restrict__ off, uint32_t n_tasks, uint64_t n_ids, const GfBegin a) {
  __shared__ BeginOffsets sm;
  const GfFirst first(a);
  begin_offsets(sm, off, n_tasks);
  gf_begin(sm, n_tasks, n_ids, a, first);
}

// The status a finished call would return, from the error bits its kernels left (fikit_gapfill_static).
__device__ __forceinline__ int32_t gf_status(uint32_t bits) {
  if (bits & (ERR_OFFSETS | ERR_TASK_INDEX | ERR_GAP_OFFSETS)) return FIKIT_INVALID_ARG;
  return bits & ERR_UNKNOWN_ID ? FIKIT_UNKNOWN_ID : FIKIT_OK;
}

constexpr int PRED_THREADS = 256;
constexpr int PRED_KPT = 8;                       // consecutive launches per thread and chunk
constexpr int PRED_CHUNK = PRED_THREADS * PRED_KPT;
constexpr int PRED_ROWS = 512;                    // rows of a task kept in an LDS hash table for the lookup
constexpr int PRED_HT = 2 * PRED_ROWS;
constexpr int PRED_READS = 2;                     // pairs of launches that a lane reads at a time (k_gf_predict32)

constexpr uint32_t WIDE32 = 0xffffffffu;   // 32-bit predictions must be below this

// The prediction read from a row's statistics: median, or mean = sum / count (Section 3.2: SK_j, SG_j).
__device__ __forceinline__ int64_t predicted_of(const fikit_stats& st, uint32_t predictor) {
  if (predictor == FIKIT_PREDICT_P50) return st.p50;
  return st.count ? static_cast<int64_t>(st.sum / st.count) : 0;
}

// Predicted execution time and idle time of a launch: taken from its ID's row.  Rows of a
// task with few IDs sit in an LDS hash table keyed by the ID; otherwise the task's sorted rows
// are searched in memory.
struct PredTable {
  uint64_t key[PRED_HT];
  int64_t e[PRED_HT];
  int64_t g[PRED_HT];
};

__device__ __forceinline__ bool find_row(uint64_t id, const fikit_row* __restrict__ rows, uint64_t r0, uint64_t nr, uint32_t predictor,
                                         int64_t& e, int64_t& g) {
  uint64_t lo = 0, hi = nr;
  while (lo < hi) { const uint64_t mid = (lo + hi) >> 1; if (rows[r0 + mid].kernel_id < id) lo = mid + 1; else hi = mid; }
  if (lo < nr && rows[r0 + lo].kernel_id == id) {
    e = predicted_of(rows[r0 + lo].exec, predictor);
    g = predicted_of(rows[r0 + lo].gap, predictor);
    return true;
  }
  return false;
}

__device__ __forceinline__ bool predict_one(uint64_t id, bool in_lds, const PredTable& tb, const fikit_row* __restrict__ rows,
                                            uint64_t r0, uint64_t nr, uint32_t predictor, int64_t& e, int64_t& g) {
  if (in_lds) {
    uint32_t h = (static_cast<uint32_t>(id >> 32) ^ static_cast<uint32_t>(id)) & (PRED_HT - 1);
    for (int probe = 0; probe < PRED_HT; ++probe) {
      const uint64_t k = tb.key[h];
      if (k == ~0ull) return false;   // (first: the ID looked for may be that value, and no row's is)
      if (k == id) { e = tb.e[h]; g = tb.g[h]; return true; }
      h = (h + 1) & (PRED_HT - 1);
    }
    return false;
  }
  return find_row(id, rows, r0, nr, predictor, e, g);
}

// One workgroup and one task that takes part in a scenario (rl: as what).  For every launch i of the task:
//   as low-priority queue:   pe[i]   = sum of predicted execution times of launches 0..i
//   as high-priority trace:  pg[i]   = predicted idle time after launch i
//                            open[i] = predicted time at which launch i ends (its gap opens):
//                                      sum_{k<=i} E_k + sum_{k<i} G_k   (not written if open is null)
// Prefix sums run thread -> wave -> workgroup, with a running carry from chunk to chunk.
__device__ __forceinline__ void gf_predict_task(PredTable& tb, uint32_t t, uint32_t rl, const uint64_t* __restrict__ ids,
                                                const uint64_t* __restrict__ off, const fikit_row* __restrict__ rows,
                                                const uint64_t* __restrict__ row_off, int64_t* __restrict__ pe, int64_t* __restrict__ pg,
                                                int64_t* __restrict__ open, uint32_t predictor, Ctrl* ctrl) {
  const uint64_t base = off[t], len = off[t + 1] - base;
  const uint64_t r0 = row_off[t], nr = row_off[t + 1] - r0;
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  // (an ID equal to the table's "empty" mark can only be the largest one)
  const bool in_lds = nr <= PRED_ROWS && (nr == 0 || rows[r0 + nr - 1].kernel_id != ~0ull);
  if (in_lds) {
    for (uint32_t h = tid; h < PRED_HT; h += PRED_THREADS) tb.key[h] = ~0ull;
    __syncthreads();
    for (uint32_t r = tid; r < nr; r += PRED_THREADS) {
      const fikit_row* row = rows + r0 + r;
      const uint64_t id = row->kernel_id;
      uint32_t h = (static_cast<uint32_t>(id >> 32) ^ static_cast<uint32_t>(id)) & (PRED_HT - 1);
      for (;;) {   // IDs of a task are distinct and fill at most half the table: a free slot exists
        const uint64_t old = atomicCAS(reinterpret_cast<unsigned long long*>(&tb.key[h]), ~0ull, id);
        if (old == ~0ull) break;
        h = (h + 1) & (PRED_HT - 1);
      }
      tb.e[h] = predicted_of(row->exec, predictor);
      tb.g[h] = predicted_of(row->gap, predictor);
    }
  }
  __syncthreads();
  uint64_t carry_e = 0, carry_o = 0;  // sums over all earlier launches: E, and E + G
  bool unknown = false;
  // A chunk is PRED_SUB sub-chunks of 2 * PRED_THREADS launches; in a sub-chunk every thread owns
  // two neighbouring launches, so that a wave reads and writes 1 KiB of consecutive memory per access.
  constexpr int PRED_SUB = PRED_KPT / 2;
  __shared__ uint64_t sub_sum[2][PRED_SUB * 4];
  const bool even = ((base & 1) == 0);   // 16-byte accesses to the workspace arrays need an even first index
  const bool ids_vec = (reinterpret_cast<uintptr_t>(ids + base) & 15) == 0;   // and those to the caller's IDs an aligned address
  for (uint64_t c0 = 0; c0 < len; c0 += PRED_CHUNK) {
    int64_t e[PRED_KPT], g[PRED_KPT];
    uint64_t ie[PRED_SUB], io[PRED_SUB];
#pragma unroll
    for (int k = 0; k < PRED_SUB; ++k) {
      const uint64_t i0 = c0 + static_cast<uint64_t>(k) * (2 * PRED_THREADS) + 2 * tid;
      uint64_t id0 = 0, id1 = 0;
      if (ids_vec && i0 + 1 < len) {
        const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(ids + base + i0);
        id0 = v.x; id1 = v.y;
      } else {
        if (i0 < len) id0 = ids[base + i0];
        if (i0 + 1 < len) id1 = ids[base + i0 + 1];
      }
      e[2 * k] = e[2 * k + 1] = g[2 * k] = g[2 * k + 1] = 0;
      if (i0 < len) unknown |= !predict_one(id0, in_lds, tb, rows, r0, nr, predictor, e[2 * k], g[2 * k]);
      if (i0 + 1 < len) unknown |= !predict_one(id1, in_lds, tb, rows, r0, nr, predictor, e[2 * k + 1], g[2 * k + 1]);
      const uint64_t se = static_cast<uint64_t>(e[2 * k]) + static_cast<uint64_t>(e[2 * k + 1]);
      const uint64_t so = se + static_cast<uint64_t>(g[2 * k]) + static_cast<uint64_t>(g[2 * k + 1]);
      // a task needs the sums of the role it plays only (the branch is the same for the whole workgroup)
      ie[k] = io[k] = 0;
      if (rl & ROLE_LP) { ie[k] = wave_incl_scan_u64(se); if (lane == 63) sub_sum[0][k * 4 + w] = ie[k]; ie[k] -= se; }
      if (rl & ROLE_HP) { io[k] = wave_incl_scan_u64(so); if (lane == 63) sub_sum[1][k * 4 + w] = io[k]; io[k] -= so; }
    }
    __syncthreads();
    uint64_t run_e = carry_e, run_o = carry_o;
#pragma unroll
    for (int k = 0; k < PRED_SUB; ++k) {
      uint64_t be = run_e, bo = run_o;
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) {
        const uint64_t te = (rl & ROLE_LP) ? sub_sum[0][k * 4 + ww] : 0, to = (rl & ROLE_HP) ? sub_sum[1][k * 4 + ww] : 0;
        if (static_cast<uint32_t>(ww) < w) { be += te; bo += to; }
        run_e += te; run_o += to;
      }
      be += ie[k]; bo += io[k];
      const uint64_t i0 = c0 + static_cast<uint64_t>(k) * (2 * PRED_THREADS) + 2 * tid;
      const uint64_t pe0 = be + static_cast<uint64_t>(e[2 * k]), pe1 = pe0 + static_cast<uint64_t>(e[2 * k + 1]);
      const uint64_t op0 = bo + static_cast<uint64_t>(e[2 * k]);   // E and G of earlier launches + own E
      const uint64_t op1 = op0 + static_cast<uint64_t>(g[2 * k]) + static_cast<uint64_t>(e[2 * k + 1]);
      if (even && i0 + 1 < len) {
        if (rl & ROLE_LP) *reinterpret_cast<ulonglong2*>(pe + base + i0) = make_ulonglong2(pe0, pe1);
        if (rl & ROLE_HP) {
          *reinterpret_cast<ulonglong2*>(pg + base + i0) = make_ulonglong2(static_cast<uint64_t>(g[2 * k]), static_cast<uint64_t>(g[2 * k + 1]));
          if (open) *reinterpret_cast<ulonglong2*>(open + base + i0) = make_ulonglong2(op0, op1);
        }
      } else {
        if (i0 < len) {
          if (rl & ROLE_LP) pe[base + i0] = static_cast<int64_t>(pe0);
          if (rl & ROLE_HP) { pg[base + i0] = g[2 * k]; if (open) open[base + i0] = static_cast<int64_t>(op0); }
        }
        if (i0 + 1 < len) {
          if (rl & ROLE_LP) pe[base + i0 + 1] = static_cast<int64_t>(pe1);
          if (rl & ROLE_HP) { pg[base + i0 + 1] = g[2 * k + 1]; if (open) open[base + i0 + 1] = static_cast<int64_t>(op1); }
        }
      }
    }
    carry_e = run_e;
    carry_o = run_o;
    __syncthreads();   // sub_sum is rewritten by the next chunk
  }
  if (unknown) atomicOr(&ctrl->status, ERR_UNKNOWN_ID);
}
// One workgroup per task.
__global__ void __launch_bounds__(PRED_THREADS) __attribute__((amdgpu_waves_per_eu(5, 8)))
k_gf_predict(const uint64_t* __restrict__ ids, const uint64_t* __restrict__ off, uint32_t n_tasks,
             const fikit_row* __restrict__ rows, const uint64_t* __restrict__ row_off, const uint32_t* __restrict__ role,
             int64_t* __restrict__ pe, int64_t* __restrict__ pg, int64_t* __restrict__ open, uint32_t predictor, Ctrl* ctrl) {
  __shared__ PredTable tb;
  // only bits that earlier kernels set: the decision must be the same for the whole workgroup
  if (ctrl->status & (ERR_OFFSETS | ERR_TASK_INDEX | ERR_GAP_OFFSETS)) return;
  if (!ctrl->wide) return;
  const uint32_t t = rotated_item(blockIdx.x, n_tasks), rl = role[t];
  if (rl) gf_predict_task(tb, t, rl, ids, off, rows, row_off, pe, pg, open, predictor, ctrl);
}

// The walk on 64-bit prefix sums, one wave per scenario: for calls with a prediction that does not fit 32 bits.
__device__ __forceinline__ int64_t lane_value(int64_t v, uint32_t idx) {   // (idx: the same in all lanes)
  return static_cast<int64_t>(read_lane_u64(static_cast<uint64_t>(v), idx));
}

__device__ __forceinline__ void gf_walk_scenario(uint64_t s, const uint64_t* __restrict__ off, const uint32_t* __restrict__ hp_task,
                                                 const uint32_t* __restrict__ lp_task, const uint64_t* __restrict__ gap_off, const int64_t* pe,
                                                 const int64_t* pg, const int64_t* open, int64_t margin, int64_t min_gap,
                                                 uint32_t* __restrict__ fill_count, int64_t* __restrict__ filled_ns,
                                                 int64_t* __restrict__ completion_out, uint64_t* __restrict__ placed_out) {
  const uint32_t lane = lane_id();

  const uint32_t hp = hp_task[s], lp = lp_task[s];
  const uint64_t h0 = off[hp], H = off[hp + 1] - h0;
  const uint64_t l0 = off[lp], L = off[lp + 1] - l0;
  const uint64_t g0 = gap_off[s];
  const uint64_t n_gaps = H > 0 ? H - 1 : 0;

  uint64_t p = 0;         // low-priority kernels issued so far
  int64_t consumed = 0;   // their total predicted duration = pe[l0 + p - 1]
  bool done = (L == 0);
  int64_t completion = 0;
  // The wave keeps 128 consecutive prefix sums of the low-priority queue in registers (win0: entries
  // wb .. wb+63, win1: the next 64), with wb <= p < wb + 64, so that most gaps are searched without
  // touching memory.
  uint64_t wb = 0;
  int64_t win0 = lane < L ? pe[l0 + lane] : INT64_MAX;
  int64_t win1 = WAVE + lane < L ? pe[l0 + WAVE + lane] : INT64_MAX;

  // The predicted gaps of the next round are read while this round is worked on.
  int64_t next_g = lane < n_gaps ? pg[h0 + lane] : 0;
  for (uint64_t i0 = 0; i0 < n_gaps; i0 += WAVE) {
    const uint64_t mine = i0 + lane;
    const int64_t my_g = next_g;
    next_g = mine + WAVE < n_gaps ? pg[h0 + mine + WAVE] : 0;
    uint32_t my_c = 0;
    int64_t my_f = 0;
    const uint32_t steps = static_cast<uint32_t>(n_gaps - i0 < WAVE ? n_gaps - i0 : WAVE);
    uint32_t k = 0;
    while (k < steps) {
      // Gaps that the head of the queue does not fit into take nothing and change nothing: every lane tests
      // its own gap against the head, and the wave goes straight to the first gap that takes something.
      const int64_t head_abs = lane_value(win0, static_cast<uint32_t>(p - wb));
      const int64_t head = p < L ? head_abs - consumed : INT64_MAX;
      const bool takes = lane >= k && lane < steps && my_g >= min_gap && my_g >= margin && head <= my_g - margin;
      const uint64_t tb = ballot(takes);
      if (tb == 0) break;
      k = static_cast<uint32_t>(__builtin_ctzll(tb));
      const int64_t G = lane_value(my_g, k);
      uint32_t c = 0;
      int64_t f = 0;
      if (G >= min_gap && G >= margin && p < L) {
        const int64_t limit = consumed + (G - margin);
        int64_t last_fit = consumed;
        for (;;) {
          // candidate of this lane: queue entry p + c + lane, which lives in the window at idx
          const uint32_t idx = static_cast<uint32_t>(p + c - wb) + lane;          // 0 .. 126
          const int64_t a0 = static_cast<int64_t>(shfl_u64(static_cast<uint64_t>(win0), idx & (WAVE - 1)));
          const int64_t a1 = static_cast<int64_t>(shfl_u64(static_cast<uint64_t>(win1), idx & (WAVE - 1)));
          const int64_t val = idx < WAVE ? a0 : a1;    // INT64_MAX beyond the end of the queue
          const uint64_t b = ballot(val <= limit);
          const uint32_t cnt = b == ~0ull ? WAVE : static_cast<uint32_t>(__builtin_ctzll(~b));
          if (cnt > 0) last_fit = lane_value(val, cnt - 1);
          c += cnt;
          // keep the window under the search position
          if (p + c >= wb + WAVE) {
            wb += WAVE;
            win0 = win1;
            win1 = wb + WAVE + lane < L ? pe[l0 + wb + WAVE + lane] : INT64_MAX;
          }
          if (cnt < WAVE) break;
        }
        f = last_fit - consumed;
        consumed = last_fit;
        p += c;
        if (p == L && c > 0 && !done) {
          completion = open[h0 + i0 + k] + f;
          done = true;
        }
      }
      if (lane == k) { my_c = c; my_f = f; }
      ++k;
    }
    if (mine < n_gaps) {
      fill_count[g0 + mine] = my_c;
      filled_ns[g0 + mine] = my_f;
    }
  }
  if (!done) {
    const int64_t t_end = H > 0 ? open[h0 + H - 1] : 0;
    const int64_t rest = L > 0 ? pe[l0 + L - 1] - consumed : 0;
    completion = t_end + rest;
  }
  if (lane == 0) {
    completion_out[s] = completion;
    placed_out[s] = p;
  }
}
__global__ void __launch_bounds__(256)
k_gf_walk(const uint64_t* __restrict__ off, const uint32_t* __restrict__ hp_task, const uint32_t* __restrict__ lp_task,
          uint64_t n_scen, const uint64_t* __restrict__ gap_off, const int64_t* __restrict__ pe,
          const int64_t* __restrict__ pg, const int64_t* __restrict__ open, int64_t margin, int64_t min_gap,
          uint32_t* __restrict__ fill_count, int64_t* __restrict__ filled_ns, int64_t* __restrict__ completion_out,
          uint64_t* __restrict__ placed_out, int32_t* __restrict__ status_out, const Ctrl* ctrl) {
  // (status_out may be null: the call's status, which no kernel changes from here on)
  if (status_out && blockIdx.x == 0 && threadIdx.x == 0) *status_out = gf_status(ctrl->status);
  if (ctrl->status || !ctrl->wide) return;
  const uint64_t s = static_cast<uint64_t>(blockIdx.x) * (256 / WAVE) + threadIdx.x / WAVE;
  if (s >= n_scen) return;  // whole waves leave together
  gf_walk_scenario(s, off, hp_task, lp_task, gap_off, pe, pg, open, margin, min_gap, fill_count, filled_ns, completion_out, placed_out);
}

// Both in one launch, for a call of few scenarios that enqueues them before it knows whether they are needed
// (fikit_gapfill_static): the workgroup of a scenario looks its two tasks up (what several scenarios share is written by all of
// their workgroups, each the same values) and one of its waves walks.  Also where the call's status is published, which nothing
// before or in this launch changes by then: an ID without a row has been found by k_gf_predict32.  A launch that finds nothing to
// do costs 2.2 us of the chip's time and 3 of the host's: static calls in us, two launches / one: 64 scenarios of 1500 gaps 69.8
// / 68.4, a few of 100 gaps 22 / 19.4; with predictions beyond 32 bits one scenario 260 / 233, 64 of 16 tasks 322 / 280, 256 of
// 32 tasks 329 / 282, 256 that share a queue of 400,000 launches 1939 / 1991, 900 of 60 tasks 345 / 439, which decides the line.
constexpr uint64_t GF_WIDE_SCENARIOS = 256;
__global__ void __launch_bounds__(PRED_THREADS)
k_gf_wide(const uint64_t* __restrict__ ids, const uint64_t* __restrict__ off, const fikit_row* __restrict__ rows,
          const uint64_t* __restrict__ row_off, const uint32_t* __restrict__ role, const uint32_t* __restrict__ hp_task,
          const uint32_t* __restrict__ lp_task, const uint64_t* __restrict__ gap_off, int64_t* pe, int64_t* pg, int64_t* open,
          uint32_t predictor, int64_t margin, int64_t min_gap, uint32_t* __restrict__ fill_count, int64_t* __restrict__ filled_ns,
          int64_t* __restrict__ completion_out, uint64_t* __restrict__ placed_out, int32_t* __restrict__ status_out, Ctrl* ctrl) {
  __shared__ PredTable tb;
  const uint32_t status = ctrl->status;
  if (blockIdx.x == 0 && threadIdx.x == 0) *status_out = gf_status(status);
  if (status || !ctrl->wide) return;
  const uint64_t s = blockIdx.x;
  const uint32_t hp = hp_task[s], lp = lp_task[s];
  gf_predict_task(tb, hp, role[hp], ids, off, rows, row_off, pe, pg, open, predictor, ctrl);
  __syncthreads();   // (the table is built anew)
  if (lp != hp) gf_predict_task(tb, lp, role[lp], ids, off, rows, row_off, pe, pg, open, predictor, ctrl);
  __threadfence_block();
  __syncthreads();
  if (threadIdx.x < WAVE)
    gf_walk_scenario(s, off, hp_task, lp_task, gap_off, pe, pg, open, margin, min_gap, fill_count, filled_ns, completion_out, placed_out);
}

// ---------------------------------------------------------------------------------------------
// One lane per scenario.
//
// When there are many scenarios, the cheapest way to run Algorithm 1 is its literal form, one lane per
// scenario: keep what is left of the current gap, and issue the head of the low-priority queue while
// its predicted duration fits.  A lane needs the predicted execution time of every low-priority
// launch once, in order, and the predicted (execution time, idle time) of every high-priority launch
// once, in order: two streams per lane.  They are stored as 32-bit numbers (4 and 8 bytes per launch
// instead of three 8-byte arrays); a prediction that does not fit 32 bits sets Ctrl::wide and the
// call is redone with the 64-bit kernels above.
//
// Each lane steps through its own scenario: a sub-step either opens the next gap or tries the next
// queue entry, so lanes of a wave do not wait for the slowest gap.  Streams are read 64 bytes per lane
// at a time into registers and parked in per-lane LDS rings one period later, which hides the memory
// latency; a lane whose ring is empty simply idles for a sub-step.  Results are staged
// in LDS and written 8 gaps at a time.  With one wave per SIMD (65,536 scenarios fill the chip exactly
// once) a SIMD issues one instruction of its wave every four cycles at best, so the kernel's time is its
// number of instructions: the tries after an opening read all their queue entries at once and ahead of
// use, and whatever can be derived when a gap's result is staged (its count, its filled time, its opening
// time) is not carried through the tries.


// The table of k_gf_predict32: both predictions of an ID in one 8-byte word (WIDE32: does not fit 32 bits).  16 KB, so that a
// compute unit holds eight workgroups.
struct PredTable32 {
  uint64_t key[PRED_HT];
  uint2 eg[PRED_HT];
};
__device__ __forceinline__ uint32_t clamp32(int64_t v) {   // (predictions are not negative)
  return static_cast<uint64_t>(v) >= WIDE32 ? WIDE32 : static_cast<uint32_t>(v);
}

// Predicted values of every launch of the tasks that take part, in 32 bits (gridDim.y workgroups per task, each a
// part of its launches: with few tasks one workgroup per task leaves most of the chip idle; see predict_parts):
//   lp_e[i]  execution time, for tasks used as low-priority queue; lp_total[t] their sum (zero at the start)
//   hp_eg[i] (execution time, idle time), for tasks used as high-priority trace
// With the tasks in plain order the lengths' pattern decides: 16,384 tasks of 4096 and 16,384 launches in turn 652 us, the same
// in two halves 511 us; in rotated order (rotated_item) 496 and 501 us.  One task of 15,000 launches in eight, the others of
// 500: 599 -> 216 us.
// For the replay against actual idle times (actual != nullptr) the first word of hp_eg[i] holds the idle
// time that really followed launch i instead (clamped to WIDE32, which no filled time can reach).
// Bound by the memory that reads and writes by turns, once a lane has PRED_READS pairs of IDs on their way and both halves of an
// odd task's pairs come in one read: 6000 ragged scenarios 146 us with one read per pair where the task starts at an even place
// and two where not, 133 so; 6000 of 2048 and 8192 launches 195 / 186 = 5.5 TB/s (four pairs 139 and 184 us, one 152 and 211).
// pred_done (may be null): tasks whose predictions exist already and are left alone.  prof (may be null, as in the walks): the
// profile in the same call that this was enqueued behind.
__global__ void __launch_bounds__(PRED_THREADS)
k_gf_predict32(const uint64_t* __restrict__ ids, const uint64_t* __restrict__ off, uint32_t n_tasks,
               const fikit_row* __restrict__ rows, const uint64_t* __restrict__ row_off, const uint32_t* __restrict__ role,
               const int64_t* __restrict__ actual, uint32_t* __restrict__ lp_e, uint2* __restrict__ hp_eg,
               uint64_t* __restrict__ lp_total, uint32_t predictor, const uint32_t* __restrict__ pred_done, const Ctrl* prof,
               uint64_t row_capacity, Ctrl* ctrl) {
  __shared__ PredTable32 tb;
  __shared__ uint64_t wave_tot[PRED_THREADS / WAVE];
  if ((ctrl->status & (ERR_OFFSETS | ERR_TASK_INDEX | ERR_GAP_OFFSETS)) || !may_follow(prof, row_capacity)) return;
  const uint32_t t = rotated_item(blockIdx.x, n_tasks);
  const uint64_t part0 = static_cast<uint64_t>(blockIdx.y) * (2 * PRED_THREADS);   // first launch of this workgroup's part
  const uint32_t rl = role[t];
  if (rl == 0) return;
  if (pred_done && pred_done[t]) return;   // (the profile kernels wrote this task's predictions already)
  const uint64_t base = off[t], len = off[t + 1] - base;
  if (part0 >= len) return;
  const uint64_t r0 = row_off[t], nr = row_off[t + 1] - r0;
  const uint32_t tid = threadIdx.x;
  const bool in_lds = nr <= PRED_ROWS && (nr == 0 || rows[r0 + nr - 1].kernel_id != ~0ull);
  if (in_lds) {
    for (uint32_t h = tid; h < PRED_HT; h += PRED_THREADS) tb.key[h] = ~0ull;
    __syncthreads();
    for (uint32_t r = tid; r < nr; r += PRED_THREADS) {
      const fikit_row* row = rows + r0 + r;
      const uint64_t id = row->kernel_id;
      uint32_t h = (static_cast<uint32_t>(id >> 32) ^ static_cast<uint32_t>(id)) & (PRED_HT - 1);
      for (;;) {   // IDs of a task are distinct and fill at most half the table: a free slot exists
        const uint64_t old = atomicCAS(reinterpret_cast<unsigned long long*>(&tb.key[h]), ~0ull, id);
        if (old == ~0ull) break;
        h = (h + 1) & (PRED_HT - 1);
      }
      tb.eg[h] = make_uint2(clamp32(predicted_of(row->exec, predictor)), clamp32(predicted_of(row->gap, predictor)));
    }
  }
  __syncthreads();
  bool unknown = false, wide = false, bad_actual = false;
  auto predict = [&](uint64_t id) -> uint2 {
    if (in_lds) {
      unknown |= id == ~0ull;   // (no row's ID then, but what a free slot holds)
      uint32_t h = (static_cast<uint32_t>(id >> 32) ^ static_cast<uint32_t>(id)) & (PRED_HT - 1);
      for (int probe = 0; probe < PRED_HT; ++probe) {
        const uint64_t k = tb.key[h];
        if (k == id) return tb.eg[h];
        if (k == ~0ull) break;
        h = (h + 1) & (PRED_HT - 1);
      }
      unknown = true;
      return make_uint2(0, 0);
    }
    int64_t e = 0, g = 0;
    unknown |= !find_row(id, rows, r0, nr, predictor, e, g);
    return make_uint2(clamp32(e), clamp32(g));
  };
  uint64_t total = 0;
  // Pairs of launches start at even elements, so that they are read as 16 bytes and written as 8 and 16; an odd first launch goes
  // by itself. (IDs that lie on 8 bytes only are read one by one.)
  const bool ids_vec = (reinterpret_cast<uintptr_t>(ids) & 15) == 0;
  const uint32_t lead = static_cast<uint32_t>(base & 1);
  const uint64_t step = static_cast<uint64_t>(gridDim.y) * (2 * PRED_THREADS);
  uint64_t i0 = lead + part0 + 2 * static_cast<uint64_t>(tid);
  const bool hp_role = (rl & ROLE_HP) != 0, lp_role = (rl & ROLE_LP) != 0, with_actual = actual && hp_role;
  // what is left of a launch pair once its IDs and idle times are there
  auto finish = [&](uint64_t i, bool two, uint64_t id0, uint64_t id1, int64_t x0, int64_t x1) {
    const uint2 p0 = predict(id0);
    uint2 p1 = make_uint2(0, 0);
    if (two) p1 = predict(id1);
    const uint32_t a0 = p0.x, b0 = p0.y, a1 = p1.x, b1 = p1.y;
    wide |= a0 == WIDE32 || b0 == WIDE32 || a1 == WIDE32 || b1 == WIDE32;
    total += static_cast<uint64_t>(a0) + a1;
    uint32_t h0w = a0, h1w = a1;   // first word of the high-priority entries
    if (with_actual) {
      // (the task's last launch has no idle time after it and its entry is never used as a gap)
      x0 = i + 1 < len ? x0 : 0; x1 = i + 2 < len ? x1 : 0;
      bad_actual |= x0 < 0 || x1 < 0;
      h0w = static_cast<uint64_t>(x0) >= WIDE32 ? WIDE32 : static_cast<uint32_t>(x0);
      h1w = static_cast<uint64_t>(x1) >= WIDE32 ? WIDE32 : static_cast<uint32_t>(x1);
    }
    if (two) {
      if (lp_role) *reinterpret_cast<uint2*>(lp_e + base + i) = make_uint2(a0, a1);
      if (hp_role) *reinterpret_cast<uint4*>(hp_eg + base + i) = make_uint4(h0w, b0, h1w, b1);
    } else {
      if (lp_role) lp_e[base + i] = a0;
      if (hp_role) hp_eg[base + i] = make_uint2(h0w, b0);
    }
  };
  if (ids_vec) {
    for (; i0 + (PRED_READS - 1) * step + 1 < len; i0 += PRED_READS * step) {
      ulonglong2 v[PRED_READS];
      int64_t x[PRED_READS][2];
#pragma unroll
      for (int u = 0; u < PRED_READS; ++u) v[u] = load_once(reinterpret_cast<const ulonglong2*>(ids + base + i0 + u * step));
#pragma unroll
      for (int u = 0; u < PRED_READS; ++u) {
        x[u][0] = x[u][1] = 0;
        if (with_actual) { x[u][0] = actual[base + i0 + u * step]; x[u][1] = actual[base + i0 + u * step + 1]; }
      }
#pragma unroll
      for (int u = 0; u < PRED_READS; ++u) finish(i0 + u * step, true, v[u].x, v[u].y, x[u][0], x[u][1]);
    }
  }
  auto plain = [&](uint64_t i, bool two) {
    const uint64_t id0 = ids[base + i], id1 = two ? ids[base + i + 1] : 0;
    const int64_t x0 = with_actual ? actual[base + i] : 0, x1 = with_actual && two ? actual[base + i + 1] : 0;
    finish(i, two, id0, id1, x0, x1);
  };
  for (; i0 < len; i0 += step) plain(i0, i0 + 1 < len);
  if (lead && part0 == 0 && tid == PRED_THREADS - 1) plain(0, false);
  total = wave_sum_u64(total);
  if (lane_id() == 0) wave_tot[tid >> 6] = total;
  __syncthreads();
  if (tid == 0) {
    uint64_t sum = 0;
    for (int w = 0; w < PRED_THREADS / WAVE; ++w) sum += wave_tot[w];
    if (rl & ROLE_LP) atomicAdd(reinterpret_cast<unsigned long long*>(&lp_total[t]), static_cast<unsigned long long>(sum));
  }
  if (unknown) atomicOr(&ctrl->status, ERR_UNKNOWN_ID);
  if (bad_actual) atomicOr(&ctrl->status, ERR_ACTUAL_GAP);
  if (wide) atomicOr(&ctrl->wide, 1u);
}

// The replay for predictions that do not fit 32 bits (Ctrl::wide): one lane per scenario steps through
// its gaps literally, on the 64-bit arrays of k_gf_predict (a low-priority kernel's predicted duration is the
// difference of two prefix sums).  Rare and slow on purpose; results are those of the 32-bit kernels.
__global__ void __launch_bounds__(256)
k_gf_replay_wide(const uint64_t* __restrict__ off, const uint32_t* __restrict__ hp_task, const uint32_t* __restrict__ lp_task,
                 uint64_t n_scen, const uint64_t* __restrict__ gap_off, const int64_t* __restrict__ pe,
                 const int64_t* __restrict__ pg, const int64_t* __restrict__ actual, int64_t margin, int64_t min_gap,
                 uint32_t feedback, uint32_t* __restrict__ fill_count, int64_t* __restrict__ filled_ns,
                 int64_t* __restrict__ delay_out, uint64_t* __restrict__ placed_out, Ctrl* ctrl) {
  if ((ctrl->status & ~ERR_ACTUAL_GAP) || !ctrl->wide) return;   // (the one bit this kernel itself may set)
  const uint64_t s = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= n_scen) return;
  const uint32_t hp = hp_task[s], lp = lp_task[s];
  const uint64_t h0 = off[hp], H = off[hp + 1] - h0;
  const uint64_t l0 = off[lp], L = off[lp + 1] - l0;
  const uint64_t g0 = gap_off[s];
  uint64_t p = 0;
  int64_t consumed = 0, delay = 0;
  bool bad_actual = false;
  for (uint64_t i = 0; i + 1 < H; ++i) {
    const int64_t G = pg[h0 + i], a = actual[h0 + i];
    bad_actual |= a < 0;
    uint32_t c = 0;
    int64_t f = 0;
    if (G >= min_gap && G >= margin) {
      int64_t rem = G - margin;
      while (p < L) {
        const int64_t d = pe[l0 + p] - consumed;
        if (d > rem || (feedback && f >= a)) break;
        rem -= d; f += d; consumed += d;
        ++p; ++c;
      }
      if (f > a) delay += f - a;
    }
    fill_count[g0 + i] = c;
    filled_ns[g0 + i] = f;
  }
  if (bad_actual) atomicOr(&ctrl->status, ERR_ACTUAL_GAP);
  delay_out[s] = delay;
  placed_out[s] = p;
}

// MODE 0: the plan on predictions (fill counts, filled time, completion time of the low-priority task).
// MODE 1 / 2: the same decisions replayed against the idle times that occurred, without / with real-time
// feedback (the runtime-feedback paragraph of the paper's scheduling section): the first word of a
// high-priority entry is then the actual idle time; with feedback nothing more is issued into a gap once
// the time filled has reached it; what runs past it delays the high-priority task, and the sum of these
// delays is written in place of the completion time.
enum : int { LW_PLAN = 0, LW_REPLAY = 1, LW_REPLAY_FEEDBACK = 2 };

// ---------------------------------------------------------------------------------------------
// One wave per scenario, on the same 32-bit predictions.
//
// What a gap takes depends on where the queue stands after the gap before it: a scenario is one chain of dependent
// decisions, and with few scenarios the length of one link decides.  Here a link never leaves the registers.  The
// wave's lanes hold 63 consecutive entries of the queue as running sums from the window's start (win) and 64
// consecutive gaps (b1: one more than what may be filled, 0 for a gap that is skipped).  The position o in the window
// and the consumed time C are scalars.  "How far does the queue get in this gap" is one comparison of all lanes with
// C + b1 and a population count: entries already consumed compare true as well, so the count is the new position
// itself.  "Which gap takes something next" is one comparison of all lanes' C + b1 with the head's running sum: gaps
// that take nothing cost nothing.  The next entries of the queue and the next gaps are read ahead into registers.
//
// Running sums saturate at 2^32 - 1, which compares as "does not fit" (C + b1 saturates there too).  The lane behind
// the window holds that value, and so do entries behind the queue's end: a walk that stops at it has to look closer,
// at any other value it is done.  If the sums themselves passed 32 bits, the window is reloaded at the head, where
// C = 0 and everything that can fit is exact.
//
// What bounds it: with few scenarios the chain of one gap (eight steps that pass between the vector and the scalar unit; 100
// cycles per gap, the windows' ends included), with many the issue of
// scalar instructions (the gap's fourteen scalar instructions go through one port per SIMD).  A gap that takes the window's
// rest and ends inside the next window has a way of its own: with kernels of a fifth of a gap that is every twelfth gap, and the
// general loop goes through twice its instructions for it (ms with the loop / now: 64 scenarios of 1500 gaps 0.076 / 0.063,
// 16,384 of 4095 gaps 1.43 / 1.18, 6000 ragged ones of up to 2800 0.25 / 0.22, replay of 6000 of 2047 gaps with feedback 0.44 /
// 0.376). The 64-bit kernel above, which passes 64-bit sums through the LDS crossbar, takes 0.23 ms for the first of these, one
// lane each 3.2 ms for the second.  The loop written in assembly with a quarter fewer instructions per gap is no faster (call 97
// / 99 us).
constexpr int WW_THREADS = 256;
constexpr uint32_t WW_WIN = WAVE - 1;
constexpr int WW_BLOCKS = 4;   // blocks of 64 gaps per round (their reads are one round ahead)

__device__ __forceinline__ uint32_t wave_incl_scan_sat_u32(uint32_t v) {
  v = __builtin_elementwise_add_sat(v, dpp_or_zero<0x111, 0xf>(v));   // (see wave_incl_scan_u32)
  v = __builtin_elementwise_add_sat(v, dpp_or_zero<0x112, 0xf>(v));
  v = __builtin_elementwise_add_sat(v, dpp_or_zero<0x114, 0xf>(v));
  v = __builtin_elementwise_add_sat(v, dpp_or_zero<0x118, 0xf>(v));
  v = __builtin_elementwise_add_sat(v, dpp_or_zero<0x142, 0xa>(v));
  v = __builtin_elementwise_add_sat(v, dpp_or_zero<0x143, 0xc>(v));
  return v;
}

__device__ int llvm_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ uint32_t write_lane_u32(uint32_t v, uint32_t value, uint32_t dst) {   // v with lane dst replaced
  return static_cast<uint32_t>(llvm_writelane(static_cast<int>(value), static_cast<int>(dst), static_cast<int>(v)));
}
__device__ __forceinline__ uint32_t sat32(uint64_t v) { return v > WIDE32 ? WIDE32 : static_cast<uint32_t>(v); }

// Before the loop over the gaps that take something: it is 116 to 148 bytes long and runs as one wave's chain, so that it matters
// where the instructions lie in the 32 bytes that are fetched at a time.  Between byte 8 and 16 of such a piece is the best place
// in all of its forms; where the compiler happens to put it costs up to 7 %.  Gap fills in us, 256 scenarios of 65,535 gaps that
// never repeat, for starts at byte 0, 4, 8, 12, 16, 20, 24: by a wave 1532, 1564, 1473, 1489, 1466, 1487, 1558; by eight 1560,
// 1579, 1502, 1491, 1500, 1524, 1584. The instructions that fill the piece are run once per block of 64 gaps, so there should be
// few (where nearly every gap takes something, 256 long scenarios by eight waves: 358 us with three, 361 with four).
template <int TEAM>
__device__ __forceinline__ void place_loop() {
  if constexpr (TEAM > 1) asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
  else asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0");
}

// The wave's scenario: its own number, or what order holds at that place.  (Everything that is the same in the whole wave is kept
// in scalar registers: the scenario number has to be seen as one.)
__device__ __forceinline__ uint32_t scenario_of_wave(const GfOrder& order, uint32_t n_scen) {
  const uint32_t place = static_cast<uint32_t>(
      __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x * (WW_THREADS / WAVE) + threadIdx.x / WAVE)));
  if (!order.count || place >= n_scen) return place;
  const uint32_t lane = lane_id();
  const uint32_t upto = wave_incl_scan_u32(lane < GF_BUCKETS ? order.count[lane] : 0u);
  const uint32_t bucket = popc64(ballot(lane < GF_BUCKETS && upto <= place));
  const uint32_t longest = popc64(ballot(lane < GF_BUCKETS && upto == 0));
  if (popc64(ballot(lane < GF_BUCKETS && upto == n_scen)) + longest == GF_BUCKETS) return place;   // (one bucket holds them all)
  if (bucket >= GF_BUCKETS) return n_scen;   // (cannot happen: every scenario is on a list)
  const uint32_t before = bucket ? read_lane_u32(upto, bucket - 1) : 0u;
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(order.list[bucket * n_scen + (place - before)])));
}

// ---- what repeats is copied -------------------------------------------------------------------------------------------
//
// A service runs the same kernels pass after pass, so its predicted idle times repeat, and so do the queue's entries.  A gap's
// result follows from the queue's next entries and the idle time alone.  If the walk stands before gap a and entry ja, stood before
// gap a - D and entry ja - dq earlier, and from there on the idle times equal those D gaps earlier and the entries those dq entries
// earlier, everything that follows is what followed then: a unit of D gaps issues the same dq entries again.  The walk looks for
// such a place at multiples of the trace's period; from it on the inputs are compared, all of them, and the results copied.  No
// step of this waits for the one before, so it runs at the rate of the memory instead of at the length of a chain.
//
// Traces of passes reach such a place after two to five periods as a rule: whatever the queue's first entry was, it soon stands
// at one that only few of a pass's gaps can take.  Calls in us, walked to the end / with the copy: 256 scenarios of 65,535 gaps
// 705 / 347 (the slowest wave walks 21,000 gaps), 16,384 of 4095 7565 / 7130 (the walk 1170 / 775: 1100 gaps walked, 2600 copied,
// and the queue's 13,000 entries compared), 6000 ragged ones of up to 2800 396 / 379.  Kernels drawn at random never repeat and
// pay for the search: about 0.3 us a round while it lasts (24 rounds as a rule), then one comparison a round (the same calls 635
// / 656, 7755 / 7775, 386 / 387). The rounds without the search as a second copy of the code: 82 to 86 registers instead of 67 to
// 71, and both copies' loops are compiled worse (256 traces of 65,535 gaps that never repeat 1518 -> 1648 us, the step of 16,384
// 7760 -> 7960).
struct Repeat {
  uint32_t a, ja;         // the place
  uint32_t D, dq;         // gaps and entries of a unit (the unit before the place is the one that is copied)
  uint32_t x0;            // gaps from here on have no result yet
  uint32_t units, X;      // units compared and copied (0: there is nothing to copy), and the gap at which they end
};
struct RepeatSums {
  uint32_t c;             // entries issued
  uint64_t used, line;    // time filled; predicted time line (replay: delay)
  uint32_t bad_x, bad_y;  // the first gap and the first entry found to differ
};
constexpr uint32_t NOT_BAD = ~0u;
constexpr int REPEAT_BLOCKS = 2;   // blocks of 64 gaps and of 256 entries per stripe (four: 30 registers more, no faster)

// Four entries of a queue, which starts anywhere.
struct __attribute__((packed, aligned(4))) FourEntries { uint32_t e[4]; };

// One of `parts` waves: its share of the units, in stripes of BLOCKS times 64 gaps and 256 entries.  The sums are the lane's own.
template <int MODE, int BLOCKS>
__device__ __forceinline__ RepeatSums repeat_part(const Repeat& r, uint32_t part, uint32_t parts, uint32_t H, const uint2* __restrict__ trace,
                                                  const uint32_t* __restrict__ queue, uint32_t* fill_count, int64_t* filled_ns) {
  RepeatSums sum{0, 0, 0, NOT_BAD, NOT_BAD};
  const uint32_t lane = lane_id();
  const uint32_t end = r.X + 1 == H ? H : r.X;   // (the trace's last launch has no gap, but its time counts)
  // (of what lies before x0 only the idle times are compared)
  const uint32_t stride = 64 * BLOCKS * parts, step = stride % r.D;
  uint32_t at[BLOCKS];                           // place in the unit
#pragma unroll
  for (uint32_t k = 0; k < BLOCKS; ++k) at[k] = (64 * (BLOCKS * part + k) + lane) % r.D;
  const uint2* __restrict__ unit = trace + (r.a - r.D);
  const uint32_t* unit_c = fill_count + (r.a - r.D);
  const int64_t* unit_f = filled_ns + (r.a - r.D);
  for (uint32_t x1 = r.a + 64 * BLOCKS * part; x1 < end; x1 += stride) {
    uint2 t[BLOCKS];
    uint32_t g[BLOCKS], c[BLOCKS], f[BLOCKS];
#pragma unroll
    for (uint32_t k = 0; k < BLOCKS; ++k) {
      t[k] = trace[min_u32(x1 + 64 * k + lane, H - 1)];
      g[k] = unit[at[k]].y;
      c[k] = unit_c[at[k]];
      f[k] = static_cast<uint32_t>(unit_f[at[k]]);
    }
#pragma unroll
    for (uint32_t k = 0; k < BLOCKS; ++k) {
      const uint32_t x = x1 + 64 * k + lane;
      const bool gap = x < r.X, open = x >= r.x0;
      if (gap && t[k].y != g[k]) sum.bad_x = min_u32(sum.bad_x, x);
      if (gap && open) {
        fill_count[x] = c[k];
        filled_ns[x] = f[k];
        sum.c += c[k];
        sum.used += f[k];
      }
      if (MODE == LW_PLAN) {
        sum.line += (open && x < end ? static_cast<uint64_t>(t[k].x) : 0ull) + (open && gap ? static_cast<uint64_t>(t[k].y) : 0ull);
      } else {
        sum.line += open && gap && f[k] > t[k].x ? f[k] - t[k].x : 0u;
      }
      at[k] += step;
      at[k] -= at[k] >= r.D ? r.D : 0u;
    }
    if (ballot(sum.bad_x != NOT_BAD)) return sum;   // (the sums are of no use, and what comes behind is looked at again)
  }
  if (r.dq == 0) return sum;
  // (the entry behind the last unit's belongs to it too: it is the one that no longer fits)
  const uint32_t last = r.ja + r.units * r.dq;
  for (uint32_t y1 = r.ja + 256 * BLOCKS * part; y1 <= last; y1 += 4 * stride) {
    FourEntries now[BLOCKS], then[BLOCKS];
    uint32_t from[BLOCKS];
#pragma unroll
    for (uint32_t k = 0; k < BLOCKS; ++k) {
      from[k] = min_u32(y1 + 256 * k + 4 * lane, last);   // (up to three entries behind it are read, and their place is in the workspace)
      now[k] = *reinterpret_cast<const FourEntries*>(queue + from[k]);
      then[k] = *reinterpret_cast<const FourEntries*>(queue + (from[k] - r.dq));
    }
#pragma unroll
    for (uint32_t k = 0; k < BLOCKS; ++k)
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e)
        if (from[k] + e <= last && now[k].e[e] != then[k].e[e]) sum.bad_y = min_u32(sum.bad_y, from[k] + e);
    if (ballot(sum.bad_y != NOT_BAD)) return sum;
  }
  return sum;
}
// How many units hold, by the first places that differ (the first entry behind a unit belongs to that unit too).
__device__ __forceinline__ uint32_t units_that_hold(const Repeat& r, uint32_t bad_x, uint32_t bad_y) {
  uint32_t units = r.units;
  if (bad_x != NOT_BAD) units = min_u32(units, (bad_x - r.a) / r.D);
  if (bad_y != NOT_BAD) units = min_u32(units, bad_y > r.ja ? (bad_y - r.ja - 1) / r.dq : 0u);
  return units;
}
// Something differed: what holds is left, to be copied once more for the sums.  False if all of it holds.
__device__ __forceinline__ bool repeat_shorten(Repeat& r, const RepeatSums& part) {
  const uint32_t hold = units_that_hold(r, part.bad_x, part.bad_y);
  if (hold == r.units) return false;
  r.units = hold;
  r.X = r.a + hold * r.D;
  return true;
}
__device__ __forceinline__ uint32_t uniform(uint32_t v) {   // (v is the same in all lanes: kept in a scalar register)
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}
__device__ __forceinline__ uint32_t wave_total_u32(uint32_t v) { return read_lane_u32(wave_incl_scan_u32(v), WAVE - 1); }

struct RepeatTeam {   // (in LDS)
  Repeat rep;         // what the walking wave has found; no units: the others leave
  RepeatSums sum;
};
// All waves of a scenario: what repeats is compared and copied.  Returns the number of entries issued and the first places that
// differ; `used` and `line` are the lane's own, and the other waves' sums are added to lane 0 of the first.
template <int MODE, int TEAM>
__device__ __forceinline__ RepeatSums repeat_copy(const Repeat& rep, uint32_t wave, uint32_t H, const uint2* __restrict__ trace,
                                                  const uint32_t* __restrict__ queue, uint32_t* fill_count, int64_t* filled_ns,
                                                  RepeatTeam* team) {
  const uint32_t lane = lane_id();
  if (TEAM > 1) {
    if (threadIdx.x == 0) team->sum = RepeatSums{0, 0, 0, NOT_BAD, NOT_BAD};
    __syncthreads();
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // (the unit that is copied has been stored by the walk)
  RepeatSums part = repeat_part<MODE, REPEAT_BLOCKS>(rep, wave, TEAM, H, trace, queue, fill_count, filled_ns);
  if (TEAM > 1) {
    if (part.bad_x != NOT_BAD) atomicMin(&team->sum.bad_x, part.bad_x);
    if (part.bad_y != NOT_BAD) atomicMin(&team->sum.bad_y, part.bad_y);
    part.c = wave_total_u32(part.c);
    if (lane == 0) atomicAdd(&team->sum.c, part.c);
    if (wave != 0) {
      part.used = wave_sum_u64(part.used); part.line = wave_sum_u64(part.line);
      if (lane == 0) {
        atomicAdd(reinterpret_cast<unsigned long long*>(&team->sum.used), static_cast<unsigned long long>(part.used));
        atomicAdd(reinterpret_cast<unsigned long long*>(&team->sum.line), static_cast<unsigned long long>(part.line));
      }
    }
    __syncthreads();
    part.bad_x = uniform(team->sum.bad_x); part.bad_y = uniform(team->sum.bad_y); part.c = uniform(team->sum.c);
    if (wave == 0 && lane == 0) { part.used += team->sum.used; part.line += team->sum.line; }
    __syncthreads();
  } else {
    part.bad_x = ballot(part.bad_x != NOT_BAD) ? uniform(wave_min_u32(part.bad_x)) : NOT_BAD;
    part.bad_y = ballot(part.bad_y != NOT_BAD) ? uniform(wave_min_u32(part.bad_y)) : NOT_BAD;
    part.c = wave_total_u32(part.c);
  }
  return part;
}
// The waves of a scenario that do not walk: they copy what the walking wave finds until it finds no more.
template <int MODE, int TEAM>
__device__ __forceinline__ void repeat_helper(uint32_t wave, uint32_t H, const uint2* __restrict__ trace, const uint32_t* __restrict__ queue,
                                              uint32_t* fill_count, int64_t* filled_ns, RepeatTeam* team) {
  for (;;) {
    __syncthreads();
    Repeat rep = team->rep;
    rep = Repeat{uniform(rep.a), uniform(rep.ja), uniform(rep.D), uniform(rep.dq), uniform(rep.x0), uniform(rep.units), uniform(rep.X)};
    if (!rep.units) return;
    while (rep.X > rep.x0) {   // (as the walking wave does)
      const RepeatSums part = repeat_copy<MODE, TEAM>(rep, wave, H, trace, queue, fill_count, filled_ns, team);
      if (!repeat_shorten(rep, part)) break;
    }
  }
}

// Where it is worth the search.  The search costs a wave 1 to 2 us until there is a period and 0.4 us a note; 64 traces of 1500
// gaps (a call of 73 us) gain nothing by it, 6000 of up to 2800 gaps 396 -> 379 us.  A queue of a few passes is soon used up, or
// hardly moves.
constexpr uint32_t REPEAT_GAPS = 2048, REPEAT_ENTRIES = 1024;
// A wave by itself copies a gap in 9 to 16 cycles and walks one that takes nothing in 5, one that takes something in 100 and
// more: a unit is copied if at least every eighth of its gaps takes something (three traces of 12,192 gaps whose queue hardly
// moves, all copied 181 us, walked 157).  Eight waves copy one in 2 cycles, and copy whatever repeats.
constexpr uint32_t REPEAT_WORTH = 8;
constexpr uint32_t REPEAT_LEAST = 128;     // a shorter period counts as a multiple of it, so that a round has few places to look at
constexpr uint32_t REPEAT_NOTES = 48;      // places noted; the period is doubled at every 16th (at every eighth: 256 long traces 345 -> 367 us)
// Starts of a period (counted once) and repeats (twice) that may turn out to be none; one that held for REPEAT_ANCHOR gaps has
// paid for the search, and the count starts again.
constexpr uint32_t REPEAT_MISSES = 4;
// Gaps from a start without a period after which another start is looked for, and how often; then the search ends.  What comes
// before the first pass may be 2048 launches long, and a pass 4096.
constexpr uint32_t REPEAT_ANCHOR = 2048, REPEAT_ANCHORS = 2;

// The search, by the wave that walks.  Two idle times in a row that equal those at the anchor may be the start of the next pass,
// and are if 64 are equal.  From then on the wave notes, once a period, where the queue stands and what it holds there (a lane
// per note: the gap, the entry, a sum over the next 64 entries).
struct RepeatSearch {
  // Rounds that start before this gap are looked at; 0: the search is over.  (One comparison per round is what a trace pays that
  // never repeats, or that is too short.)
  uint32_t until;
  uint32_t misses = 0;
  uint32_t period = 0, next_place = 0, notes = 0, note_i = 0, note_j = 0, note_sum = 0;
  uint32_t anchor = 0;                                   // (what is needed until there is a period is kept in lanes too: scalar registers are few)
  // Where a round's gaps may be the start of the next pass (0: nowhere), and what has to be compared for it.
  struct Start { uint32_t at, pass0, pass1, anchor_q; };

  enum : uint32_t { A_GAP, A_ENTRY, A_G0, A_G1, A_NEXT, A_COUNT };
  __device__ __forceinline__ uint32_t anchor_of(uint32_t what) const { return read_lane_u32(anchor, what); }
  __device__ __forceinline__ static uint32_t sum_of(uint32_t e) { return wave_total_u32(e * ((2 * lane_id() + 1) * 0x9e3779b1u)); }

  __device__ __forceinline__ void miss(uint32_t times) {
    misses += times;
    until = misses >= REPEAT_MISSES ? 0u : until;
  }

  // The round's idle times (G) are at hand, its gaps not walked yet: what has to be compared is read now and looked at behind the
  // round.
  template <typename Entry>
  __device__ __forceinline__ Start look(uint32_t i0, uint32_t queue_at, uint32_t H, const uint2* __restrict__ trace,
                                        const uint32_t (&G)[WW_BLOCKS], Entry entry) {
    Start start{0, 0, 0, 0};
    if (period) return start;
    if (i0 >= anchor_of(A_NEXT)) {
      const uint32_t n = anchor_of(A_COUNT);
      anchor = write_lane_u32(anchor, i0, A_GAP);
      anchor = write_lane_u32(anchor, queue_at, A_ENTRY);
      anchor = write_lane_u32(anchor, read_lane_u32(G[0], 0), A_G0);
      anchor = write_lane_u32(anchor, read_lane_u32(G[0], 1), A_G1);
      anchor = write_lane_u32(anchor, n + 1 < REPEAT_ANCHORS ? i0 + REPEAT_ANCHOR : i0 + 2 * REPEAT_ANCHOR, A_NEXT);
      anchor = write_lane_u32(anchor, n + 1, A_COUNT);
      if (n == REPEAT_ANCHORS) { until = 0; return start; }
    }
    const uint32_t from = anchor_of(A_GAP), g0 = anchor_of(A_G0), g1 = anchor_of(A_G1);
    uint64_t alike[WW_BLOCKS], any = 0;
#pragma unroll
    for (uint32_t j = 0; j < WW_BLOCKS; ++j) {
      // (two ballots: lanes are read from their neighbours, so all have to take part)
      alike[j] = ballot(G[j] == g0) & ballot(from_next_lane(G[j]) == g1) & ~(j == 0 && i0 == from ? 1ull | 1ull << 63 : 1ull << 63);
      any |= alike[j];
    }
    if (any) {
#pragma unroll
      for (uint32_t j = 0; j < WW_BLOCKS; ++j)
        if (!start.at && alike[j]) start.at = i0 + 64 * j + static_cast<uint32_t>(__builtin_ctzll(alike[j]));
      const uint32_t lane = lane_id();
      start.pass0 = trace[from + lane].y;
      start.pass1 = trace[min_u32(start.at + lane, H - 1)].y;
      start.anchor_q = entry(anchor_of(A_ENTRY) + lane);
    }
    return start;
  }

  // Behind the round that started at gap `first`: count: entries that its gaps took, queue_at: where the queue stands.  Returns
  // what can be compared and copied (units == 0: nothing).
  template <int TEAM, typename Entry>
  __device__ __forceinline__ Repeat note(const Start& start, uint32_t first, uint32_t queue_at, uint32_t H, uint32_t L, uint32_t n_gaps,
                                         const uint32_t (&count)[WW_BLOCKS], Entry entry) {
    Repeat rep{0, 0, 0, 0, 0, 0, 0};
    const uint32_t lane = lane_id(), end = first + 64 * WW_BLOCKS;
    if (start.at) {
      if (ballot(start.at + lane < H && start.pass0 == start.pass1) == ~0ull) {
        const uint32_t from = anchor_of(A_GAP);
        note_i = from; note_j = anchor_of(A_ENTRY); note_sum = sum_of(start.anchor_q); notes = 1;
        period = start.at - from;
        if (period < REPEAT_LEAST) period *= (REPEAT_LEAST + period - 1) / period;
        next_place = from + period;   // (not before this round: a pass that starts in it is found in it)
      } else {
        miss(1);
      }
    }
    if (!period || next_place > end) return rep;
    while (next_place + period <= end) next_place += period;
    uint32_t behind = 0;   // entries issued from the place on
#pragma unroll
    for (uint32_t j = 0; j < WW_BLOCKS; ++j) behind += first + 64 * j + lane >= next_place ? count[j] : 0u;
    const uint32_t here_j = queue_at - wave_total_u32(behind), here_sum = sum_of(entry(here_j + lane));
    const uint64_t alike = ballot(lane < notes && note_sum == here_sum);
    if (alike) {
      const uint32_t n = 63u - static_cast<uint32_t>(__builtin_clzll(alike));
      rep.a = next_place; rep.ja = here_j;
      rep.D = rep.a - read_lane_u32(note_i, n); rep.dq = rep.ja - read_lane_u32(note_j, n);
      rep.x0 = end;
      const uint32_t wanted = (n_gaps - rep.a + rep.D - 1) / rep.D;
      const uint32_t there = rep.dq ? (L - 1 - rep.ja) / rep.dq : wanted;   // (units whose entries lie in the queue, with the one behind)
      rep.units = min_u32(wanted, there);
      rep.X = rep.units == wanted ? n_gaps : rep.a + rep.units * rep.D;
      if (rep.X <= rep.x0) rep.units = 0;
      if (there == 0) until = 0;   // (the queue ends first)
      if (TEAM == 1 && rep.dq < rep.D / REPEAT_WORTH) { rep.units = 0; until = 0; }
    }
    const uint32_t n = notes;
    note_i = write_lane_u32(note_i, next_place, n);
    note_j = write_lane_u32(note_j, here_j, n);
    note_sum = write_lane_u32(note_sum, here_sum, n);
    ++notes;
    period <<= (notes & 15) == 0 ? 1 : 0;     // (what comes back after c periods comes back after 2 c)
    until = notes >= REPEAT_NOTES ? 0u : until;
    next_place += period;
    return rep;
  }
};

// (completion_out receives the delay in the replay modes).  TEAM waves per scenario, of which the first walks and all copy what
// repeats; 0: one wave, and nothing is looked for.
template <int MODE, int TEAM>
__global__ void __launch_bounds__(TEAM <= 1 ? WW_THREADS : TEAM * WAVE)
k_gf_walk_wave(const uint64_t* __restrict__ off, const uint32_t* __restrict__ hp_task, const uint32_t* __restrict__ lp_task,
               uint32_t n_scen, const uint64_t* __restrict__ gap_off, const uint32_t* __restrict__ lp_e,
               const uint2* __restrict__ hp_eg, const uint64_t* __restrict__ lp_total, int64_t margin, int64_t min_gap,
               uint32_t* fill_count, int64_t* filled_ns, int64_t* __restrict__ completion_out,
               uint64_t* __restrict__ placed_out, const Ctrl* prof, uint64_t row_capacity, const GfOrder order, const Ctrl* ctrl) {
  // (with feedback the decisions follow the idle times that occurred, which do not repeat)
  constexpr bool REPEATS = TEAM > 0;
  static_assert(!REPEATS || MODE != LW_REPLAY_FEEDBACK, "decisions that do not repeat");
  if (ctrl->status || ctrl->wide || !may_follow(prof, row_capacity)) return;
  const uint32_t lane = lane_id();
  const uint32_t wave = TEAM <= 1 ? 0u : static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / WAVE)));
  const uint32_t s = TEAM <= 1 ? scenario_of_wave(order, n_scen) : blockIdx.x;
  if (s >= n_scen) return;
  const uint32_t hp = hp_task[s], lp = lp_task[s];
  const uint32_t h0 = static_cast<uint32_t>(off[hp]), H = static_cast<uint32_t>(off[hp + 1]) - h0;
  const uint32_t l0 = static_cast<uint32_t>(off[lp]), L = static_cast<uint32_t>(off[lp + 1]) - l0;
  const uint64_t g0 = gap_off[s];
  const uint32_t n_gaps = H > 0 ? H - 1 : 0;
  const uint32_t* __restrict__ queue = lp_e + l0;
  const uint2* __restrict__ trace = hp_eg + h0;
  const int64_t floor64 = min_gap > margin ? min_gap : margin;   // (32-bit idle times are below WIDE32)
  const uint32_t gap_floor = floor64 >= static_cast<int64_t>(WIDE32) ? WIDE32 : static_cast<uint32_t>(floor64);
  const uint32_t margin32 = margin >= static_cast<int64_t>(WIDE32) ? WIDE32 : static_cast<uint32_t>(margin);

  uint32_t wb = 0, o = 0, C = 0, sum = 0;    // window start, position in it, time consumed since its start, running sum of the head
  uint32_t win = 0, before = 0, r1 = 0;      // running sums of the window, and before each entry; the entries of the window after it
  // (read without a branch, so that the walk's loop stays free of divergent ones; what lies behind the end is told apart
  // when the entries are used, so that nothing waits for a read where it is issued)
  auto entry = [&](uint32_t j) -> uint32_t { return queue[j < L ? j : L - 1]; };
  // (behind the end: saturates, never fits)
  auto set_window = [&](uint32_t r) {
    win = wave_incl_scan_sat_u32(lane == WW_WIN || wb + lane >= L ? WIDE32 : r);
    before = dpp_or_zero<0x138, 0xf>(win);   // wave_shr:1
  };
  auto load_window = [&](uint32_t at) {
    wb = at; o = 0; C = 0;
    const uint32_t r0 = entry(at + lane);
    r1 = entry(at + WW_WIN + lane);
    set_window(r0);
  };
  __shared__ RepeatTeam team;
  if (TEAM > 1 && wave != 0) { repeat_helper<MODE, TEAM>(wave, H, trace, queue, fill_count + g0, filled_ns + g0, &team); return; }
  auto share = [&](const Repeat& rep) {
    if (threadIdx.x == 0) team.rep = rep;
    __syncthreads();
  };
  bool done = L == 0;    // the whole queue has been issued
  uint32_t f_last = 0;   // time filled in the gap that took the last of it
  if (!done) { load_window(0); sum = read_lane_u32(win, 0); }

  uint64_t time_line = 0, consumed = 0, delay = 0;   // (per lane; summed over the lanes at the end)
  RepeatSearch search;
  // (what lies behind a round can be copied)
  search.until = REPEATS && n_gaps >= REPEAT_GAPS && L >= REPEAT_ENTRIES ? n_gaps - 64 * WW_BLOCKS : 0u;

  uint32_t i0 = 0;
  for (;;) {
    Repeat rep{0, 0, 0, 0, 0, 0, 0};
    // (launches are read without a branch too, so that what is in flight can be counted: the lane behind the trace's end
    // reads its last launch again, and nothing of it is used)
    uint2 ahead[WW_BLOCKS];
#pragma unroll
    for (uint32_t j = 0; j < WW_BLOCKS; ++j) ahead[j] = H ? trace[min_u32(i0 + 64 * j + lane, H - 1)] : make_uint2(0, 0);
#pragma unroll
    for (uint32_t j = 0; j < WW_BLOCKS; ++j) asm volatile("" : "+v"(ahead[j].x), "+v"(ahead[j].y));   // (the loop starts with nothing in flight)
    while (i0 < H && !done) {
      uint32_t E[WW_BLOCKS], G[WW_BLOCKS], b1[WW_BLOCKS];   // (replay: E is the idle time that occurred)
#pragma unroll
      for (uint32_t j = 0; j < WW_BLOCKS; ++j) {
        E[j] = ahead[j].x; G[j] = ahead[j].y;
        b1[j] = (i0 + 64 * j + lane < n_gaps && G[j] >= gap_floor) ? G[j] - margin32 + 1 : 0u;
        if (MODE == LW_REPLAY_FEEDBACK) b1[j] = E[j] == 0 ? 0u : b1[j];   // (the next request is there at once: nothing is issued)
        asm volatile("" : "+v"(E[j]), "+v"(G[j]), "+v"(b1[j]));           // (waited for here, before the next round's reads go out)
      }
      __builtin_amdgcn_sched_barrier(0);
      // (the results of a round are stored without a branch, so that the wait for the next round's reads can leave them in
      // flight: lanes behind the last gap fall outside the buffer)
      const uint32_t left = n_gaps - min_u32(i0, n_gaps), gaps_here = min_u32(left, 64 * WW_BLOCKS);
      const bounded out_c = bounded_at(fill_count + g0 + i0, 4 * gaps_here), out_f = bounded_at(filled_ns + g0 + i0, 8 * gaps_here);
#pragma unroll
      for (uint32_t j = 0; j < WW_BLOCKS; ++j) ahead[j] = trace[min_u32(i0 + 64 * (WW_BLOCKS + j) + lane, H - 1)];
      const bool looking = REPEATS && i0 < search.until;
      RepeatSearch::Start start{0, 0, 0, 0};
      if (looking) start = search.look(i0, wb + o, H, trace, G, entry);
      uint32_t count[WW_BLOCKS];
#pragma unroll
      for (uint32_t j = 0; j < WW_BLOCKS; ++j) {
        const uint32_t i = i0 + 64 * j + lane;
        const bool has_gap = i < n_gaps;
        uint32_t my_c = 0, my_f = 0;
        if (!done) {
          uint32_t k = 0, lim = __builtin_elementwise_add_sat(b1[j], C);
          uint64_t takes = ballot(lim > sum);
          // (one way out of the loop, at its end, and the rare case inside it: otherwise the compiler carries flags and copies
          // through every gap)
          if (takes) {
            place_loop<TEAM>();
            do {
              k = static_cast<uint32_t>(__builtin_ctzll(takes));
              uint64_t todo = (~1ull) << k;
              // How far the queue gets: the entries (consumed ones too) that end within what may be filled; with feedback
              // an entry is issued only while the time filled before it is below the actual gap.
              const uint32_t limit = read_lane_u32(lim, k);
              uint64_t ends = ballot(win < limit);
              const uint32_t arrived = MODE == LW_REPLAY_FEEDBACK ? read_lane_u32(__builtin_elementwise_add_sat(E[j], C), k) : 0u;
              if (MODE == LW_REPLAY_FEEDBACK) ends &= ballot(before < arrived);   // (both are true up to some entry)
              uint32_t o2 = popc64(ends);
              uint32_t C2 = read_lane_u32(before, o2), sum2 = read_lane_u32(win, o2);   // (o2 >= 1: the head fits)
              // the common case: the gap ends inside the window, at an entry whose running sum is exact
              uint32_t c = o2 - o, f = C2 - C;
              if (__builtin_expect(sum2 != WIDE32, 1)) {
                o = o2; C = C2; sum = sum2;
              } else {
                // the rest: the gap reaches the window's end or the queue's, or the window has to be reloaded first
                uint32_t left = read_lane_u32(b1[j], k);
                const uint32_t actual = MODE == LW_REPLAY_FEEDBACK ? read_lane_u32(E[j], k) : 0u;
                bool ended = false;
                // (with feedback: nothing is issued after these)
                const bool over = MODE == LW_REPLAY_FEEDBACK && popc64(ballot(win < arrived)) < o2;
                if (o2 == WW_WIN && !over && wb + WW_WIN < L) {
                  // nearly all of these: the gap takes the rest of the window (c and f so far) and ends inside the next one
                  left -= f;
                  wb += WW_WIN;
                  set_window(r1);
                  r1 = entry(wb + WW_WIN + lane);
                  o2 = popc64(ballot(win < left));
                  if (MODE == LW_REPLAY_FEEDBACK) {
                    const uint32_t o3 = popc64(ballot(win < actual - f)) + 1;
                    o2 = o3 < o2 ? o3 : o2;
                  }
                  C2 = read_lane_u32(before, o2);
                  sum2 = read_lane_u32(win, o2);
                  ended = sum2 != WIDE32;
                  o = ended ? o2 : 0u; C = ended ? C2 : 0u; sum = sum2;
                  c += o; f += C;
                } else {
                  c = f = 0;
                }
                if (!ended) for (;;) {
                  if (static_cast<uint64_t>(C) + left > WIDE32) load_window(wb + o);
                  o2 = popc64(ballot(win < C + left));
                  bool stop = false;
                  if (MODE == LW_REPLAY_FEEDBACK) {
                    const uint32_t o3 = popc64(ballot(win < sat32(static_cast<uint64_t>(C) + (actual - f)))) + 1;
                    stop = o3 <= o2;
                    o2 = stop ? o3 : o2;
                  }
                  const uint32_t C3 = read_lane_u32(before, o2);
                  c += o2 - o; f += C3 - C; left -= C3 - C;
                  o = o2; C = C3;
                  if (wb + o >= L) { done = true; break; }
                  bool again = false;
                  if (o == WW_WIN) {   // the window is used up: the next one, in which this gap goes on
                    wb += WW_WIN; o = 0; C = 0;
                    set_window(r1);
                    r1 = entry(wb + WW_WIN + lane);
                    again = !stop;
                  }
                  sum = read_lane_u32(win, o);
                  if (sum == WIDE32 && C != 0) { load_window(wb + o); sum = read_lane_u32(win, 0); again = !stop; }
                  if (!again) break;
                }
                if (done) { f_last = f; todo = 0; }
              }
              my_c = write_lane_u32(my_c, c, k);
              my_f = write_lane_u32(my_f, f, k);
              lim = __builtin_elementwise_add_sat(b1[j], C);
              takes = ballot(lim > sum) & todo;
            } while (takes);
          }
          if (MODE == LW_PLAN) {
            consumed += my_f;
            // predicted time line: all launches of the block and the idle times after them, or, if the queue ran empty in
            // gap k, up to the launch before it
            const bool ran = !done || lane <= k, idled = !done || lane < k;
            time_line += (i < H && ran ? static_cast<uint64_t>(E[j]) : 0ull) + (has_gap && idled ? static_cast<uint64_t>(G[j]) : 0ull);
          } else {
            delay += my_f > E[j] ? my_f - E[j] : 0u;
          }
        }
        store_below(out_c, 256u * j + 4u * lane, my_c);
        store_below(out_f, 512u * j + 8u * lane, my_f, 0u);
        count[j] = my_c;
      }
      const uint32_t first = i0;
      i0 += 64 * WW_BLOCKS;
      if (looking && !done) {
        rep = search.note<TEAM>(start, first, wb + o, H, L, n_gaps, count, entry);
        if (rep.units) break;
      }
    }
    if (!REPEATS || !rep.units) break;
    if (TEAM > 1) share(rep);
    uint32_t queue_at = wb + o;   // (the window is read again behind the copy: it needs the registers)
    const uint32_t units = rep.units;
    while (rep.X > rep.x0) {
      const RepeatSums part = repeat_copy<MODE, TEAM>(rep, 0, H, trace, queue, fill_count + g0, filled_ns + g0, &team);
      if (!repeat_shorten(rep, part)) {
        if (MODE == LW_PLAN) time_line += part.line; else delay += part.line;
        consumed += part.used;
        i0 = rep.X;
        search.next_place = rep.X + search.period;
        queue_at = rep.X == n_gaps ? queue_at + part.c : rep.ja + rep.units * rep.dq;
        break;
      }
    }
    if (rep.units != units) {   // something differed: the walk goes on behind what held and looks for another period
      if (i0 < rep.x0 + REPEAT_ANCHOR) search.miss(2);
      else search.misses = 0;
      search.period = 0; search.anchor = 0;
    }
    if (i0 == n_gaps) { wb = queue_at; o = 0; break; }   // (the last launch's time has been added too)
    load_window(queue_at);
    sum = read_lane_u32(win, 0);
  }
  if (TEAM > 1) share(Repeat{0, 0, 0, 0, 0, 0, 0});
  for (uint32_t i = i0 + lane; i < n_gaps; i += WAVE) {   // (after the queue ran empty)
    fill_count[g0 + i] = 0;
    filled_ns[g0 + i] = 0;
  }
  int64_t result;
  if (MODE == LW_PLAN) {
    const uint64_t line = wave_sum_u64(time_line), used = wave_sum_u64(consumed);
    result = static_cast<int64_t>(done ? line + f_last : line + (lp_total[lp] - used));
  } else {
    result = static_cast<int64_t>(wave_sum_u64(delay));
  }
  if (lane == 0) {
    completion_out[s] = result;
    placed_out[s] = wb + o;
  }
}

constexpr int LW_THREADS = 256;
constexpr uint32_t LW_OPENS = 4, LW_TRIES = 4;     // per period (between two rounds of stream reads / result writes):
                                                   // gaps opened, and queue entries tried per gap opened
constexpr uint32_t LW_LP_CHUNK = 16, LW_LP_CAP = 32;   // low-priority ring: entries read at a time, capacity
constexpr uint32_t LW_HP_CHUNK = 8, LW_HP_CAP = 16;    // high-priority ring
constexpr uint32_t LW_OUT_CHUNK = 8, LW_OUT_CAP = 32;  // staged results
// The first rows of the low-priority ring are kept a second time behind its last row, so that the LW_TRIES entries
// from any position on are consecutive rows (one address, constant offsets).
constexpr uint32_t LW_LP_MIRROR = LW_TRIES - 1;
static_assert(LW_LP_MIRROR < LW_LP_CHUNK, "the rows that are mirrored land together");

struct LaneWalkSmem {   // [entry][lane]: a lane's entries fall on one bank whatever position it is at
  uint32_t lp[LW_LP_CAP + LW_LP_MIRROR][LW_THREADS];
  uint32_t hp_e[LW_HP_CAP][LW_THREADS];
  uint32_t hp_g[LW_HP_CAP][LW_THREADS];
  uint32_t out_c[LW_OUT_CAP][LW_THREADS];
  uint32_t out_f[LW_OUT_CAP][LW_THREADS];
};

// Writes the staged results of gaps [first, first + count) (global gap numbers) of the calling lane.
__device__ __forceinline__ void lw_store_scalar(const LaneWalkSmem& sm, uint32_t tid, uint32_t first, uint32_t count,
                                                uint32_t* __restrict__ fill_count, int64_t* __restrict__ filled_ns) {
  for (uint32_t k = 0; k < count; ++k) {
    const uint32_t at = first + k;
    fill_count[at] = sm.out_c[at & (LW_OUT_CAP - 1)][tid];
    filled_ns[at] = static_cast<int64_t>(sm.out_f[at & (LW_OUT_CAP - 1)][tid]);
  }
}

template <int MODE>
__global__ void __launch_bounds__(LW_THREADS)
k_gf_walk_lanes(const uint64_t* __restrict__ off, const uint32_t* __restrict__ hp_task, const uint32_t* __restrict__ lp_task,
                uint64_t n_scen, const uint64_t* __restrict__ gap_off, const uint32_t* __restrict__ lp_e,
                const uint2* __restrict__ hp_eg, const uint64_t* __restrict__ lp_total, int64_t margin, int64_t min_gap,
                uint32_t* __restrict__ fill_count, int64_t* __restrict__ filled_ns, int64_t* __restrict__ completion_out,
                uint64_t* __restrict__ placed_out, uint32_t vec_ok, const Ctrl* prof, uint64_t row_capacity, const Ctrl* ctrl) {
  extern __shared__ __align__(16) unsigned char lw_raw[];
  LaneWalkSmem& sm = *reinterpret_cast<LaneWalkSmem*>(lw_raw);
  if (ctrl->status || ctrl->wide || !may_follow(prof, row_capacity)) return;
  const uint32_t tid = threadIdx.x;
  const uint64_t s = static_cast<uint64_t>(blockIdx.x) * LW_THREADS + tid;
  const bool valid = s < n_scen;

  // positions are global element numbers (all below 2^32)
  uint32_t h0 = 0, hp_end = 0, l0 = 0, lp_end = 0, g_first = 0, n_gaps = 0;
  uint64_t total_lp = 0;
  if (valid) {
    const uint32_t hp = hp_task[s], lp = lp_task[s];
    h0 = static_cast<uint32_t>(off[hp]); hp_end = static_cast<uint32_t>(off[hp + 1]);
    l0 = static_cast<uint32_t>(off[lp]); lp_end = static_cast<uint32_t>(off[lp + 1]);
    g_first = static_cast<uint32_t>(gap_off[s]);
    n_gaps = hp_end > h0 ? hp_end - h0 - 1 : 0;
    total_lp = (MODE == LW_PLAN && lp_end > l0) ? lp_total[lp] : 0;
  }
  uint32_t hp_pos = h0, lp_pos = l0;                    // next entry of either stream
  uint32_t hp_landed = h0 & ~(LW_HP_CHUNK - 1), lp_landed = l0 & ~(LW_LP_CHUNK - 1);   // ring holds entries below these
  uint32_t hp_req = 0, lp_req = 0;
  bool hp_fly = false, lp_fly = false;
  uint4 hr[4], lr[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) hr[k] = lr[k] = make_uint4(0, 0, 0, 0);

  uint32_t g = g_first;              // global number of the next gap to report
  uint32_t flushed = g_first;        // results below this are in memory
  const uint32_t g_end = g_first + n_gaps;
  int64_t t_open = 0;                // predicted time line of the high-priority task
  uint32_t g_cur = 0;                // idle time of the gap opened last (its opening time is t_open - g_cur)
  int64_t completion;
  uint64_t consumed = 0;
  uint32_t rem = 0, rem_open = 0;    // what is left of the open gap's budget; the budget it opened with
  uint32_t lp_open = l0;             // position in the queue when the gap opened
  uint32_t ga = 0;                   // replay: the idle time that occurred after the launch whose gap is open
  int64_t delay = 0;                 // replay: by how much issued kernels ran past the gaps so far
  // a gap is used if it is at least min_gap and at least the margin long (32-bit idle times are below WIDE32)
  const int64_t floor64 = min_gap > margin ? min_gap : margin;
  const uint32_t gap_floor = floor64 >= static_cast<int64_t>(WIDE32) ? WIDE32 : static_cast<uint32_t>(floor64);
  const uint32_t margin32 = margin >= static_cast<int64_t>(WIDE32) ? WIDE32 : static_cast<uint32_t>(margin);
  bool in_gap = false;
  bool pending = false;               // a gap has closed and its result (c, f) is not staged yet
  bool finished = !valid || lp_end == l0;  // nothing left to step through (remaining gaps, if any, get zeros)

  for (;;) {
    // ---- once per period: park what was read, read on, write complete groups of results ----
    if (hp_fly) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t at = (hp_req + 2 * k) & (LW_HP_CAP - 1);
        sm.hp_e[at][tid] = hr[k].x; sm.hp_g[at][tid] = hr[k].y;
        sm.hp_e[at + 1][tid] = hr[k].z; sm.hp_g[at + 1][tid] = hr[k].w;
      }
      hp_landed = hp_req + LW_HP_CHUNK;
      hp_fly = false;
    }
    if (lp_fly) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t at = (lp_req + 4 * k) & (LW_LP_CAP - 1);
        const uint32_t v[4] = {lr[k].x, lr[k].y, lr[k].z, lr[k].w};
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
          sm.lp[at + i][tid] = v[i];
          if (at + i < LW_LP_MIRROR) sm.lp[LW_LP_CAP + at + i][tid] = v[i];
        }
      }
      lp_landed = lp_req + LW_LP_CHUNK;
      lp_fly = false;
    }
    if (!finished && hp_landed < hp_end && static_cast<int32_t>(hp_landed - hp_pos) <= static_cast<int32_t>(LW_HP_CAP - LW_HP_CHUNK)) {
      const uint4* src = reinterpret_cast<const uint4*>(hp_eg + hp_landed);
#pragma unroll
      for (int k = 0; k < 4; ++k) hr[k] = src[k];
      hp_req = hp_landed;
      hp_fly = true;
    }
    if (!finished && lp_landed < lp_end && static_cast<int32_t>(lp_landed - lp_pos) <= static_cast<int32_t>(LW_LP_CAP - LW_LP_CHUNK)) {
      const uint4* src = reinterpret_cast<const uint4*>(lp_e + lp_landed);
#pragma unroll
      for (int k = 0; k < 4; ++k) lr[k] = src[k];
      lp_req = lp_landed;
      lp_fly = true;
    }
    if (flushed < g && (flushed & (LW_OUT_CHUNK - 1))) {   // (first results of a scenario, up to a multiple of 8)
      const uint32_t to8 = LW_OUT_CHUNK - (flushed & (LW_OUT_CHUNK - 1));
      const uint32_t cnt = g - flushed < to8 ? g - flushed : to8;
      lw_store_scalar(sm, tid, flushed, cnt, fill_count, filled_ns);
      flushed += cnt;
    }
    while (flushed + LW_OUT_CHUNK <= g) {
      if (vec_ok) {
        const uint32_t at = flushed & (LW_OUT_CAP - 1);
        uint32_t cc[LW_OUT_CHUNK], ff[LW_OUT_CHUNK];
#pragma unroll
        for (uint32_t k = 0; k < LW_OUT_CHUNK; ++k) { cc[k] = sm.out_c[at + k][tid]; ff[k] = sm.out_f[at + k][tid]; }
        uint4* oc = reinterpret_cast<uint4*>(fill_count + flushed);
        oc[0] = make_uint4(cc[0], cc[1], cc[2], cc[3]);
        oc[1] = make_uint4(cc[4], cc[5], cc[6], cc[7]);
        uint4* of = reinterpret_cast<uint4*>(filled_ns + flushed);
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) of[k] = make_uint4(ff[2 * k], 0u, ff[2 * k + 1], 0u);
      } else {
        lw_store_scalar(sm, tid, flushed, LW_OUT_CHUNK, fill_count, filled_ns);
      }
      flushed += LW_OUT_CHUNK;
    }
    if (__all(finished)) break;

    // ---- one period: LW_OPENS times { stage the result of the gap that closed, take the next
    // high-priority launch and open its gap; LW_TRIES times try the head of the queue }.  Written
    // without branches; a lane whose ring is empty, or whose gap is still open when a new one could be
    // taken, simply idles in that sub-step. ----
    const uint32_t lp_lim = lp_landed < lp_end ? lp_landed : lp_end;   // tries look at entries below this
#pragma unroll
    for (uint32_t o = 0; o < LW_OPENS; ++o) {
      // the queue entries that the tries after this opening may look at, read ahead of the opening's own work
      uint32_t w[LW_TRIES];
#pragma unroll
      for (uint32_t k = 0; k < LW_TRIES; ++k) w[k] = sm.lp[(lp_pos & (LW_LP_CAP - 1)) + k][tid];
      {
        // the whole queue has been issued (noticed here, not in the tries): the open gap is its last, the time line and f
        // stay as they are from here on
        const bool emptied = in_gap && lp_pos == lp_end;
        pending = pending || emptied;
        in_gap = in_gap && !emptied;
        finished = finished || emptied;
        // what the gap that is open, or has just closed, took (the tries only move lp_pos and rem; a gap that was
        // skipped took nothing)
        const uint32_t c = lp_pos - lp_open, f = rem_open - rem;
        // (a staging slot that is written early is simply written again)
        sm.out_c[g & (LW_OUT_CAP - 1)][tid] = c;
        sm.out_f[g & (LW_OUT_CAP - 1)][tid] = f;
        g += pending ? 1u : 0u;
        consumed += pending ? f : 0u;
        if (MODE != LW_PLAN) delay += (pending && f > ga) ? static_cast<int64_t>(f - ga) : 0;
        const uint32_t E = sm.hp_e[hp_pos & (LW_HP_CAP - 1)][tid], G = sm.hp_g[hp_pos & (LW_HP_CAP - 1)][tid];
        // between gaps: the next high-priority launch runs, then its gap opens (the last launch has none)
        const bool idle = !finished && !in_gap;
        const bool at_end = idle && hp_pos == hp_end;
        const bool take = idle && !at_end && hp_pos < hp_landed;
        hp_pos += take ? 1u : 0u;
        const bool last = take && hp_pos == hp_end;
        const bool gap = take && !last;
        if (MODE == LW_PLAN) {
          t_open += take ? static_cast<int64_t>(E) : 0;
          t_open += gap ? static_cast<int64_t>(G) : 0;     // (the time line after the gap: the gap opened g_cur earlier)
          g_cur = gap ? G : g_cur;
        }
        const bool usable = gap && G >= gap_floor;
        if (MODE != LW_PLAN) ga = usable ? E : ga;
        in_gap = in_gap || usable;
        // a gap that is skipped is closed at once and reports zeros when the next one is opened
        pending = gap && !usable;
        rem = gap ? G - margin32 : rem;
        rem_open = gap ? rem : rem_open;
        lp_open = gap ? lp_pos : lp_open;
        finished = finished || at_end || last;
      }
      // In a gap: does the head of the queue fit into what is left?  Then the entry behind it, and so on: an entry is
      // tried only behind one that fit, so the k-th try of an opening looks at the k-th entry from where the queue stood,
      // and the tries end at the first entry that does not fit.  The running sums of those entries only grow (a sum
      // beyond 32 bits stays at the largest value, which no gap reaches), so the number of entries that fit is the
      // number of running sums within what is left, at most the entries that have landed.
      const int32_t room = static_cast<int32_t>(lp_lim - lp_pos);   // entries that have landed (<= 0: none)
      uint32_t run[LW_TRIES];
      run[0] = w[0];
#pragma unroll
      for (uint32_t k = 1; k < LW_TRIES; ++k) run[k] = __builtin_elementwise_add_sat(run[k - 1], w[k]);
      uint32_t n = 0;
#pragma unroll
      for (uint32_t k = 0; k < LW_TRIES; ++k) n += run[k] <= rem ? 1u : 0u;
      if (MODE == LW_REPLAY_FEEDBACK) {
        // (with feedback: the next high-priority request has arrived once the time filled reaches the actual gap;
        // an entry is issued only while the time filled before it is below that)
        const uint32_t f0 = rem_open - rem;
        uint32_t n2 = f0 < ga ? 1u : 0u;
#pragma unroll
        for (uint32_t k = 1; k < LW_TRIES; ++k) n2 += __builtin_elementwise_add_sat(f0, run[k - 1]) < ga ? 1u : 0u;
        n = n < n2 ? n : n2;
      }
      const int32_t capped = room < static_cast<int32_t>(LW_TRIES) ? room : static_cast<int32_t>(LW_TRIES);
      const uint32_t avail = capped > 0 ? static_cast<uint32_t>(capped) : 0u;
      const uint32_t nfit = in_gap ? (n < avail ? n : avail) : 0u;
      const bool close = in_gap && n < avail;   // an entry that was there did not fit: the gap is closed
      uint32_t taken = 0;
#pragma unroll
      for (uint32_t k = 0; k < LW_TRIES; ++k) taken = nfit > k ? run[k] : taken;
      rem -= taken;
      pending = pending || close;
      in_gap = in_gap && !close;
      lp_pos += nfit;
    }
  }

  if (!valid) return;
  const uint32_t c = lp_pos - lp_open, f = rem_open - rem;   // of the last gap that was opened
  if (pending) {
    sm.out_c[g & (LW_OUT_CAP - 1)][tid] = c;
    sm.out_f[g & (LW_OUT_CAP - 1)][tid] = f;
    ++g;
    consumed += f;
    if (MODE != LW_PLAN && f > ga) delay += static_cast<int64_t>(f - ga);
  }
  // what is still staged, then zeros for the gaps after the queue ran empty
  lw_store_scalar(sm, tid, flushed, g - flushed, fill_count, filled_ns);
  uint32_t z = g;
  while (z < g_end && (z & (LW_OUT_CHUNK - 1))) { fill_count[z] = 0; filled_ns[z] = 0; ++z; }
  if (vec_ok) {
    for (; z + LW_OUT_CHUNK <= g_end; z += LW_OUT_CHUNK) {
      uint4* oc = reinterpret_cast<uint4*>(fill_count + z);
      oc[0] = oc[1] = make_uint4(0, 0, 0, 0);
      uint4* of = reinterpret_cast<uint4*>(filled_ns + z);
      of[0] = of[1] = of[2] = of[3] = make_uint4(0, 0, 0, 0);
    }
  }
  for (; z < g_end; ++z) { fill_count[z] = 0; filled_ns[z] = 0; }
  // the whole queue has been issued: the last of it into the gap opened last, after which the time line stood still
  const bool done = lp_pos == lp_end;
  completion = done ? t_open - static_cast<int64_t>(g_cur) + static_cast<int64_t>(f) : t_open + static_cast<int64_t>(total_lp - consumed);
  completion_out[s] = MODE == LW_PLAN ? completion : delay;
  placed_out[s] = lp_pos - l0;
}


}  // namespace fikit
