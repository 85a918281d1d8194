// C ABI of the FIKIT trace-profiling and gap-fill library: argument checks, workspace
// carving and kernel sequencing.  All arithmetic of the method runs in the HIP kernels.
#include "fikit.h"

#include <hip/hip_runtime.h>

#include <chrono>
#include <cstring>
#include <mutex>
#include <thread>

#include "common.hip.h"
#include "gapfill_kernels.hip.h"
#include "profile_kernels.hip.h"
#include "sort_kernels.hip.h"
#include "stats_kernels.hip.h"
#include "task_kernels.hip.h"
#include "msd_kernels.hip.h"
#include "unit_kernels.hip.h"
#include "stream_kernels.hip.h"
#include "prio_kernels.hip.h"
#include "pairing_kernels.hip.h"
#include "merge_kernels.hip.h"

namespace {

using namespace fikit;

constexpr uint64_t MAX_ELEMS = (1ull << 32) - (1ull << 24);

#define FIKIT_HIP(expr)                           \
  do {                                            \
    if ((expr) != hipSuccess) {                   \
      (void)hipGetLastError();                    \
      return FIKIT_HIP_ERROR;                     \
    }                                             \
  } while (0)

// Launches of this thread since the last wait of a call, and how long it looked in the last one of many (see Reads::wait).
thread_local uint32_t t_launches = 0;
thread_local int64_t t_looked = 0;
#define FIKIT_COUNT_LAUNCH(...)      \
  do {                               \
    ++t_launches;                    \
    hipLaunchKernelGGL(__VA_ARGS__); \
  } while (0)

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
inline uint64_t align_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }
inline uint32_t blocks_for(uint64_t items, uint32_t per_block) {
  uint64_t b = (items + per_block - 1) / per_block;
  return static_cast<uint32_t>(b == 0 ? 1 : b);
}

// Carves consecutive 256-byte aligned regions out of the workspace.
struct Carver {
  uint64_t at = 0;
  uint64_t take(uint64_t bytes) {
    const uint64_t here = at;
    at = align_up(at + bytes, 256);
    return here;
  }
};

struct ProfileLayout {
  uint64_t ctrl, k0, k1, k2, e0, e1, g0, g1, tiles, hist, sums, bits, word_prefix, gflag, dcount, total;
  uint64_t is_long, mtiles, mflag, wflag, bsize, units, lists;   // long-task partition path; work lists
  uint64_t max_tiles, max_ptiles, n_words, max_units;
};

ProfileLayout profile_layout(uint64_t n, uint32_t n_tasks) {
  ProfileLayout L;
  Carver c;
  L.n_words = (n + 63) / 64;
  uint64_t big_tasks = n / (static_cast<uint64_t>(LEAF) + 1);
  if (big_tasks > n_tasks) big_tasks = n_tasks;
  L.max_tiles = n / TILE + big_tasks;
  L.ctrl = c.take(256);
  L.k0 = c.take(n * 8);
  // (six arrays, evenly spaced: rows of one-workgroup tasks are staged in them, see Staging)
  L.k1 = c.take(n * 8);      // long tasks: tile-ordered IDs; general path: keys (sorted in the end)
  L.e0 = c.take(n * 8);
  L.e1 = c.take(n * 8);      // also: first half of the rows that a long task's units stage
  L.g0 = c.take(n * 8);
  L.g1 = c.take(n * 8);      // also: second half of them
  L.k2 = c.take(n * 8 + 8);  // long tasks: tile-ordered values; general path: second key buffer, then segment starts (one word more)
  L.tiles = c.take((static_cast<uint64_t>(n_tasks) + 1) * 4);
  uint64_t long_tasks = n / (static_cast<uint64_t>(FUSE_MAX) + 1);
  if (long_tasks > n_tasks) long_tasks = n_tasks;
  L.max_ptiles = n / PT_TILE + long_tasks;
  {
    // digit counts and look-back words of the sort passes; before them the bucket boundaries of the long tasks' tiles live here
    const uint64_t a = L.max_tiles * (DIGIT_WORDS_PER_TILE * 4 + 256 * 8), b = L.max_ptiles * PT_ROWS * 2;
    L.hist = c.take(a > b ? a : b);
  }
  uint64_t longest = L.max_tiles * 256;
  if (longest < static_cast<uint64_t>(n_tasks) + 1) longest = static_cast<uint64_t>(n_tasks) + 1;
  if (longest < L.n_words) longest = L.n_words;
  L.sums = c.take((longest / SCAN_TILE + 2) * 4);
  L.bits = c.take(L.n_words * 8);
  L.word_prefix = c.take(L.n_words * 4);
  L.gflag = c.take(static_cast<uint64_t>(n_tasks) * 4);
  L.dcount = c.take((static_cast<uint64_t>(n_tasks) + 1) * 4);
  L.is_long = c.take((static_cast<uint64_t>(n_tasks) + 1) * 4);
  L.mtiles = c.take((static_cast<uint64_t>(n_tasks) + 1) * 4);
  L.mflag = c.take(static_cast<uint64_t>(n_tasks) * 4);
  L.wflag = c.take(static_cast<uint64_t>(n_tasks) * 4);
  L.bsize = c.take(long_tasks * MSD_SLOTS * 4);   // bucket sizes of the long tasks
  L.max_units = long_tasks * MSD_SLOTS;
  L.units = c.take(L.max_units * 4 * 6);   // start, length, task, row count, first row, buckets
  {
    const uint64_t longest_list = L.max_units > n_tasks ? L.max_units : n_tasks;
    L.lists = c.take(longest_list * 4 * 4);
  }
  L.total = c.at;
  return L;
}
static_assert(STAGING_ARRAYS == 6, "k1 .. k2");

// In-place exclusive prefix sum of `count` 32-bit words; the grand total goes to *d_total (may be null).
int scan_u32(uint32_t* d_data, uint64_t count, uint32_t* d_sums, uint64_t* d_total, hipStream_t st) {
  const uint32_t nb = blocks_for(count, SCAN_TILE);
  FIKIT_COUNT_LAUNCH(k_scan_reduce, dim3(nb), dim3(SCAN_BLOCK), 0, st, d_data, count, d_sums);
  FIKIT_COUNT_LAUNCH(k_scan_spine, dim3(1), dim3(SCAN_BLOCK), 0, st, d_sums, static_cast<uint64_t>(nb), d_total);
  FIKIT_COUNT_LAUNCH(k_scan_apply, dim3(nb), dim3(SCAN_BLOCK), 0, st, d_data, count, d_sums);
  FIKIT_HIP(hipGetLastError());
  return FIKIT_OK;
}

// 64-bit offsets and their total (ctrl->n_rows) from `count` 32-bit row counts, the last of which is 0; see k_row_offsets.
int row_offsets_enqueue(const uint32_t* d_counts, uint64_t count, uint32_t* d_sums, uint64_t* d_out, Ctrl* ctrl, hipStream_t st) {
  if (count <= ROW_SCAN_ONE) {
    FIKIT_COUNT_LAUNCH(k_row_offsets, dim3(blocks_for(count, ROW_SCAN_TILE)), dim3(1024), 0, st, d_counts, count, d_out, ctrl);
  } else {
    const uint32_t nb = blocks_for(count, SCAN_TILE);
    FIKIT_COUNT_LAUNCH(k_scan_reduce, dim3(nb), dim3(SCAN_BLOCK), 0, st, d_counts, count, d_sums);
    FIKIT_COUNT_LAUNCH(k_scan_spine, dim3(1), dim3(SCAN_BLOCK), 0, st, d_sums, static_cast<uint64_t>(nb), &ctrl->n_rows);
    FIKIT_COUNT_LAUNCH(k_row_offsets_apply, dim3(nb), dim3(SCAN_BLOCK), 0, st, d_counts, count, d_sums, d_out, ctrl);
  }
  FIKIT_HIP(hipGetLastError());
  return FIKIT_OK;
}

// ---- optional per-kernel timing (fikit_trace_*) ---------------------------------------------
// When enabled, every launch site records a HIP event on the caller's stream; at the end of
// the call the time between consecutive events is added to the entry of the launch that
// opened the interval.  Process-wide and not thread safe: a measurement aid, off by default.
constexpr int TRACE_MAX_MARKS = 192;
constexpr int TRACE_MAX_NAMES = 48;
struct TraceEntry { const char* name; double ms; int launches; };
bool g_trace_on = false;
uint32_t g_wait_limit = LOOK_SPIN_LIMIT;   // fikit_set_wait_limit
TraceEntry g_trace[TRACE_MAX_NAMES];
int g_trace_n = 0;

struct Tracer {
  hipStream_t st;
  hipEvent_t ev[TRACE_MAX_MARKS];
  const char* name[TRACE_MAX_MARKS];
  int n = 0;
  bool on;
  explicit Tracer(hipStream_t s, bool allowed = true) : st(s), on(allowed && g_trace_on) {}
  void mark(const char* what) {
    if (!on || n >= TRACE_MAX_MARKS) return;
    if (hipEventCreate(&ev[n]) != hipSuccess) { on = false; return; }
    (void)hipEventRecord(ev[n], st);
    name[n++] = what;
  }
  // Called once the stream has been synchronised (or on any early return).
  ~Tracer() {
    if (n == 0) return;
    if (n < TRACE_MAX_MARKS) mark("end");
    (void)hipStreamSynchronize(st);
    for (int i = 0; i + 1 < n; ++i) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, ev[i], ev[i + 1]) != hipSuccess) { (void)hipGetLastError(); continue; }
      int k = 0;
      while (k < g_trace_n && g_trace[k].name != name[i]) ++k;
      if (k == g_trace_n) {
        if (g_trace_n == TRACE_MAX_NAMES) continue;
        g_trace[g_trace_n++] = TraceEntry{name[i], 0.0, 0};
      }
      g_trace[k].ms += ms;
      g_trace[k].launches += 1;
    }
    for (int i = 0; i < n; ++i) (void)hipEventDestroy(ev[i]);
  }
};

int status_from_bits(uint32_t bits) {
  if (bits & (ERR_OFFSETS | ERR_TASK_INDEX | ERR_GAP_OFFSETS | ERR_ACTUAL_GAP | ERR_LP_LIST | ERR_ROWS | ERR_TOO_MANY)) return FIKIT_INVALID_ARG;
  if (bits & ERR_BAD_RECORD) return FIKIT_BAD_RECORD;
  if (bits & ERR_UNKNOWN_ID) return FIKIT_UNKNOWN_ID;
  if (bits & ERR_LP_LIMIT) return FIKIT_UNSUPPORTED;
  if (bits & ERR_WAIT) return FIKIT_HIP_ERROR;
  return FIKIT_OK;
}

// Where device words arrive on the host: a few pinned bytes per calling thread, allocated on its first call and freed when
// it ends.  A kernel writes them there, and behind them the number of the wait.
struct Mailbox {
  static constexpr size_t BYTES = 256, WAIT_AT = BYTES;
  unsigned char* at = nullptr;
  uint32_t waits = 0;      // of this thread so far
  hipEvent_t end = nullptr;
  int end_device = -1;
  // (another thread may be capturing a graph, which an allocation, a release, a question or a wait in the default mode would break)
  struct Relaxed {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    ~Relaxed() { if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode); }
  };
  ~Mailbox() {
    if (!at && !end) return;
    const Relaxed relaxed;
    if (end) (void)hipEventDestroy(end);
    if (at) (void)hipHostFree(at);
  }
  // The event that is recorded behind short calls, on the current device (null: there is none).  In the relaxed mode.
  hipEvent_t end_event() {
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return nullptr;
    if (end && end_device != device) {
      (void)hipEventDestroy(end);
      end = nullptr;
    }
    if (!end && hipEventCreateWithFlags(&end, hipEventDisableTiming) != hipSuccess) end = nullptr;
    end_device = device;
    return end;
  }
  unsigned char* get() {
    if (!at) {
      const Relaxed relaxed;
      void* p = nullptr;
      if (hipHostMalloc(&p, BYTES + 64, hipHostMallocPortable | hipHostMallocCoherent) == hipSuccess) {
        at = static_cast<unsigned char*>(p);
        std::memset(at, 0, BYTES + 64);
      }
      (void)hipGetLastError();
    }
    return at;
  }
};
thread_local Mailbox t_mailbox;

// Up to MOST reads of device words; they have arrived, and everything enqueued on the stream before is done, once wait() returns.
//
// One small kernel stores the words in the mailbox and the number of the wait behind them; the host looks at that number for a
// while, and lets the runtime wait for the stream if it takes longer.  A kernel and this take 8.7 us; the same words copied
// to pinned memory and the stream waited for 13.6 us with one copy, 16.2 us with two (a call that looks at two counts first: 14.3
// against 6.5 us).  Stores of the kernels before have left the caches of their dies when this kernel starts, as for any kernel
// that follows in the stream, so outputs are final for every stream, copy and thread.
//
// The runtime does not know then that the stream is empty, and a synchronisation of the caller's right behind the call pays for
// that.  It goes by the commands since its own last wait: up to RUNTIME_WAITS, the one of the wait among them, it waits itself,
// beyond them it leaves it to its handler thread, which takes 20 us longer.  (A synchronisation behind N empty kernels and a
// report that has been seen: 9 us up to N = 6, 24 us from 7 on; with an event recorded behind the report 5.6 us up to N = 5.)  So
// behind the last report of a call of few launches an event is recorded, which nobody waits for; in a longer one the runtime is
// asked whether the stream is empty, which sets the handler to work.  Asking takes 14 us of the host's time, which have to pass
// while the call does: the runtime is asked at once if the thread's last such call had it look for ASK_AT_ONCE_NS, otherwise once
// it has looked for ASK_NS (asked after 30 us in every call, those that end soon after are 12 to 14 us longer: merge of 22 tasks
// of 724 rows 64 / 78, step of 15 and 25 short tasks 66 / 78).
// Calls in us, with copies and the runtime's wait / reports alone / now:    one behind the other     each with a synchronisation
//   fikit_measure, 1000 launches                                              30 / 26 / 27             33 / 36 / 30
//   pairing of 16 scenarios                                                   33 / 27 / 28             36 / 36 / 30
//   step of a pair of 1000 launches                                           59 / 48 / 48             61 / 60 / 52
//   merge of 16 tasks of 20 rows (seven launches, over before it is asked)    51 / 34 / 35             54 / 47 / 47
//   priority queues, one scenario of two                                     122 / 100 / 105          123 / 129 / 111
//   merge of 20,000 tasks of 90 rows                                         286 / 233 / 233          296 / 245 / 241
//   step of 256 scenarios of 65,536 launches                                 365 / 341 / 350          370 / 375 / 352
//   priority queues, 4096 scenarios of three                                1057 / 1034 / 1042       1060 / 1071 / 1048
// (asked at once in every call: fikit_measure 38 to 44, the small merge 51 to 55, the step of a pair 47 to 51 one behind the
// other.)  The sort's way through a profile ends in a report too: the runtime's wait at its end took the 20 us longer (4 tasks of
// 98 launches of as many kernels 162 / 135, 144 with copies).
//
// The host gives way to other threads while it looks, which may have calls of their own to enqueue (us per step of a pair of 1000
// launches, all threads together, runtime's wait / looking without giving way / so: 8 threads on 2 processors 48 / 51 to 54 / 48,
// 4 on 1 processor 66 / 54 / 32, 1 thread 64 / 51 / 51).
struct Reads {
  static constexpr int MOST = 4;
  static constexpr int64_t LOOK_NS = 1000000;   // (the runtime's wait adds 4 us, which a call of this length no longer feels)
  static constexpr int64_t ASK_NS = 150000, ASK_AT_ONCE_NS = 40000;
  static constexpr uint32_t RUNTIME_WAITS = 8;
  static constexpr size_t place(size_t bytes) { return (bytes + 15) / 16 * 16; }
  hipStream_t st;
  unsigned char* box = t_mailbox.get();
  struct { void* to; const void* from; size_t bytes, at; } item[MOST];
  int n = 0;
  size_t used = 0;
  explicit Reads(hipStream_t s) : st(s) {}
  int add(void* to, const void* from, size_t bytes) {
    if (n == MOST || used + place(bytes) > Mailbox::BYTES || bytes % 4) return FIKIT_HIP_ERROR;   // (cannot happen: see below)
    item[n].to = to; item[n].from = from; item[n].bytes = bytes; item[n].at = used;
    used += place(bytes);
    ++n;
    return FIKIT_OK;
  }
  // (last: nothing of the call follows)
  int wait(bool last) {
    if (!box) {
      for (int i = 0; i < n; ++i) FIKIT_HIP(hipMemcpyAsync(item[i].to, item[i].from, item[i].bytes, hipMemcpyDeviceToHost, st));
      FIKIT_HIP(hipStreamSynchronize(st));
      return FIKIT_OK;
    }
    uint32_t* seen = reinterpret_cast<uint32_t*>(box + Mailbox::WAIT_AT);
    const uint32_t number = ++t_mailbox.waits;
    Report r{};
    for (int i = 0; i < n; ++i) {
      r.from[i] = static_cast<const uint32_t*>(item[i].from);
      r.to[i] = reinterpret_cast<uint32_t*>(box + item[i].at);
      r.words[i] = static_cast<uint32_t>(item[i].bytes / 4);
    }
    FIKIT_COUNT_LAUNCH(k_report, dim3(1), dim3(64), 0, st, r, seen, number);
    FIKIT_HIP(hipGetLastError());
    const auto from = std::chrono::steady_clock::now();
    auto looked = [&] { return std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now() - from).count(); };
    auto arrived = [&] { return __atomic_load_n(seen, __ATOMIC_ACQUIRE) == number; };
    const bool few = t_launches + 2 <= RUNTIME_WAITS, many = last && !few;   // (the event and the wait's own command)
    if (last) t_launches = 0;
    if (last && few) {
      const Mailbox::Relaxed relaxed;
      if (const hipEvent_t end = t_mailbox.end_event()) (void)hipEventRecord(end, st);   // (the thread's own: made anew it costs 1 us)
      (void)hipGetLastError();
    }
    bool to_ask = many;
    auto ask = [&] {
      to_ask = false;
      const Mailbox::Relaxed relaxed;
      (void)hipStreamQuery(st);   // (the answer is that it is not, which would stand as the last error)
      (void)hipGetLastError();
    };
    if (many && t_looked >= ASK_AT_ONCE_NS) ask();
    for (uint32_t looks = 1; !arrived(); ++looks) {
      __builtin_ia32_pause();   // (x86, as the hosts of these GPUs are)
      if (looks % 64 != 0) continue;
      std::this_thread::yield();
      const int64_t ns = looked();
      if (to_ask && ns > ASK_NS) ask();
      if (ns > LOOK_NS) {
        const Mailbox::Relaxed relaxed;
        FIKIT_HIP(hipStreamSynchronize(st));
        if (!arrived()) return FIKIT_HIP_ERROR;
        break;
      }
    }
    if (many) t_looked = looked();
    for (int i = 0; i < n; ++i) std::memcpy(item[i].to, box + item[i].at, item[i].bytes);
    return FIKIT_OK;
  }
};
static_assert(2 * Reads::place(sizeof(Ctrl)) <= Mailbox::BYTES && 3 * Reads::place(8) <= Mailbox::BYTES,
              "what one wait brings fits: two control blocks, or three counts");
static_assert(Reads::MOST == REPORT_READS && sizeof(Ctrl) % 4 == 0, "what a report holds");

int read_ctrl(const Ctrl* d_ctrl, Ctrl* h, hipStream_t st, bool last = true) {
  Reads r(st);
  if (int rc = r.add(h, d_ctrl, sizeof(Ctrl))) return rc;
  return r.wait(last);
}

template <int NT, int KPT, int DMAX, int WPE>
int launch_units(dim3 grid, const FusedArgs& args, hipStream_t st) {
  if (grid.x == 0) return FIKIT_OK;
  constexpr size_t lds = sizeof(UnitSmem<NT, KPT, DMAX>);
  static_assert(lds <= 160 * 1024, "fits a compute unit's LDS");
  auto kernel = k_unit_sorted<NT, KPT, DMAX, WPE>;
  FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
  FIKIT_COUNT_LAUNCH(kernel, dim3(xcd_grid(grid.x)), dim3(NT), lds, st, args);
  return FIKIT_OK;
}

template <int W>
int launch_prio_walk(hipStream_t st, const uint64_t* off, const uint32_t* hp_task, const uint64_t* lp_off,
                     const uint32_t* lp_task, const uint32_t* lp_prio, uint64_t n_scen, const uint64_t* gap_off,
                     const uint32_t* lp_e, const uint2* hp_eg, int64_t margin, int64_t min_gap, uint32_t* fill_count,
                     int64_t* filled_ns, uint64_t* placed, int64_t* placed_ns, uint32_t vec_ok, const Ctrl* ctrl) {
  FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_pf_walk<W>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                static_cast<int>(sizeof(PrioWalkSmem<W>))));
  FIKIT_COUNT_LAUNCH(k_pf_walk<W>, dim3(blocks_for(n_scen * W, PW_THREADS)), dim3(PW_THREADS), sizeof(PrioWalkSmem<W>), st, off,
                     hp_task, lp_off, lp_task, lp_prio, n_scen, gap_off, lp_e, hp_eg, margin, min_gap, fill_count, filled_ns,
                     placed, placed_ns, vec_ok, ctrl);
  return FIKIT_OK;
}

}  // namespace

extern "C" {

int fikit_version(void) { return 1; }

void fikit_set_wait_limit(uint32_t polls) { g_wait_limit = polls ? polls : LOOK_SPIN_LIMIT; }

void fikit_trace_enable(int on) {
  g_trace_on = on != 0;
  g_trace_n = 0;
}

int fikit_trace_read(int index, const char** name, double* total_ms, int* launches) {
  if (index >= 0 && index < g_trace_n) {
    if (name) *name = g_trace[index].name;
    if (total_ms) *total_ms = g_trace[index].ms;
    if (launches) *launches = g_trace[index].launches;
  }
  return g_trace_n;
}

const char* fikit_status_string(int status) {
  switch (status) {
    case FIKIT_OK: return "ok";
    case FIKIT_INVALID_ARG: return "invalid argument";
    case FIKIT_WORKSPACE_TOO_SMALL: return "workspace too small";
    case FIKIT_ROW_CAPACITY: return "row capacity exceeded";
    case FIKIT_BAD_RECORD: return "record with end_ns < start_ns";
    case FIKIT_UNKNOWN_ID: return "launch ID missing from its task's profile";
    case FIKIT_HIP_ERROR: return "HIP runtime error";
    case FIKIT_UNSUPPORTED: return "beyond a stated limit of this call (list entries and launches of a scenario number 2^32 or more)";
    case FIKIT_TOO_LARGE: return "input larger than the built-in scratch buffer of fikit_gapfill_static";
    default: return "unknown status";
  }
}

size_t fikit_profile_workspace_bytes(uint64_t n_records, uint32_t n_tasks) {
  if (n_records >= MAX_ELEMS) return 0;
  return static_cast<size_t>(profile_layout(n_records, n_tasks).total);
}

}  // extern "C"

namespace {

// Where the one-workgroup kernels of the profile put the predictions for a gap fill that follows (see FusedArgs).
struct PredEmit {
  const uint32_t* role;
  uint32_t* lp_e;
  uint2* hp_eg;
  uint64_t* lp_total;
  uint32_t* done;
  uint32_t predictor;
};

// fikit_profile; with `emit` the kernels that hold a whole task in one workgroup also write the task's predictions.  `begin` (may
// be null): the first checks of a gap fill that follows, which share a launch with the profile's if both are few.  ahead(tracer,
// reads, ctrl, any long tasks) enqueues what follows once the rows are final, and what it wants read back, before the host knows
// whether they are: *was_ahead says that they were (see may_follow).
template <typename Ahead>
int profile_run(const fikit_launch* d_records, uint64_t n_records, const uint64_t* d_task_offsets,
                uint32_t n_tasks, uint64_t* d_ids_out, fikit_row* d_rows_out, uint64_t row_capacity,
                uint64_t* d_task_row_offsets, uint64_t* h_n_rows, void* d_workspace, size_t workspace_bytes,
                void* hip_stream, const PredEmit* emit, const GfBegin* begin, Ahead ahead, bool* was_ahead) {
  *was_ahead = false;
  if (!h_n_rows) return FIKIT_INVALID_ARG;
  *h_n_rows = 0;
  if (!d_task_offsets || !d_task_row_offsets || !d_workspace) return FIKIT_INVALID_ARG;
  if (n_records >= MAX_ELEMS) return FIKIT_INVALID_ARG;
  if (n_records > 0 && (!d_records || n_tasks == 0)) return FIKIT_INVALID_ARG;
  if (row_capacity > 0 && !d_rows_out) return FIKIT_INVALID_ARG;
  if (!aligned(d_records, 16) || !aligned(d_task_offsets, 8) || !aligned(d_ids_out, 8) || !aligned(d_rows_out, 16) ||
      !aligned(d_task_row_offsets, 8) || !aligned(d_workspace, 256))
    return FIKIT_INVALID_ARG;
  const ProfileLayout L = profile_layout(n_records, n_tasks);
  if (workspace_bytes < L.total) return FIKIT_WORKSPACE_TOO_SMALL;

  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  unsigned char* ws = static_cast<unsigned char*>(d_workspace);
  Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + L.ctrl);
  const uint64_t n = n_records;
  uint64_t* ids = d_ids_out ? d_ids_out : reinterpret_cast<uint64_t*>(ws + L.k0);
  uint64_t* k1 = reinterpret_cast<uint64_t*>(ws + L.k1);
  uint64_t* k2 = reinterpret_cast<uint64_t*>(ws + L.k2);
  int64_t* e0 = reinterpret_cast<int64_t*>(ws + L.e0);
  int64_t* e1 = reinterpret_cast<int64_t*>(ws + L.e1);
  int64_t* g0 = reinterpret_cast<int64_t*>(ws + L.g0);
  int64_t* g1 = reinterpret_cast<int64_t*>(ws + L.g1);
  uint32_t* tiles = reinterpret_cast<uint32_t*>(ws + L.tiles);
  uint32_t* hist = reinterpret_cast<uint32_t*>(ws + L.hist);
  uint32_t* sums = reinterpret_cast<uint32_t*>(ws + L.sums);

  Tracer tr(st);
  tr.mark("setup");
  Ctrl h{};
  if (n == 0) {
    FIKIT_COUNT_LAUNCH(k_clear_ctrl, dim3(1), dim3(64), 0, st, ctrl);
    FIKIT_COUNT_LAUNCH(k_validate_offsets, dim3(blocks_for(n_tasks, 256)), dim3(256), 0, st, d_task_offsets, n_tasks, n, ctrl);
    FIKIT_COUNT_LAUNCH(k_fill_u32, dim3(blocks_for(2 * (static_cast<uint64_t>(n_tasks) + 1), 256)), dim3(256), 0, st,
                       reinterpret_cast<uint32_t*>(d_task_row_offsets), 2 * (static_cast<uint64_t>(n_tasks) + 1), 0u);
    FIKIT_HIP(hipGetLastError());
    if (int rc = read_ctrl(ctrl, &h, st)) return rc;
    return status_from_bits(h.status);
  }

  uint32_t* gflag = reinterpret_cast<uint32_t*>(ws + L.gflag);
  uint32_t* dcount = reinterpret_cast<uint32_t*>(ws + L.dcount);
  uint64_t* bits = reinterpret_cast<uint64_t*>(ws + L.bits);
  uint32_t* word_prefix = reinterpret_cast<uint32_t*>(ws + L.word_prefix);
  uint32_t* seg_start = reinterpret_cast<uint32_t*>(k2);

  // Short tasks with few distinct IDs: one workgroup each, records read once, rows staged.
  tr.mark("plan");
  uint32_t* lists = reinterpret_cast<uint32_t*>(ws + L.lists);
  uint32_t* is_long = reinterpret_cast<uint32_t*>(ws + L.is_long);
  uint32_t* mtiles = reinterpret_cast<uint32_t*>(ws + L.mtiles);
  uint32_t* mflag = reinterpret_cast<uint32_t*>(ws + L.mflag);
  uint32_t* ustart = reinterpret_cast<uint32_t*>(ws + L.units);
  uint32_t* ulen = ustart + L.max_units;
  uint32_t* utask = ulen + L.max_units;
  uint32_t* udcount = utask + L.max_units;
  uint32_t* urow = udcount + L.max_units;
  uint32_t* ubuckets = urow + L.max_units;
  uint32_t* bucket_size = reinterpret_cast<uint32_t*>(ws + L.bsize);
  uint32_t* ustage = bucket_size;   // (one word per unit slot too, which k_msd_units has done with)
  uint32_t* wflag = reinterpret_cast<uint32_t*>(ws + L.wflag);
  const bool few_tasks = n_tasks <= BEGIN_TASKS;
  if (few_tasks) {
    const ProfileBegin pb{n, FUSE_SMALL_MAX, FUSE_MID_MAX, FUSE_MAX, PT_TILE, gflag, dcount, lists, is_long, mtiles, wflag, ctrl};
    if (begin)
      FIKIT_COUNT_LAUNCH(k_step_begin, dim3(1), dim3(BEGIN_THREADS), 0, st, d_task_offsets, n_tasks, pb, *begin);
    else
      FIKIT_COUNT_LAUNCH(k_profile_begin, dim3(1), dim3(BEGIN_THREADS), 0, st, d_task_offsets, n_tasks, pb);
  } else {
    FIKIT_COUNT_LAUNCH(k_clear_ctrl, dim3(1), dim3(64), 0, st, ctrl);
    FIKIT_COUNT_LAUNCH(k_validate_offsets, dim3(blocks_for(n_tasks, 256)), dim3(256), 0, st, d_task_offsets, n_tasks, n, ctrl);
    FIKIT_COUNT_LAUNCH(k_classify, dim3(blocks_for(static_cast<uint64_t>(n_tasks) + 1, 256)), dim3(256), 0, st, d_task_offsets,
                       n_tasks, FUSE_SMALL_MAX, FUSE_MID_MAX, FUSE_MAX, gflag, dcount, lists, ctrl);
  }
  FIKIT_HIP(hipGetLastError());
  // Workgroups per class of task: their numbers if the host has to wait for them anyway (there may be long tasks, which are
  // launched for by number), otherwise what the launches suffice for.
  uint64_t n_class[3] = {n < n_tasks ? n : n_tasks, n / (FUSE_SMALL_MAX + 1), n / (FUSE_MID_MAX + 1)};
  if (n > FUSE_MAX) {
    tr.mark("host_sync");
    if (int rc = read_ctrl(ctrl, &h, st, false)) return rc;
    if (int rc = status_from_bits(h.status)) return rc;
    for (int k = 0; k < 3; ++k) n_class[k] = h.n_class[k];
  }
  uint16_t* bound = reinterpret_cast<uint16_t*>(hist);
  uint2* part_kg = reinterpret_cast<uint2*>(k2);
  auto small = k_task_fused<FUSE_S_THREADS, FUSE_SMALL_MAX / FUSE_S_THREADS, 256, 7168, FUSE_S_LB, FUSE_S_WPE>;
  auto medium = k_task_fused<FUSE_M_THREADS, FUSE_MAX / FUSE_M_THREADS, FUSE_M_DMAX, FUSE_M_HIST, 2, 4, FUSE_M_ESTATS>;
  auto mid = k_task_fused<512, 16, 256, 7168, 2, 4>;
  constexpr size_t mid_lds = sizeof(FusedSmem<512, 256, 7168>);
  FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(mid), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(mid_lds)));
  constexpr size_t small_lds = sizeof(FusedSmem<FUSE_S_THREADS, 256, 7168>),
                   medium_lds = sizeof(FusedSmem<FUSE_M_THREADS, FUSE_M_DMAX, FUSE_M_HIST, FUSE_M_ESTATS>);
  FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(small), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(small_lds)));
  FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(medium), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(medium_lds)));
  FusedArgs fa{};
  fa.rec = d_records; fa.off = d_task_offsets; fa.ids = ids; fa.e0 = e0; fa.g0 = g0; fa.key0 = k1;
  fa.staging = Staging{k1, (L.e0 - L.k1) / 8};
  fa.stage_a = e1; fa.stage_b = g1; fa.dcount = dcount; fa.gflag = gflag; fa.ctrl = ctrl;
  if (emit) {
    fa.pred_role = emit->role; fa.pred_lp_e = emit->lp_e; fa.pred_hp_eg = emit->hp_eg; fa.pred_lp_total = emit->lp_total;
    fa.pred_done = emit->done; fa.predictor = emit->predictor;
  }
  if (n_class[0]) {
    tr.mark("k_task_fused_small");
    fa.list = lists; fa.count = &ctrl->n_class[0]; fa.max_len = FUSE_SMALL_MAX;
    FIKIT_COUNT_LAUNCH(small, dim3(static_cast<uint32_t>(n_class[0])), dim3(FUSE_S_THREADS), small_lds, st, fa);
  }
  if (n_class[1]) {
    tr.mark("k_task_fused_mid");
    fa.list = lists + n_tasks; fa.count = &ctrl->n_class[1]; fa.max_len = FUSE_MID_MAX;
    FIKIT_COUNT_LAUNCH(mid, dim3(static_cast<uint32_t>(n_class[1])), dim3(512), mid_lds, st, fa);
  }
  if (n_class[2]) {
    tr.mark("k_task_fused_medium");
    fa.list = lists + 2 * static_cast<uint64_t>(n_tasks); fa.count = &ctrl->n_class[2]; fa.max_len = FUSE_MAX;
    FIKIT_COUNT_LAUNCH(medium, dim3(static_cast<uint32_t>(n_class[2])), dim3(FUSE_M_THREADS), medium_lds, st, fa);
  }
  FIKIT_HIP(hipGetLastError());
  uint64_t n_units = 0, n_msd_tiles = 0;
  if (h.n_long > 0) {
    // Long tasks: one pass over the records orders every tile by the top ID bits (IDs out in launch order on
    // the way), then the one-workgroup kernel on units of buckets, which gathers its launches from the tiles.
    const uint64_t n_long = h.n_long;
    n_units = n_long * MSD_SLOTS;
    if (n_units > L.max_units) return FIKIT_HIP_ERROR;   // cannot happen: a long task has more than FUSE_MAX launches
    if (!few_tasks) {
      tr.mark("plan");
      FIKIT_COUNT_LAUNCH(k_plan_msd, dim3(blocks_for(static_cast<uint64_t>(n_tasks) + 1, 256)), dim3(256), 0, st, d_task_offsets,
                         n_tasks, gflag, is_long, mtiles, wflag);
      if (int rc = scan_u32(is_long, static_cast<uint64_t>(n_tasks) + 1, sums, nullptr, st)) return rc;
      if (int rc = scan_u32(mtiles, static_cast<uint64_t>(n_tasks) + 1, sums, &ctrl->n_big_tiles, st)) return rc;
      tr.mark("host_sync");
      if (int rc = read_ctrl(ctrl, &h, st, false)) return rc;
    }
    n_msd_tiles = h.n_big_tiles;
    if (n_msd_tiles == 0 || n_msd_tiles > L.max_ptiles) return FIKIT_HIP_ERROR;
    tr.mark("k_tile_partition");
    FIKIT_COUNT_LAUNCH(k_msd_clear, dim3(blocks_for(n_units, 256)), dim3(256), 0, st, bucket_size, n_units, ctrl);
    FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_tile_partition), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  static_cast<int>(sizeof(PartSmem))));
    FIKIT_COUNT_LAUNCH(k_tile_partition, dim3(static_cast<uint32_t>(n_msd_tiles)), dim3(PT_THREADS), sizeof(PartSmem), st, d_records,
                       d_task_offsets, n_tasks, mtiles, is_long, ids, k1, part_kg, bound, bucket_size, wflag, ctrl);
    tr.mark("k_msd_units");
    FIKIT_COUNT_LAUNCH(k_msd_units, dim3(n_tasks), dim3(MSD_SLOTS), 0, st, d_task_offsets, n_tasks, is_long, mtiles, bucket_size, ustage, wflag,
                       ustart, ulen, utask, udcount, ubuckets, mflag, gflag, lists, static_cast<uint32_t>(n_units), ctrl);
    FusedArgs ua = fa;
    ua.pred_role = nullptr;   // (units are parts of tasks: their task's predictions are left to the gap fill)
    ua.ustart = ustart; ua.ulen = ulen; ua.utask = utask; ua.ubuckets = ubuckets; ua.tile_prefix = mtiles; ua.bound = bound;
    ua.tile_len = PT_TILE; ua.part_id = k1; ua.part_kg = part_kg; ua.mflag = mflag; ua.dcount = udcount;
    ua.staged = dcount; ua.ustage = ustage;   // (a long task's row count is 0 until k_msd_task_rows: the sum of what was staged)
    // (how many units of a class there can be: two neighbours of a task are longer than FUSE_SMALL_MAX together, or one
    // of them would have taken the other's first bucket)
    auto at_most = [&](uint64_t most) { return dim3(static_cast<uint32_t>(most < n_units ? most : n_units)); };
    // (the launch whose units hold most launches per ID of their tables first: a task that holds too many IDs is given up there,
    // and the other launches' units leave it alone)
    tr.mark("k_unit_sorted_mid");
    ua.list = lists + n_units; ua.count = &ctrl->n_class[1];
    if (int rc = launch_units<512, FUSE_MID_MAX / 512, UNIT_DMAX, 4>(at_most(n / (FUSE_SMALL_MAX + 1)), ua, st)) return rc;
    tr.mark("k_unit_sorted_small");
    ua.list = lists; ua.count = &ctrl->n_class[0];
    if (int rc = launch_units<512, FUSE_SMALL_MAX / 512, UNIT_DMAX, 6>(at_most(2 * (n / FUSE_SMALL_MAX) + n_long), ua, st)) return rc;
    // (streamed units behind these, so that a task that one of them has left to the sort, for holding too many IDs, is not streamed
    // in vain; units of more than FUSE_MID_MAX launches run beside them, see unit_streamed; a streamed unit has more than FUSE_MAX
    // launches, or is one of the MSD_SLOTS buckets of a task of more than UNIT_RUNS_MAX tiles)
    tr.mark("k_unit_large");
    FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_unit_large), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  static_cast<int>(UNIT_LARGE_LDS)));
    const uint64_t large_most = n / (FUSE_MID_MAX + 1) + n / (static_cast<uint64_t>(UNIT_RUNS_MAX) * PT_TILE) * MSD_SLOTS;
    ua.list = lists + 2 * n_units;
    FIKIT_COUNT_LAUNCH(k_unit_large, dim3(static_cast<uint32_t>(large_most < UNIT_LARGE_WORKGROUPS ? large_most : UNIT_LARGE_WORKGROUPS)),
                       dim3(SU_THREADS), UNIT_LARGE_LDS, st, ua, lists + 3 * n_units, static_cast<uint32_t>(n_units),
                       reinterpret_cast<uint2*>(e0), g0);
    tr.mark("plan");
    FIKIT_COUNT_LAUNCH(k_msd_task_rows, dim3(n_tasks), dim3(MSD_SLOTS), 0, st, n_tasks, is_long, mflag, udcount, urow, dcount);
    FIKIT_HIP(hipGetLastError());
  }

  // Row offsets and rows of the tasks so far.  They are the call's if no task is left to the general path, which is known
  // when the host has waited: the kernels look at the control block and do nothing if there is one.
  auto gather_rows = [&](uint64_t general_done) {
    tr.mark("k_gather_rows");
    FIKIT_COUNT_LAUNCH(k_gather_rows, dim3(xcd_grid(n_tasks)), dim3(256), 0, st, d_task_offsets, d_task_row_offsets, gflag, is_long,
                       n_units > 0 ? 1 : 0, fa.staging, n_tasks, d_rows_out, row_capacity, general_done, ctrl);
    if (n_units > 0)
      FIKIT_COUNT_LAUNCH(k_gather_units, dim3(xcd_grid(static_cast<uint32_t>(n_units))), dim3(256), 0, st, d_task_offsets, ulen,
                         utask, udcount, urow, ustage, mflag, d_task_row_offsets, e1, g1, static_cast<uint32_t>(n_units), d_rows_out, row_capacity,
                         general_done, ctrl);
  };
  const bool any_long = n_units > 0;
  if (!any_long && n_tasks <= ROWS_ONE_TASKS) {
    tr.mark("k_gather_rows");
    FIKIT_COUNT_LAUNCH(k_rows_one, dim3(n_tasks), dim3(256), 0, st, d_task_offsets, dcount, fa.staging, n_tasks, d_task_row_offsets, d_rows_out,
                       row_capacity, ctrl);
  } else {
    tr.mark("row_offsets");
    if (int rc = row_offsets_enqueue(dcount, static_cast<uint64_t>(n_tasks) + 1, sums, d_task_row_offsets, ctrl, st)) return rc;
    gather_rows(0);
  }
  FIKIT_HIP(hipGetLastError());
  {
    Reads reads(st);
    if (int rc = ahead(tr, reads, ctrl, any_long)) return rc;
    tr.mark("host_sync");
    if (int rc = reads.add(&h, ctrl, sizeof(Ctrl))) return rc;
    if (int rc = reads.wait(true)) return rc;
  }
  if (int rc = status_from_bits(h.status)) return rc;
  if (h.n_general == 0) {
    *h_n_rows = h.n_rows;
    if (h.n_rows > row_capacity) return FIKIT_ROW_CAPACITY;
    *was_ahead = true;
    return FIKIT_OK;
  }
  const uint64_t n_general = h.n_general;
  t_launches += Reads::RUNTIME_WAITS;   // (that was not the call's last wait)
  if (n_units > 0) {
    tr.mark("k_long_general_values");
    FIKIT_COUNT_LAUNCH(k_long_general_values, dim3(static_cast<uint32_t>(n_msd_tiles)), dim3(256), 0, st, d_records, d_task_offsets,
                       n_tasks, mtiles, gflag, wflag, ids, k1, part_kg, e0, g0);
  }
  uint64_t n_heads = 0;

  {
    // General path: per-launch values are in memory (written by whichever kernel gave the task up);
    // sort by ID, find the segment heads.
    tr.mark("plan");
    FIKIT_COUNT_LAUNCH(k_plan_tiles, dim3(blocks_for(static_cast<uint64_t>(n_tasks) + 1, 256)), dim3(256), 0, st,
                       d_task_offsets, n_tasks, gflag, tiles, ctrl);
    if (int rc = scan_u32(tiles, static_cast<uint64_t>(n_tasks) + 1, sums, &ctrl->n_big_tiles, st)) return rc;
    tr.mark("host_sync");
    if (int rc = read_ctrl(ctrl, &h, st, false)) return rc;
    if (int rc = status_from_bits(h.status)) return rc;
    const uint64_t n_big_tiles = h.n_big_tiles;
    if (n_big_tiles > L.max_tiles) return FIKIT_HIP_ERROR;  // cannot happen for valid offsets

    // keys start in k1 (in whatever order each task's triples were handed over) and end there sorted, payload in e0 / g0
    FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_leaf_sort), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  static_cast<int>(sizeof(LeafSmem))));
    tr.mark("k_leaf_sort");
    FIKIT_COUNT_LAUNCH(k_leaf_sort, dim3(xcd_grid(n_tasks)), dim3(LEAF_THREADS), sizeof(LeafSmem), st, d_task_offsets, n_tasks, gflag, k1,
                       k1, e0, g0, ctrl);
    FIKIT_HIP(hipGetLastError());
    // Eight stable passes over the eight key bytes sort any keys.  Kernel IDs are hashes: a task's distinct IDs
    // almost always differ in their upper four bytes already, so four passes over those are tried first; the
    // head search below also notices keys that are still out of order, and then all eight passes are run on
    // what the four left (any order of the (key, values) triples is a valid start).
    FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_onesweep_pass), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  static_cast<int>(sizeof(TileSmem))));
    uint32_t* digit_counts = hist;                                                    // [tile][DIGIT_WORDS_PER_TILE]
    unsigned long long* look = reinterpret_cast<unsigned long long*>(ws + L.hist + L.max_tiles * DIGIT_WORDS_PER_TILE * 4);   // [tile][256]
    uint32_t* tickets = wflag;                                                        // one per task (the long-task path is done with this array)
    // Four passes over four key bytes, least significant first; each pass is one launch (see sort_kernels.hip.h).
    auto sort_passes = [&](int first_byte) -> int {
      uint64_t *kin = k1, *kout = k2;
      int64_t *ein = e0, *eout = e1, *gin = g0, *gout = g1;
      const uint32_t nt = static_cast<uint32_t>(n_big_tiles);
      tr.mark("k_digit_hist");
      FIKIT_COUNT_LAUNCH(k_fill_u32, dim3(blocks_for(n_big_tiles * DIGIT_WORDS_PER_TILE, 1024)), dim3(256), 0, st, digit_counts,
                         n_big_tiles * DIGIT_WORDS_PER_TILE, 0u);
      FIKIT_COUNT_LAUNCH(k_digit_hist, dim3(nt), dim3(256), 0, st, d_task_offsets, n_tasks, tiles, kin, first_byte, digit_counts);
      FIKIT_COUNT_LAUNCH(k_digit_bases, dim3(n_tasks), dim3(256), 0, st, n_tasks, tiles, digit_counts);
      for (int pass = 0; pass < SORT_PASSES_PER_ROUND; ++pass) {
        tr.mark("k_onesweep_pass");
        FIKIT_COUNT_LAUNCH(k_fill_u32, dim3(blocks_for(n_big_tiles * 512, 1024)), dim3(256), 0, st, reinterpret_cast<uint32_t*>(look),
                           n_big_tiles * 512, 0u);
        FIKIT_COUNT_LAUNCH(k_fill_u32, dim3(blocks_for(n_tasks, 1024)), dim3(256), 0, st, tickets, static_cast<uint64_t>(n_tasks), 0u);
        FIKIT_COUNT_LAUNCH(k_onesweep_pass, dim3(onesweep_grid(nt)), dim3(TILE_THREADS), sizeof(TileSmem), st, d_task_offsets, n_tasks,
                           tiles, digit_counts, pass, 8 * (first_byte + pass), nt, tickets, look, kin, kout, ein, eout, gin, gout, g_wait_limit, ctrl);
        FIKIT_HIP(hipGetLastError());
        uint64_t* tk = kin; kin = kout; kout = tk;
        int64_t* t = ein; ein = eout; eout = t;
        t = gin; gin = gout; gout = t;
      }
      return FIKIT_OK;   // (an even number of passes: keys and values end in the arrays they started in)
    };
    auto find_heads = [&]() -> int {
      tr.mark("heads");
      FIKIT_COUNT_LAUNCH(k_head_bits, dim3(blocks_for(n, 256)), dim3(256), 0, st, k1, n, d_task_offsets, n_tasks, gflag, bits, ctrl);
      FIKIT_COUNT_LAUNCH(k_popcount_words, dim3(blocks_for(L.n_words, 256)), dim3(256), 0, st, bits, L.n_words, word_prefix);
      if (int rc = scan_u32(word_prefix, L.n_words, sums, &ctrl->n_heads, st)) return rc;
      tr.mark("host_sync");
      if (int rc = read_ctrl(ctrl, &h, st, false)) return rc;
      return status_from_bits(h.status);   // (a wait of the sort that ran out)
    };
    if (n_big_tiles > 0)
      if (int rc = sort_passes(4)) return rc;
    if (int rc = find_heads()) return rc;
    if (h.wide) {
      FIKIT_COUNT_LAUNCH(k_fill_u32, dim3(1), dim3(64), 0, st, &ctrl->wide, static_cast<uint64_t>(1), 0u);
      if (int rc = sort_passes(0)) return rc;   // all eight bytes, least significant first
      if (int rc = sort_passes(4)) return rc;
      if (int rc = find_heads()) return rc;
      if (h.wide) return FIKIT_HIP_ERROR;   // cannot happen: eight passes sort
    }
    n_heads = h.n_heads;
    tr.mark("heads");
    FIKIT_COUNT_LAUNCH(k_general_row_counts, dim3(blocks_for(n_tasks, 256)), dim3(256), 0, st, d_task_offsets, n_tasks, gflag,
                       bits, word_prefix, n, static_cast<uint32_t>(n_heads), dcount);
  }

  // Row offsets of every task, and the total.
  tr.mark("row_offsets");
  if (int rc = scan_u32(dcount, static_cast<uint64_t>(n_tasks) + 1, sums, &ctrl->n_rows, st)) return rc;
  FIKIT_COUNT_LAUNCH(k_widen_offsets, dim3(blocks_for(static_cast<uint64_t>(n_tasks) + 1, 256)), dim3(256), 0, st, dcount,
                     static_cast<uint64_t>(n_tasks) + 1, d_task_row_offsets);
  tr.mark("host_sync");
  if (int rc = read_ctrl(ctrl, &h, st, false)) return rc;
  const uint64_t n_rows = h.n_rows;
  *h_n_rows = n_rows;
  if (n_rows > row_capacity) return FIKIT_ROW_CAPACITY;

  gather_rows(n_general);
  if (n_heads > 0) {
    tr.mark("seg_starts");
    FIKIT_COUNT_LAUNCH(k_seg_starts, dim3(blocks_for(L.n_words, 256)), dim3(256), 0, st, bits, word_prefix, L.n_words, n, n_heads,
                       seg_start);
    tr.mark("k_stats_small");
    FIKIT_COUNT_LAUNCH(k_stats_small, dim3(blocks_for(n_heads, 4)), dim3(256), 0, st, seg_start, n_heads, d_task_offsets,
                       n_tasks, k1, e0, g0, bits, word_prefix, n, dcount, d_rows_out);
    // rows with long segments: by work list (the staging areas e1 / g1 are free once the rows are gathered)
    tr.mark("k_stats_lists");
    uint32_t* rlist = reinterpret_cast<uint32_t*>(e1);
    FIKIT_COUNT_LAUNCH(k_fill_u32, dim3(1), dim3(64), 0, st, &ctrl->n_class[0], static_cast<uint64_t>(2), 0u);
    FIKIT_COUNT_LAUNCH(k_stats_lists, dim3(blocks_for(n_heads, 256)), dim3(256), 0, st, seg_start, n_heads, d_task_offsets,
                       n_tasks, rlist, ctrl);
    tr.mark("k_stats_big");
    const uint32_t big_grid = static_cast<uint32_t>(n_heads < 4096 ? n_heads : 4096);
    const uint32_t huge_grid = static_cast<uint32_t>(n_heads < 512 ? n_heads : 512);
    FIKIT_COUNT_LAUNCH(k_stats_big<BIG_THREADS>, dim3(big_grid), dim3(BIG_THREADS), 0, st, seg_start, n_heads, d_task_offsets,
                       n_tasks, k1, e0, g0, bits, word_prefix, n, dcount, d_rows_out, rlist, &ctrl->n_class[0], 0u);
    tr.mark("k_stats_huge");
    FIKIT_COUNT_LAUNCH(k_stats_big<HUGE_THREADS>, dim3(huge_grid), dim3(HUGE_THREADS), 0, st, seg_start, n_heads,
                       d_task_offsets, n_tasks, k1, e0, g0, bits, word_prefix, n, dcount, d_rows_out, rlist, &ctrl->n_class[1],
                       1u);
  }
  FIKIT_HIP(hipGetLastError());
  Reads end(st);
  return end.wait(true);
}

}  // namespace

extern "C" {

int fikit_profile(const fikit_launch* d_records, uint64_t n_records, const uint64_t* d_task_offsets,
                  uint32_t n_tasks, uint64_t* d_ids_out, fikit_row* d_rows_out, uint64_t row_capacity,
                  uint64_t* d_task_row_offsets, uint64_t* h_n_rows, void* d_workspace, size_t workspace_bytes,
                  void* hip_stream) {
  bool was_ahead;
  return profile_run(d_records, n_records, d_task_offsets, n_tasks, d_ids_out, d_rows_out, row_capacity, d_task_row_offsets,
                     h_n_rows, d_workspace, workspace_bytes, hip_stream, nullptr, nullptr,
                     [](Tracer&, Reads&, const Ctrl*, bool) { return FIKIT_OK; }, &was_ahead);
}

// The per-launch arrays of the gap fill are read in 64-byte pieces that may reach past the last launch.
constexpr uint64_t GF_PAD = 256;
// From this many scenarios on, one lane steps through a scenario (k_gf_walk_lanes), below it a wave (k_gf_walk_wave).  The
// lanes' time hardly depends on how many there are (to 65,536); the waves' grows with them, and with the gaps that take
// something.  Traces of 4096 and queues of 16,384 launches: the lanes 3.3 ms, the waves 0.08 ms per 1024 scenarios once the chip
// is full (1.18 ms against 3.2 ms at 16,384).  Calls over shorter tasks, waves / lanes in ms (gap fill; replay with feedback):
//   1024 gaps that take about one kernel each   16,384: 0.53 / 0.71; 0.64 / 0.74   24,000: 0.74 / 0.82; 0.89 / 0.86
//                                               32,000: 0.94 / 0.95; 1.14 / 0.99
//   512 gaps that take about ten each           16,384: 0.58 / 1.08; 0.65 / 1.12   32,000: 1.05 / 1.33; 1.19 / 1.38
//   2048 gaps of which few take anything        16,384: 0.39 / 1.11; 0.44 / 1.17   32,000: 0.72 / 1.58; 0.80 / 1.48
// The line lies where the first of these shapes has the waves and the lanes level; with feedback it has from about 24,000 scenarios
// on, but what gaps take is not known when the line is drawn.
constexpr uint64_t GF_LANES_MIN_SCENARIOS = 32768;
// Up to this many scenarios of traces of so many launches on average, a workgroup takes each: one of its waves walks, all copy what
// repeats.  Three workgroups of eight waves are on a compute unit at a time, so the 769th waits until a scenario is through (traces
// and queues of 16,384 launches that never repeat, in us by a wave / by a workgroup each: 768 scenarios 441 / 455, 784 429 / 563,
// 1024 447 / 700).  Shorter traces are copied fast enough by one wave, and the walk by the first of several is 2 to 4 % slower
// (queues four times as long as the traces, repeating, 16 scenarios: 4096 launches 195 / 185, 8192 190 / 154, 16,384 265 / 176,
// 32,768 381 / 201; 256 scenarios: 222 / 223, 249 / 231, 310 / 263, 439 / 273; never repeating: 334 / 341, 618 / 634, 1195 /
// 1228, 2320 / 2387).  Of 256 scenarios of 65,535 gaps, four waves take 382 us, eight 355, sixteen 341, but of workgroups of
// sixteen waves only 256 would be there at a time.
constexpr uint64_t GF_TEAM_SCENARIOS = 768, GF_TEAM_LAUNCHES = 8192;
constexpr int GF_TEAM_WAVES = 8;
// From this average on some traces are long enough for the search (if lengths are spread up to twice the average).  The walk with
// it has 67 registers instead of 54, which many scenarios feel.  Without / with it in us: 12,000 scenarios of 1000 gaps 312 /
// 318, 30,000 252 / 256, 12,000 ragged ones of 700 on average 369 / 373; 64 of 1500 gaps 73 / 73; 6000 ragged ones of 1400 on
// average 390 / 356 (if they repeat) and 377 / 380 (if not), 12,000 of 2100 563 / 449 and 559 / 563.
constexpr uint64_t GF_REPEAT_LAUNCHES = REPEAT_GAPS / 2;

}  // extern "C"

namespace {

constexpr uint64_t ws_align(uint64_t v) { return (v + 255) / 256 * 256; }

// Workspace of the gap fill: control block, task roles, queue totals, three per-launch arrays.
constexpr uint64_t gapfill_ws_bytes(uint64_t n_ids, uint64_t n_tasks) {
  return 256 + ws_align(n_tasks * 4) + ws_align(n_tasks * 8) + 2 * ws_align(n_ids * 8 + GF_PAD) + ws_align(n_ids * 8);
}

struct GapfillBuffers {
  uint64_t n_ids;
  Ctrl* ctrl;
  uint32_t* role;
  uint64_t* lp_total;
  int64_t *pe, *pg, *open;   // 64-bit predictions (k_gf_predict)
  uint32_t* lp_e;            // 32-bit predictions (k_gf_predict32): they share the space of pe and pg
  uint2* hp_eg;
  GapfillBuffers(unsigned char* ws, uint64_t n_launches, uint32_t n_tasks) : n_ids(n_launches) {
    Carver c;
    ctrl = reinterpret_cast<Ctrl*>(ws + c.take(256));
    role = reinterpret_cast<uint32_t*>(ws + c.take(static_cast<uint64_t>(n_tasks) * 4));
    lp_total = reinterpret_cast<uint64_t*>(ws + c.take(static_cast<uint64_t>(n_tasks) * 8));
    pe = reinterpret_cast<int64_t*>(ws + c.take(n_ids * 8 + GF_PAD));
    pg = reinterpret_cast<int64_t*>(ws + c.take(n_ids * 8 + GF_PAD));
    open = reinterpret_cast<int64_t*>(ws + c.take(n_ids * 8));
    lp_e = reinterpret_cast<uint32_t*>(pe);
    hp_eg = reinterpret_cast<uint2*>(pg);
  }
};

bool gapfill_params_ok(const fikit_gapfill_params* p) {
  return p && p->margin_ns >= 0 && p->min_gap_ns >= 0 && p->reserved == 0 && p->predictor >= FIKIT_PREDICT_P50 &&
         p->predictor <= FIKIT_PREDICT_MEAN;
}

// Workgroups per task of k_gf_predict32: about PRED_PART launches each, and with few tasks as many as give the chip a few
// workgroups per compute unit (a workgroup whose part is empty leaves at once).  Every workgroup builds its task's table, so
// tasks that fill the chip many times over by themselves are not divided: 32,768 tasks of 4096 and 16,384 launches in turn
// 1030 us with two workgroups each, 890 us with one.
uint32_t predict_parts(uint64_t n_ids, uint32_t n_tasks) {
  constexpr uint64_t PRED_PART = 8192, PRED_WORKGROUPS = 2048, PRED_ENOUGH = 8 * PRED_WORKGROUPS;
  const uint64_t tasks = n_tasks ? n_tasks : 1;
  uint64_t parts = tasks < PRED_ENOUGH ? n_ids / tasks / PRED_PART + 1 : 1;
  if (parts * tasks < PRED_WORKGROUPS) parts = PRED_WORKGROUPS / tasks;
  const uint64_t most = n_ids / (2 * PRED_THREADS) + 1;
  if (parts > most) parts = most;
  return static_cast<uint32_t>(parts > 64 ? 64 : parts);
}

// The waves' order of the scenarios is made if there are more than two for each of the chip's SIMDs (up to there the longest trace
// alone decides, wherever it runs: 1500 even scenarios 82 us without the lists, 84 us with them) and the lists fit `bytes` at `at`
// (64 per scenario).
constexpr uint64_t GF_ORDER_MIN_SCENARIOS = 2048 + 1;
static_assert(GF_ORDER_MIN_SCENARIOS > GF_BEGIN_ITEMS, "k_gf_begin makes no lists");
GfOrder scenario_order(Ctrl* ctrl, void* at, uint64_t bytes, uint64_t n_scenarios) {
  static_assert(GF_LANES_MIN_SCENARIOS <= 1u << 16, "scenarios are listed by 16-bit numbers");
  if (n_scenarios < GF_ORDER_MIN_SCENARIOS || n_scenarios >= GF_LANES_MIN_SCENARIOS || n_scenarios * GF_BUCKETS * 2 > bytes)
    return GfOrder{nullptr, nullptr};
  return GfOrder{reinterpret_cast<uint32_t*>(ctrl + 1), static_cast<uint16_t*>(at)};
}
// (in the space of the 64-bit opening times, which the 32-bit kernels leave unused)
GfOrder gapfill_order(const GapfillBuffers& b, uint64_t n_scenarios) { return scenario_order(b.ctrl, b.open, b.n_ids * 8, n_scenarios); }

bool gapfill_checks_are_few(uint32_t n_tasks, uint64_t n_scenarios) { return n_tasks <= GF_BEGIN_ITEMS && n_scenarios <= GF_BEGIN_ITEMS; }
GfBegin gapfill_begin(const GapfillBuffers& b, const uint32_t* d_hp_task, const uint32_t* d_lp_task, uint64_t n_scenarios,
                      const uint64_t* d_gap_offsets, uint64_t n_gaps, uint32_t* done) {
  return GfBegin{d_hp_task, d_lp_task, static_cast<uint32_t>(n_scenarios), d_gap_offsets, n_gaps, b.role, b.lp_total, done, b.ctrl};
}

// What every gap fill starts with: a cleared control block, checked arguments, task roles.
void gapfill_check_enqueue(hipStream_t st, const GapfillBuffers& b, const uint64_t* d_task_offsets, uint64_t n_ids, uint32_t n_tasks,
                           const uint32_t* d_hp_task, const uint32_t* d_lp_task, uint64_t n_scenarios, const uint64_t* d_gap_offsets,
                           uint64_t n_gaps, uint32_t* done) {
  if (gapfill_checks_are_few(n_tasks, n_scenarios)) {
    FIKIT_COUNT_LAUNCH(k_gf_begin, dim3(1), dim3(GF_BEGIN_THREADS), 0, st, d_task_offsets, n_tasks, n_ids,
                       gapfill_begin(b, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, n_gaps, done));
    return;
  }
  FIKIT_COUNT_LAUNCH(k_gf_clear, dim3(blocks_for(n_tasks, 256)), dim3(256), 0, st, b.ctrl, b.role, b.lp_total, done, n_tasks);
  FIKIT_COUNT_LAUNCH(k_gf_check, dim3(blocks_for(n_scenarios > n_tasks ? n_scenarios : n_tasks, 256)), dim3(256), 0, st, d_task_offsets,
                     n_tasks, n_ids, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, n_gaps, b.role, gapfill_order(b, n_scenarios), b.ctrl);
}

// The walk on 32-bit predictions in one of its modes; `result`: completion times, or delays in the replay modes.  prof (may be
// null): the profile that it follows in the same call.
template <int MODE>
int walk_enqueue(hipStream_t st, Tracer& tr, const GapfillBuffers& b, const uint64_t* d_task_offsets, uint32_t n_tasks,
                 const uint32_t* d_hp_task, const uint32_t* d_lp_task, uint64_t n_scenarios, const uint64_t* d_gap_offsets,
                 uint64_t n_gaps, int64_t margin, int64_t min_gap, uint32_t* d_fill_count, int64_t* d_filled_ns, int64_t* result, uint64_t* d_lp_placed,
                 bool set_attributes, const Ctrl* prof, uint64_t row_capacity) {
  if (n_scenarios >= GF_LANES_MIN_SCENARIOS && n_gaps < MAX_ELEMS) {
    tr.mark(MODE == LW_PLAN ? "k_gf_walk_lanes" : MODE == LW_REPLAY ? "k_gf_replay_lanes" : "k_gf_replay_feedback_lanes");
    if (set_attributes)
      FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_gf_walk_lanes<MODE>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    static_cast<int>(sizeof(LaneWalkSmem))));
    const uint32_t vec_ok = (aligned(d_fill_count, 16) && aligned(d_filled_ns, 16)) ? 1u : 0u;
    FIKIT_COUNT_LAUNCH(k_gf_walk_lanes<MODE>, dim3(blocks_for(n_scenarios, LW_THREADS)), dim3(LW_THREADS), sizeof(LaneWalkSmem), st,
                       d_task_offsets, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, b.lp_e, b.hp_eg, b.lp_total, margin, min_gap,
                       d_fill_count, d_filled_ns, result, d_lp_placed, vec_ok, prof, row_capacity, b.ctrl);
  } else {
    // launches of a trace on average; in a step, where the host does not read the number of gaps, of a task
    const uint64_t launches = n_gaps != ANY_GAPS ? n_gaps / n_scenarios + 1 : b.n_ids / n_tasks;
    const bool teams = MODE != LW_REPLAY_FEEDBACK && n_scenarios <= GF_TEAM_SCENARIOS && launches >= GF_TEAM_LAUNCHES;
    tr.mark(MODE == LW_PLAN ? (teams ? "k_gf_walk_team" : "k_gf_walk_wave")
                            : MODE == LW_REPLAY ? (teams ? "k_gf_replay_team" : "k_gf_replay_wave") : "k_gf_replay_feedback_wave");
    auto kernel = &k_gf_walk_wave<MODE, 0>;
    if constexpr (MODE != LW_REPLAY_FEEDBACK)
      kernel = teams ? &k_gf_walk_wave<MODE, GF_TEAM_WAVES> : launches >= GF_REPEAT_LAUNCHES ? &k_gf_walk_wave<MODE, 1> : kernel;
    FIKIT_COUNT_LAUNCH(kernel, dim3(teams ? static_cast<uint32_t>(n_scenarios) : blocks_for(n_scenarios, WW_THREADS / WAVE)),
                       dim3(teams ? GF_TEAM_WAVES * WAVE : WW_THREADS), 0, st, d_task_offsets, d_hp_task, d_lp_task,
                       static_cast<uint32_t>(n_scenarios), d_gap_offsets, b.lp_e, b.hp_eg, b.lp_total, margin, min_gap, d_fill_count,
                       d_filled_ns, result, d_lp_placed, prof, row_capacity, gapfill_order(b, n_scenarios), b.ctrl);
  }
  FIKIT_HIP(hipGetLastError());
  return FIKIT_OK;
}

// Enqueues the predictions and the fill on `st` (gapfill_check_enqueue has been).  done (may be null): tasks whose predictions
// exist already; all_done: those of all tasks do (a launch that would find nothing to do costs 5 us of a call of 74, and 20 us
// with 32,768 tasks).  Nothing is read back and nothing is allocated here.
int gapfill_enqueue(hipStream_t st, Tracer& tr, const GapfillBuffers& b, const uint64_t* d_ids, uint64_t n_ids,
                    const uint64_t* d_task_offsets, uint32_t n_tasks, const fikit_row* d_rows, const uint64_t* d_task_row_offsets,
                    const uint32_t* d_hp_task, const uint32_t* d_lp_task, uint64_t n_scenarios, const fikit_gapfill_params* h_params,
                    const uint64_t* d_gap_offsets, uint64_t n_gaps, uint32_t* d_fill_count, int64_t* d_filled_ns,
                    int64_t* d_lp_completion_ns, uint64_t* d_lp_placed, bool set_attributes, const uint32_t* done, bool all_done, const Ctrl* prof = nullptr,
                    uint64_t row_capacity = 0) {
  if (!all_done) {
    tr.mark("k_gf_predict32");
    FIKIT_COUNT_LAUNCH(k_gf_predict32, dim3(n_tasks, predict_parts(n_ids, n_tasks)), dim3(PRED_THREADS), 0, st, d_ids, d_task_offsets,
                       n_tasks, d_rows, d_task_row_offsets, b.role, static_cast<const int64_t*>(nullptr), b.lp_e, b.hp_eg, b.lp_total,
                       static_cast<uint32_t>(h_params->predictor), done, prof, row_capacity, b.ctrl);
  }
  return walk_enqueue<LW_PLAN>(st, tr, b, d_task_offsets, n_tasks, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, n_gaps,
                               h_params->margin_ns, h_params->min_gap_ns, d_fill_count, d_filled_ns, d_lp_completion_ns, d_lp_placed,
                               set_attributes, prof, row_capacity);
}

// The 64-bit kernels, which do the call if a prediction did not fit 32 bits (they check Ctrl::wide).
int gapfill_wide_enqueue(hipStream_t st, const GapfillBuffers& b, const uint64_t* d_ids, const uint64_t* d_task_offsets, uint32_t n_tasks,
                         const fikit_row* d_rows, const uint64_t* d_task_row_offsets, const uint32_t* d_hp_task,
                         const uint32_t* d_lp_task, uint64_t n_scenarios, const fikit_gapfill_params* h_params,
                         const uint64_t* d_gap_offsets, uint32_t* d_fill_count, int64_t* d_filled_ns, int64_t* d_lp_completion_ns,
                         uint64_t* d_lp_placed, int32_t* d_status = nullptr) {
  FIKIT_COUNT_LAUNCH(k_gf_predict, dim3(n_tasks), dim3(PRED_THREADS), 0, st, d_ids, d_task_offsets, n_tasks, d_rows,
                     d_task_row_offsets, b.role, b.pe, b.pg, b.open, static_cast<uint32_t>(h_params->predictor), b.ctrl);
  FIKIT_COUNT_LAUNCH(k_gf_walk, dim3(blocks_for(n_scenarios, 256 / WAVE)), dim3(256), 0, st, d_task_offsets, d_hp_task, d_lp_task,
                     n_scenarios, d_gap_offsets, b.pe, b.pg, b.open, h_params->margin_ns, h_params->min_gap_ns, d_fill_count, d_filled_ns,
                     d_lp_completion_ns, d_lp_placed, d_status, b.ctrl);
  FIKIT_HIP(hipGetLastError());
  return FIKIT_OK;
}

// Ends a gap fill whose control block has been read: its status, and the 64-bit kernels first if they are needed.
template <typename Wide>
int finish_gapfill(hipStream_t st, Tracer& tr, const Ctrl* ctrl, Ctrl h, Wide enqueue_wide) {
  if (int rc = status_from_bits(h.status)) return rc;
  if (!h.wide) return FIKIT_OK;
  tr.mark("gf_wide");
  if (int rc = enqueue_wide()) return rc;
  tr.mark("host_sync");
  if (int rc = read_ctrl(ctrl, &h, st)) return rc;
  return status_from_bits(h.status);
}
template <typename Wide>
int finish_gapfill(hipStream_t st, Tracer& tr, const Ctrl* ctrl, Wide enqueue_wide) {
  tr.mark("host_sync");
  Ctrl h{};
  if (int rc = read_ctrl(ctrl, &h, st)) return rc;
  return finish_gapfill(st, tr, ctrl, h, enqueue_wide);
}

}  // namespace

extern "C" {

size_t fikit_gapfill_workspace_bytes(uint64_t n_ids, uint32_t n_tasks, uint64_t n_scenarios) {
  (void)n_scenarios;
  if (n_ids >= MAX_ELEMS) return 0;
  return static_cast<size_t>(gapfill_ws_bytes(n_ids, n_tasks));
}

int fikit_gapfill(const uint64_t* d_ids, const uint64_t* d_task_offsets, uint32_t n_tasks, const fikit_row* d_rows,
                  const uint64_t* d_task_row_offsets, const uint32_t* d_hp_task, const uint32_t* d_lp_task,
                  uint64_t n_scenarios, const fikit_gapfill_params* h_params, const uint64_t* d_gap_offsets,
                  uint32_t* d_fill_count, int64_t* d_filled_ns, int64_t* d_lp_completion_ns, uint64_t* d_lp_placed,
                  void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (!gapfill_params_ok(h_params)) return FIKIT_INVALID_ARG;
  if (!d_task_offsets || !d_task_row_offsets || !d_workspace) return FIKIT_INVALID_ARG;
  if (n_scenarios >= MAX_ELEMS) return FIKIT_INVALID_ARG;
  if (n_scenarios > 0 && (!d_hp_task || !d_lp_task || !d_gap_offsets || !d_lp_completion_ns || !d_lp_placed || n_tasks == 0))
    return FIKIT_INVALID_ARG;
  if (!aligned(d_ids, 8) || !aligned(d_task_offsets, 8) || !aligned(d_rows, 16) || !aligned(d_task_row_offsets, 8) ||
      !aligned(d_hp_task, 4) || !aligned(d_lp_task, 4) || !aligned(d_gap_offsets, 8) || !aligned(d_fill_count, 4) ||
      !aligned(d_filled_ns, 8) || !aligned(d_lp_completion_ns, 8) || !aligned(d_lp_placed, 8) || !aligned(d_workspace, 256))
    return FIKIT_INVALID_ARG;
  if (n_scenarios == 0) return FIKIT_OK;

  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  // The element counts live on the device: total launches and total gaps.
  uint64_t n_ids = 0, n_gaps = 0;
  Reads counts(st);
  if (int rc = counts.add(&n_ids, d_task_offsets + n_tasks, 8)) return rc;
  if (int rc = counts.add(&n_gaps, d_gap_offsets + n_scenarios, 8)) return rc;
  if (int rc = counts.wait(false)) return rc;
  if (n_ids >= MAX_ELEMS) return FIKIT_INVALID_ARG;
  if (n_ids > 0 && (!d_ids || !d_rows)) return FIKIT_INVALID_ARG;
  if (n_gaps > 0 && (!d_fill_count || !d_filled_ns)) return FIKIT_INVALID_ARG;
  if (workspace_bytes < fikit_gapfill_workspace_bytes(n_ids, n_tasks, n_scenarios)) return FIKIT_WORKSPACE_TOO_SMALL;

  const GapfillBuffers b(static_cast<unsigned char*>(d_workspace), n_ids, n_tasks);
  Tracer tr(st);
  tr.mark("gf_setup");
  gapfill_check_enqueue(st, b, d_task_offsets, n_ids, n_tasks, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, n_gaps, nullptr);
  if (int rc = gapfill_enqueue(st, tr, b, d_ids, n_ids, d_task_offsets, n_tasks, d_rows, d_task_row_offsets, d_hp_task, d_lp_task,
                               n_scenarios, h_params, d_gap_offsets, n_gaps, d_fill_count, d_filled_ns, d_lp_completion_ns,
                               d_lp_placed, true, nullptr, false))
    return rc;
  return finish_gapfill(st, tr, b.ctrl, [&] {
    return gapfill_wide_enqueue(st, b, d_ids, d_task_offsets, n_tasks, d_rows, d_task_row_offsets, d_hp_task, d_lp_task, n_scenarios,
                                h_params, d_gap_offsets, d_fill_count, d_filled_ns, d_lp_completion_ns, d_lp_placed);
  });
}

size_t fikit_profile_gapfill_workspace_bytes(uint64_t n_records, uint32_t n_tasks, uint64_t n_scenarios) {
  const size_t a = fikit_profile_workspace_bytes(n_records, n_tasks), b = fikit_gapfill_workspace_bytes(n_records, n_tasks, n_scenarios);
  if (a == 0 || b == 0) return 0;
  return static_cast<size_t>(ws_align(a) + ws_align(b) + ws_align(static_cast<uint64_t>(n_tasks) * 4));
}

int fikit_profile_gapfill(const fikit_launch* d_records, uint64_t n_records, const uint64_t* d_task_offsets, uint32_t n_tasks,
                          uint64_t* d_ids_out, fikit_row* d_rows_out, uint64_t row_capacity, uint64_t* d_task_row_offsets,
                          uint64_t* h_n_rows, const uint32_t* d_hp_task, const uint32_t* d_lp_task, uint64_t n_scenarios,
                          const fikit_gapfill_params* h_params, const uint64_t* d_gap_offsets, uint32_t* d_fill_count,
                          int64_t* d_filled_ns, int64_t* d_lp_completion_ns, uint64_t* d_lp_placed, void* d_workspace,
                          size_t workspace_bytes, void* hip_stream) {
  if (!h_n_rows) return FIKIT_INVALID_ARG;
  *h_n_rows = 0;
  if (!gapfill_params_ok(h_params)) return FIKIT_INVALID_ARG;
  if (!d_ids_out || !d_workspace || !d_task_offsets || n_records >= MAX_ELEMS || n_scenarios >= MAX_ELEMS) return FIKIT_INVALID_ARG;
  if (n_scenarios > 0 && (!d_hp_task || !d_lp_task || !d_gap_offsets || !d_lp_completion_ns || !d_lp_placed || n_tasks == 0))
    return FIKIT_INVALID_ARG;
  if (!aligned(d_hp_task, 4) || !aligned(d_lp_task, 4) || !aligned(d_gap_offsets, 8) || !aligned(d_fill_count, 4) ||
      !aligned(d_filled_ns, 8) || !aligned(d_lp_completion_ns, 8) || !aligned(d_lp_placed, 8) || !aligned(d_workspace, 256))
    return FIKIT_INVALID_ARG;
  const size_t need = fikit_profile_gapfill_workspace_bytes(n_records, n_tasks, n_scenarios);
  if (need == 0) return FIKIT_INVALID_ARG;
  if (workspace_bytes < need) return FIKIT_WORKSPACE_TOO_SMALL;
  unsigned char* ws = static_cast<unsigned char*>(d_workspace);
  const uint64_t prof_bytes = ws_align(fikit_profile_workspace_bytes(n_records, n_tasks));
  const uint64_t gf_bytes = ws_align(fikit_gapfill_workspace_bytes(n_records, n_tasks, n_scenarios));
  unsigned char* gf_ws = ws + prof_bytes;
  uint32_t* done = reinterpret_cast<uint32_t*>(gf_ws + gf_bytes);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (n_scenarios == 0)
    return fikit_profile(d_records, n_records, d_task_offsets, n_tasks, d_ids_out, d_rows_out, row_capacity, d_task_row_offsets,
                         h_n_rows, ws, prof_bytes, hip_stream);

  uint64_t n_gaps = ANY_GAPS;   // (the number matters only where a buffer is missing, or for the lane walk)
  if (!d_fill_count || !d_filled_ns || n_scenarios >= GF_LANES_MIN_SCENARIOS) {
    Reads r(st);
    if (int rc = r.add(&n_gaps, d_gap_offsets + n_scenarios, 8)) return rc;
    if (int rc = r.wait(false)) return rc;
    if (n_gaps > 0 && (!d_fill_count || !d_filled_ns)) return FIKIT_INVALID_ARG;
  }

  // 1. the gap fill's checks and task roles; 2. the profile, whose one-workgroup kernels also write the predictions
  // of the tasks that the scenarios use; 3. the predictions of the remaining tasks, and the fill.
  const GapfillBuffers b(gf_ws, n_records, n_tasks);
  PredEmit emit{};
  emit.role = b.role; emit.lp_e = b.lp_e; emit.hp_eg = b.hp_eg; emit.lp_total = b.lp_total; emit.done = done;
  emit.predictor = static_cast<uint32_t>(h_params->predictor);
  const bool few = n_tasks <= BEGIN_TASKS && gapfill_checks_are_few(n_tasks, n_scenarios) && n_records > 0;
  const GfBegin begin = gapfill_begin(b, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, n_gaps, done);
  if (!few) {
    Tracer tr(st);
    tr.mark("gf_setup");
    gapfill_check_enqueue(st, b, d_task_offsets, n_records, n_tasks, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, n_gaps, done);
    FIKIT_HIP(hipGetLastError());
  }
  auto fill = [&](Tracer& tr, bool all_done, const Ctrl* prof) {
    return gapfill_enqueue(st, tr, b, d_ids_out, n_records, d_task_offsets, n_tasks, d_rows_out, d_task_row_offsets, d_hp_task,
                           d_lp_task, n_scenarios, h_params, d_gap_offsets, n_gaps, d_fill_count, d_filled_ns, d_lp_completion_ns,
                           d_lp_placed, true, done, all_done, prof, row_capacity);
  };
  // The fill is enqueued behind the rows and the host waits once (one pair of 1000 launches: 69 us with
  // two waits and the small kernels apart, 57 us).  Where no
  // task is long, either all have their predictions from the profile's kernels, or some are left to the general path and the
  // fill leaves at once: it is enqueued again then.
  Ctrl h{};
  bool was_ahead = false;
  if (int rc = profile_run(d_records, n_records, d_task_offsets, n_tasks, d_ids_out, d_rows_out, row_capacity, d_task_row_offsets,
                           h_n_rows, ws, prof_bytes, hip_stream, &emit, few ? &begin : nullptr,
                           [&](Tracer& tr, Reads& reads, const Ctrl* prof, bool any_long) {
                             if (int rc = fill(tr, !any_long, prof)) return rc;
                             return reads.add(&h, b.ctrl, sizeof(Ctrl));
                           },
                           &was_ahead))
    return rc;
  Tracer tr(st);
  if (!was_ahead) {
    if (int rc = fill(tr, false, nullptr)) return rc;
    tr.mark("host_sync");
    if (int rc = read_ctrl(b.ctrl, &h, st)) return rc;
  }
  return finish_gapfill(st, tr, b.ctrl, h, [&] {
    return gapfill_wide_enqueue(st, b, d_ids_out, d_task_offsets, n_tasks, d_rows_out, d_task_row_offsets, d_hp_task, d_lp_task,
                                n_scenarios, h_params, d_gap_offsets, d_fill_count, d_filled_ns, d_lp_completion_ns, d_lp_placed);
  });
}

}  // extern "C"

namespace {

// ---- fikit_gapfill_static: the gap fill for callers that cannot allocate --------------------------------------
// Its workspace is a device array that is part of the library's code object.  Every GPU the library runs on holds
// its own copy at its own address; that address is looked up once per device, with the device current.
constexpr uint64_t STATIC_SCRATCH_BYTES = gapfill_ws_bytes(FIKIT_STATIC_MAX_IDS, FIKIT_STATIC_MAX_TASKS);
static_assert(STATIC_SCRATCH_BYTES <= (32ull << 20), "the built-in scratch buffer is meant to stay modest");
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int STATIC_MAX_DEVICES = 64;
std::mutex g_static_mutex;
unsigned char* g_static_scratch[STATIC_MAX_DEVICES] = {};

// Address of the current device's scratch array (set-up on the first call on that device).
int static_scratch_of_current_device(unsigned char** out) {
  int dev = -1;
  FIKIT_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= STATIC_MAX_DEVICES) return FIKIT_HIP_ERROR;
  std::lock_guard<std::mutex> lock(g_static_mutex);
  if (!g_static_scratch[dev]) {
    unsigned char* ptr = nullptr;
    FIKIT_HIP(hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch)));
    if (!ptr) return FIKIT_HIP_ERROR;
    FIKIT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_gf_walk_lanes<LW_PLAN>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(sizeof(LaneWalkSmem))));
    g_static_scratch[dev] = ptr;
  }
  *out = g_static_scratch[dev];
  return FIKIT_OK;
}

// The status of a call without scenarios.
__global__ void k_publish_ok(int32_t* status_out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *status_out = FIKIT_OK;
}

}  // namespace

extern "C" {

int fikit_gapfill_static(const uint64_t* d_ids, uint64_t n_ids, const uint64_t* d_task_offsets, uint32_t n_tasks,
                         const fikit_row* d_rows, const uint64_t* d_task_row_offsets, const uint32_t* d_hp_task,
                         const uint32_t* d_lp_task, uint64_t n_scenarios, const fikit_gapfill_params* h_params,
                         const uint64_t* d_gap_offsets, uint64_t n_gaps, uint32_t* d_fill_count, int64_t* d_filled_ns,
                         int64_t* d_lp_completion_ns, uint64_t* d_lp_placed, int32_t* d_status, void* hip_stream) {
  if (!gapfill_params_ok(h_params)) return FIKIT_INVALID_ARG;
  if (!d_task_offsets || !d_task_row_offsets || !d_status || !aligned(d_status, 4)) return FIKIT_INVALID_ARG;
  if (n_scenarios >= MAX_ELEMS || n_gaps >= MAX_ELEMS) return FIKIT_INVALID_ARG;
  if (n_ids > FIKIT_STATIC_MAX_IDS || n_tasks > FIKIT_STATIC_MAX_TASKS) return FIKIT_TOO_LARGE;
  if (n_tasks == 0) return FIKIT_INVALID_ARG;
  if (n_scenarios > 0 && (!d_hp_task || !d_lp_task || !d_gap_offsets || !d_lp_completion_ns || !d_lp_placed))
    return FIKIT_INVALID_ARG;
  if (n_ids > 0 && (!d_ids || !d_rows)) return FIKIT_INVALID_ARG;
  if (n_gaps > 0 && (!d_fill_count || !d_filled_ns)) return FIKIT_INVALID_ARG;
  if (!aligned(d_ids, 8) || !aligned(d_task_offsets, 8) || !aligned(d_rows, 16) || !aligned(d_task_row_offsets, 8) ||
      !aligned(d_hp_task, 4) || !aligned(d_lp_task, 4) || !aligned(d_gap_offsets, 8) || !aligned(d_fill_count, 4) ||
      !aligned(d_filled_ns, 8) || !aligned(d_lp_completion_ns, 8) || !aligned(d_lp_placed, 8))
    return FIKIT_INVALID_ARG;
  unsigned char* ws = nullptr;
  if (int rc = static_scratch_of_current_device(&ws)) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  Tracer tr(st, false);   // (recording events would allocate)
  const GapfillBuffers b(ws, n_ids, n_tasks);
  if (n_scenarios == 0) {
    FIKIT_COUNT_LAUNCH(k_publish_ok, dim3(1), dim3(64), 0, st, d_status);
  } else {
    gapfill_check_enqueue(st, b, d_task_offsets, n_ids, n_tasks, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, n_gaps, nullptr);
    if (int rc = gapfill_enqueue(st, tr, b, d_ids, n_ids, d_task_offsets, n_tasks, d_rows, d_task_row_offsets, d_hp_task, d_lp_task,
                                 n_scenarios, h_params, d_gap_offsets, n_gaps, d_fill_count, d_filled_ns, d_lp_completion_ns,
                                 d_lp_placed, false, nullptr, false))
      return rc;
    // (whether a prediction needs 64 bits is only known on the device, and nothing is waited for here)
    if (n_scenarios <= GF_WIDE_SCENARIOS) {
      FIKIT_COUNT_LAUNCH(k_gf_wide, dim3(static_cast<uint32_t>(n_scenarios)), dim3(PRED_THREADS), 0, st, d_ids, d_task_offsets, d_rows,
                         d_task_row_offsets, b.role, d_hp_task, d_lp_task, d_gap_offsets, b.pe, b.pg, b.open,
                         static_cast<uint32_t>(h_params->predictor), h_params->margin_ns, h_params->min_gap_ns, d_fill_count, d_filled_ns,
                         d_lp_completion_ns, d_lp_placed, d_status, b.ctrl);
    } else if (int rc = gapfill_wide_enqueue(st, b, d_ids, d_task_offsets, n_tasks, d_rows, d_task_row_offsets, d_hp_task, d_lp_task,
                                             n_scenarios, h_params, d_gap_offsets, d_fill_count, d_filled_ns, d_lp_completion_ns, d_lp_placed,
                                             d_status)) {
      return rc;
    }
  }
  FIKIT_HIP(hipGetLastError());
  return FIKIT_OK;
}

size_t fikit_measure_workspace_bytes(void) { return 256; }

int fikit_measure(const fikit_launch* d_records, uint64_t n_records, const uint64_t* d_task_offsets, uint32_t n_tasks,
                  int64_t* d_exec_ns, int64_t* d_gap_ns, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (!d_task_offsets || !d_workspace) return FIKIT_INVALID_ARG;
  if (n_records >= MAX_ELEMS) return FIKIT_INVALID_ARG;
  if (n_records > 0 && (!d_records || !d_exec_ns || !d_gap_ns || n_tasks == 0)) return FIKIT_INVALID_ARG;
  if (!aligned(d_records, 8) || !aligned(d_task_offsets, 8) || !aligned(d_exec_ns, 8) || !aligned(d_gap_ns, 8) ||
      !aligned(d_workspace, 256))
    return FIKIT_INVALID_ARG;
  if (workspace_bytes < fikit_measure_workspace_bytes()) return FIKIT_WORKSPACE_TOO_SMALL;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  Ctrl* ctrl = static_cast<Ctrl*>(d_workspace);
  Tracer tr(st);
  tr.mark("k_measure");
  FIKIT_COUNT_LAUNCH(k_clear_ctrl, dim3(1), dim3(64), 0, st, ctrl);
  FIKIT_COUNT_LAUNCH(k_validate_offsets, dim3(blocks_for(n_tasks, 256)), dim3(256), 0, st, d_task_offsets, n_tasks, n_records,
                     ctrl);
  if (n_records > 0) {
    FIKIT_COUNT_LAUNCH(k_measure, dim3(blocks_for(n_records, 256)), dim3(256), 0, st, d_records, n_records, d_exec_ns, d_gap_ns,
                       ctrl);
    FIKIT_COUNT_LAUNCH(k_measure_task_ends, dim3(blocks_for(n_tasks, 256)), dim3(256), 0, st, d_task_offsets, n_tasks, d_gap_ns,
                       ctrl);
  }
  FIKIT_HIP(hipGetLastError());
  tr.mark("host_sync");
  Ctrl h{};
  if (int rc = read_ctrl(ctrl, &h, st)) return rc;
  return status_from_bits(h.status);
}

size_t fikit_replay_workspace_bytes(uint64_t n_ids, uint32_t n_tasks, uint64_t n_scenarios) {
  return fikit_gapfill_workspace_bytes(n_ids, n_tasks, n_scenarios);
}

int fikit_gapfill_replay(const uint64_t* d_ids, const uint64_t* d_task_offsets, uint32_t n_tasks, const fikit_row* d_rows,
                         const uint64_t* d_task_row_offsets, const int64_t* d_actual_gap_ns, const uint32_t* d_hp_task,
                         const uint32_t* d_lp_task, uint64_t n_scenarios, const fikit_replay_params* h_params,
                         const uint64_t* d_gap_offsets, uint32_t* d_fill_count, int64_t* d_filled_ns, int64_t* d_hp_delay_ns,
                         uint64_t* d_lp_placed, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (!h_params || h_params->margin_ns < 0 || h_params->min_gap_ns < 0 || h_params->predictor < FIKIT_PREDICT_P50 ||
      h_params->predictor > FIKIT_PREDICT_MEAN)
    return FIKIT_INVALID_ARG;
  if (!d_task_offsets || !d_task_row_offsets || !d_workspace) return FIKIT_INVALID_ARG;
  if (n_scenarios >= MAX_ELEMS) return FIKIT_INVALID_ARG;
  if (n_scenarios > 0 && (!d_hp_task || !d_lp_task || !d_gap_offsets || !d_hp_delay_ns || !d_lp_placed || n_tasks == 0))
    return FIKIT_INVALID_ARG;
  if (!aligned(d_ids, 8) || !aligned(d_task_offsets, 8) || !aligned(d_rows, 16) || !aligned(d_task_row_offsets, 8) ||
      !aligned(d_actual_gap_ns, 8) || !aligned(d_hp_task, 4) || !aligned(d_lp_task, 4) || !aligned(d_gap_offsets, 8) ||
      !aligned(d_fill_count, 4) || !aligned(d_filled_ns, 8) || !aligned(d_hp_delay_ns, 8) || !aligned(d_lp_placed, 8) ||
      !aligned(d_workspace, 256))
    return FIKIT_INVALID_ARG;
  if (n_scenarios == 0) return FIKIT_OK;

  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint64_t n_ids = 0, n_gaps = 0;
  Reads counts(st);
  if (int rc = counts.add(&n_ids, d_task_offsets + n_tasks, 8)) return rc;
  if (int rc = counts.add(&n_gaps, d_gap_offsets + n_scenarios, 8)) return rc;
  if (int rc = counts.wait(false)) return rc;
  if (n_ids >= MAX_ELEMS || n_gaps >= MAX_ELEMS) return FIKIT_INVALID_ARG;
  if (n_ids > 0 && (!d_ids || !d_rows || !d_actual_gap_ns)) return FIKIT_INVALID_ARG;
  if (n_gaps > 0 && (!d_fill_count || !d_filled_ns)) return FIKIT_INVALID_ARG;
  if (workspace_bytes < fikit_replay_workspace_bytes(n_ids, n_tasks, n_scenarios)) return FIKIT_WORKSPACE_TOO_SMALL;

  const GapfillBuffers b(static_cast<unsigned char*>(d_workspace), n_ids, n_tasks);
  Tracer tr(st);
  tr.mark("gf_setup");
  gapfill_check_enqueue(st, b, d_task_offsets, n_ids, n_tasks, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, n_gaps, nullptr);
  tr.mark("k_gf_predict32");
  FIKIT_COUNT_LAUNCH(k_gf_predict32, dim3(n_tasks, predict_parts(n_ids, n_tasks)), dim3(PRED_THREADS), 0, st, d_ids, d_task_offsets,
                     n_tasks, d_rows, d_task_row_offsets, b.role, d_actual_gap_ns, b.lp_e, b.hp_eg, b.lp_total,
                     static_cast<uint32_t>(h_params->predictor), static_cast<const uint32_t*>(nullptr),
                     static_cast<const Ctrl*>(nullptr), static_cast<uint64_t>(0), b.ctrl);
  auto walk = h_params->feedback ? walk_enqueue<LW_REPLAY_FEEDBACK> : walk_enqueue<LW_REPLAY>;
  if (int rc = walk(st, tr, b, d_task_offsets, n_tasks, d_hp_task, d_lp_task, n_scenarios, d_gap_offsets, n_gaps, h_params->margin_ns,
                    h_params->min_gap_ns, d_fill_count, d_filled_ns, d_hp_delay_ns, d_lp_placed, true, nullptr, 0))
    return rc;
  return finish_gapfill(st, tr, b.ctrl, [&]() -> int {
    FIKIT_COUNT_LAUNCH(k_gf_predict, dim3(n_tasks), dim3(PRED_THREADS), 0, st, d_ids, d_task_offsets, n_tasks, d_rows,
                       d_task_row_offsets, b.role, b.pe, b.pg, static_cast<int64_t*>(nullptr),
                       static_cast<uint32_t>(h_params->predictor), b.ctrl);
    FIKIT_COUNT_LAUNCH(k_gf_replay_wide, dim3(blocks_for(n_scenarios, 256)), dim3(256), 0, st, d_task_offsets, d_hp_task, d_lp_task,
                       n_scenarios, d_gap_offsets, b.pe, b.pg, d_actual_gap_ns, h_params->margin_ns, h_params->min_gap_ns,
                       h_params->feedback ? 1u : 0u, d_fill_count, d_filled_ns, d_hp_delay_ns, d_lp_placed, b.ctrl);
    FIKIT_HIP(hipGetLastError());
    return FIKIT_OK;
  });
}

}  // extern "C"

namespace {

// One wave per scenario up to this many scenarios, beyond it a group of lanes per scenario.  The waves' time grows with
// the scenarios, the groups' hardly does; traces of 1024 launches, queues of 2048, waves / groups in ms for the call:
//   1 task   4096: 0.35 / 1.22   16,384: 0.94 / 1.42   24,576: 1.34 / 1.54
//   2 tasks  4096: 0.87 / 1.81   8192: 1.41 / 1.87   12,288: 1.93 / 1.96
//   3 tasks  64: 0.80 / 2.2   4096: 1.07 / 2.34   8192: 1.74 / 2.39   12,288: 2.41 / 2.76
//   4 tasks  4096: 1.42 / 2.64   12,288: 2.88 / 3.11   6 tasks  4096: 1.59 / 3.41   12,288: 3.14 / 3.99
//   9 tasks  4096: 1.71 / 3.75   16,384: 3.97 / 5.47   24,576: 5.51 / 7.75
// Shorter traces: gaps of one kernel each (512, queues of 512), of ten (256, queues of 2048), few that take any (1024):
//   1 task   12,288: 0.25 / 0.55, 0.58 / 0.58, 0.13 / 0.90   24,576: 0.37 / 0.58, 1.02 / 0.61, 0.18 / 0.92
//   2 tasks  8192: 0.29 / 0.67, 0.97 / 1.01, 0.12 / 1.15   12,288: 0.37 / 0.69, 1.31 / 1.02, 0.15 / 1.17
//   3 tasks  12,288: 0.42 / 0.83, 1.40 / 1.25, 0.17 / 1.45   6 tasks  12,288: 0.55 / 1.10, 1.54 / 1.56, 0.23 / 1.91
//   9 tasks  24,576: 1.06 / 2.18, 2.96 / 3.10, 0.49 / 3.73   16 tasks  24,576: 1.37 / 2.47, 3.25 / 3.44, 0.77 / 4.01
// (Ten kernels per gap are better off with the groups from 12,288 scenarios of one task and 8192 of two to five on; what
// gaps take is not known here, and the other shapes gain more than that one loses.)
bool prio_by_wave(uint64_t widest, uint64_t n_scenarios) {
  return widest <= 16 && n_scenarios <= (widest <= 1 || widest > 8 ? 24576u : 12288u);
}

}  // namespace

extern "C" {

size_t fikit_prio_fill_workspace_bytes(uint64_t n_ids, uint32_t n_tasks, uint64_t n_scenarios) {
  (void)n_scenarios;
  if (n_ids >= MAX_ELEMS) return 0;
  Carver c;
  c.take(256);
  c.take(static_cast<uint64_t>(n_tasks) * 4);
  c.take(static_cast<uint64_t>(n_tasks) * 8);
  c.take(n_ids * 8 + GF_PAD);
  c.take(n_ids * 8 + GF_PAD);
  return static_cast<size_t>(c.at);
}

int fikit_prio_fill(const uint64_t* d_ids, const uint64_t* d_task_offsets, uint32_t n_tasks, const fikit_row* d_rows,
                    const uint64_t* d_task_row_offsets, const uint32_t* d_hp_task, const uint64_t* d_lp_offsets,
                    const uint32_t* d_lp_task, const uint32_t* d_lp_prio, uint64_t n_scenarios,
                    const fikit_gapfill_params* h_params, const uint64_t* d_gap_offsets, uint32_t* d_fill_count,
                    int64_t* d_filled_ns, uint64_t* d_lp_placed, int64_t* d_lp_placed_ns, void* d_workspace,
                    size_t workspace_bytes, void* hip_stream) {
  if (!h_params || h_params->margin_ns < 0 || h_params->min_gap_ns < 0 || h_params->reserved != 0 ||
      h_params->predictor < FIKIT_PREDICT_P50 || h_params->predictor > FIKIT_PREDICT_MEAN)
    return FIKIT_INVALID_ARG;
  if (!d_task_offsets || !d_task_row_offsets || !d_workspace) return FIKIT_INVALID_ARG;
  if (n_scenarios >= MAX_ELEMS / FIKIT_PRIO_MAX_LP) return FIKIT_INVALID_ARG;
  if (n_scenarios > 0 && (!d_hp_task || !d_lp_offsets || !d_gap_offsets || n_tasks == 0)) return FIKIT_INVALID_ARG;
  if (!aligned(d_ids, 8) || !aligned(d_task_offsets, 8) || !aligned(d_rows, 16) || !aligned(d_task_row_offsets, 8) ||
      !aligned(d_hp_task, 4) || !aligned(d_lp_offsets, 8) || !aligned(d_lp_task, 4) || !aligned(d_lp_prio, 4) ||
      !aligned(d_gap_offsets, 8) || !aligned(d_fill_count, 4) || !aligned(d_filled_ns, 8) || !aligned(d_lp_placed, 8) ||
      !aligned(d_lp_placed_ns, 8) || !aligned(d_workspace, 256))
    return FIKIT_INVALID_ARG;
  if (n_scenarios == 0) return FIKIT_OK;

  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint64_t n_ids = 0, n_gaps = 0, n_entries = 0;
  Reads counts(st);
  if (int rc = counts.add(&n_ids, d_task_offsets + n_tasks, 8)) return rc;
  if (int rc = counts.add(&n_gaps, d_gap_offsets + n_scenarios, 8)) return rc;
  if (int rc = counts.add(&n_entries, d_lp_offsets + n_scenarios, 8)) return rc;
  if (int rc = counts.wait(false)) return rc;
  if (n_ids >= MAX_ELEMS || n_gaps >= MAX_ELEMS || n_entries >= MAX_ELEMS) return FIKIT_INVALID_ARG;
  if (n_ids > 0 && (!d_ids || !d_rows)) return FIKIT_INVALID_ARG;
  if (n_gaps > 0 && (!d_fill_count || !d_filled_ns)) return FIKIT_INVALID_ARG;
  if (n_entries > 0 && (!d_lp_task || !d_lp_prio || !d_lp_placed || !d_lp_placed_ns)) return FIKIT_INVALID_ARG;
  if (workspace_bytes < fikit_prio_fill_workspace_bytes(n_ids, n_tasks, n_scenarios)) return FIKIT_WORKSPACE_TOO_SMALL;

  unsigned char* ws = static_cast<unsigned char*>(d_workspace);
  Carver c;
  Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + c.take(256));
  uint32_t* role = reinterpret_cast<uint32_t*>(ws + c.take(static_cast<uint64_t>(n_tasks) * 4));
  uint64_t* lp_total = reinterpret_cast<uint64_t*>(ws + c.take(static_cast<uint64_t>(n_tasks) * 8));
  int64_t* pe = reinterpret_cast<int64_t*>(ws + c.take(n_ids * 8 + GF_PAD));   // the 32-bit arrays share the space of the 64-bit ones
  int64_t* pg = reinterpret_cast<int64_t*>(ws + c.take(n_ids * 8 + GF_PAD));
  uint32_t* lp_e = reinterpret_cast<uint32_t*>(pe);
  uint2* hp_eg = reinterpret_cast<uint2*>(pg);
  // (behind the 32-bit execution times, in the half of their space that the 64-bit ones would take; an even number of launches in)
  const uint64_t listed_at = (n_ids + 1) / 2 * 8;
  // The waves' order is made where waves will walk.  The widest scenario, which decides that, is not known yet: the average one
  // stands in for it (30,000 scenarios of one task: 557 us with lists that nobody reads, 555 without).
  const GfOrder order = prio_by_wave((n_entries + n_scenarios - 1) / n_scenarios, n_scenarios)
                            ? scenario_order(ctrl, reinterpret_cast<unsigned char*>(pe) + listed_at + GF_PAD, n_ids * 8 - listed_at, n_scenarios)
                            : GfOrder{nullptr, nullptr};

  Tracer tr(st);
  tr.mark("pf_setup");
  FIKIT_COUNT_LAUNCH(k_gf_clear, dim3(blocks_for(n_tasks, 256)), dim3(256), 0, st, ctrl, role, lp_total,
                     static_cast<uint32_t*>(nullptr), n_tasks);
  FIKIT_COUNT_LAUNCH(k_validate_offsets, dim3(blocks_for(n_tasks, 256)), dim3(256), 0, st, d_task_offsets, n_tasks, n_ids, ctrl);
  FIKIT_COUNT_LAUNCH(k_pf_scenarios, dim3(blocks_for(n_scenarios, 256)), dim3(256), 0, st, d_task_offsets, n_tasks, d_hp_task,
                     d_lp_offsets, d_lp_task, d_lp_prio, n_scenarios, n_entries, d_gap_offsets, role, order, ctrl);
  FIKIT_HIP(hipGetLastError());
  tr.mark("host_sync");
  Ctrl h{};
  if (int rc = read_ctrl(ctrl, &h, st, false)) return rc;   // the widest scenario decides how many lanes share one
  if (int rc = status_from_bits(h.status)) return rc;
  const uint32_t widest = h.n_class[3];
  // Up to 64 low-priority tasks per scenario: a wave or a group of lanes per scenario on 32-bit predictions; the 64-bit
  // kernels then only run if a prediction did not fit (they check Ctrl::wide).  More tasks: the 64-bit kernels.
  const bool groups = widest <= PF_MAX_LP;
  if (groups) {
    tr.mark("k_gf_predict32");
    FIKIT_COUNT_LAUNCH(k_gf_predict32, dim3(n_tasks, predict_parts(n_ids, n_tasks)), dim3(PRED_THREADS), 0, st, d_ids, d_task_offsets,
                       n_tasks, d_rows, d_task_row_offsets, role, static_cast<const int64_t*>(nullptr), lp_e, hp_eg, lp_total,
                       static_cast<uint32_t>(h_params->predictor), static_cast<const uint32_t*>(nullptr),
                       static_cast<const Ctrl*>(nullptr), static_cast<uint64_t>(0), ctrl);
    const uint32_t vec_ok = (aligned(d_fill_count, 16) && aligned(d_filled_ns, 16)) ? 1u : 0u;
    int rc = FIKIT_OK;
#define FIKIT_PF_WALK(W)                                                                                                   \
  rc = launch_prio_walk<W>(st, d_task_offsets, d_hp_task, d_lp_offsets, d_lp_task, d_lp_prio, n_scenarios, d_gap_offsets, \
                           lp_e, hp_eg, h_params->margin_ns, h_params->min_gap_ns, d_fill_count, d_filled_ns, d_lp_placed, \
                           d_lp_placed_ns, vec_ok, ctrl)
#define FIKIT_PF_WAVE(K)                                                                                                      \
  FIKIT_COUNT_LAUNCH(k_pf_walk_wave<K>, dim3(blocks_for(n_scenarios, WW_THREADS / WAVE)), dim3(WW_THREADS), 0, st,            \
                     d_task_offsets, d_hp_task, d_lp_offsets, d_lp_task, d_lp_prio, static_cast<uint32_t>(n_scenarios),       \
                     d_gap_offsets, lp_e, hp_eg, h_params->margin_ns, h_params->min_gap_ns, d_fill_count, d_filled_ns,        \
                     d_lp_placed, d_lp_placed_ns, order, ctrl)
    const bool waves = prio_by_wave(widest, n_scenarios);
    tr.mark(waves ? "k_pf_walk_wave" : "k_pf_walk");
    if (waves && widest <= 1) FIKIT_PF_WAVE(64);
    else if (waves && widest <= 2) FIKIT_PF_WAVE(32);
    else if (waves && widest <= 4) FIKIT_PF_WAVE(16);
    else if (waves && widest <= 8) FIKIT_PF_WAVE(8);
    else if (waves) FIKIT_PF_WAVE(4);
    else if (widest <= 1) FIKIT_PF_WALK(1);
    else if (widest <= 2) FIKIT_PF_WALK(2);
    else if (widest <= 4) FIKIT_PF_WALK(4);
    else if (widest <= 8) FIKIT_PF_WALK(8);
    else if (widest <= 16) FIKIT_PF_WALK(16);
    else if (widest <= 32) FIKIT_PF_WALK(32);
    else FIKIT_PF_WALK(64);
#undef FIKIT_PF_WALK
#undef FIKIT_PF_WAVE
    if (rc) return rc;
  }
  if (!groups) {
    // the 64-bit kernels, as if a prediction had not fitted
    FIKIT_COUNT_LAUNCH(k_fill_u32, dim3(1), dim3(64), 0, st, &ctrl->wide, static_cast<uint64_t>(1), 1u);
  }
  return finish_gapfill(st, tr, ctrl, [&]() -> int {
    FIKIT_COUNT_LAUNCH(k_gf_predict, dim3(n_tasks), dim3(PRED_THREADS), 0, st, d_ids, d_task_offsets, n_tasks, d_rows,
                       d_task_row_offsets, role, pe, pg, static_cast<int64_t*>(nullptr), static_cast<uint32_t>(h_params->predictor),
                       ctrl);
    FIKIT_COUNT_LAUNCH(k_pf_walk_wide, dim3(blocks_for(n_scenarios, 64)), dim3(64), 0, st, d_task_offsets, d_hp_task, d_lp_offsets,
                       d_lp_task, d_lp_prio, n_scenarios, d_gap_offsets, pe, pg, h_params->margin_ns, h_params->min_gap_ns,
                       d_fill_count, d_filled_ns, d_lp_placed, d_lp_placed_ns, ctrl);
    FIKIT_HIP(hipGetLastError());
    return FIKIT_OK;
  });
}

size_t fikit_pairing_workspace_bytes(uint32_t n_tasks) {
  Carver c;
  c.take(256);
  c.take(static_cast<uint64_t>(n_tasks) * 8);
  return static_cast<size_t>(c.at);
}

int fikit_pairing_best(const uint32_t* d_hp_task, const uint32_t* d_lp_task, uint64_t n_scenarios, uint32_t n_tasks,
                       const uint64_t* d_gap_offsets, const int64_t* d_filled_ns, const int64_t* d_lp_completion_ns,
                       int64_t* d_scenario_filled_ns, uint64_t* d_best_scenario, uint32_t* d_best_lp,
                       int64_t* d_best_filled_ns, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (!d_workspace || n_scenarios >= (1ull << 31)) return FIKIT_INVALID_ARG;   // (one workgroup per scenario)
  if (n_tasks > 0 && (!d_best_scenario || !d_best_lp || !d_best_filled_ns)) return FIKIT_INVALID_ARG;
  if (n_scenarios > 0 &&
      (!d_hp_task || !d_lp_task || !d_gap_offsets || !d_lp_completion_ns || !d_scenario_filled_ns || n_tasks == 0))
    return FIKIT_INVALID_ARG;
  if (!aligned(d_hp_task, 4) || !aligned(d_lp_task, 4) || !aligned(d_gap_offsets, 8) || !aligned(d_filled_ns, 8) ||
      !aligned(d_lp_completion_ns, 8) || !aligned(d_scenario_filled_ns, 8) || !aligned(d_best_scenario, 8) ||
      !aligned(d_best_lp, 4) || !aligned(d_best_filled_ns, 8) || !aligned(d_workspace, 256))
    return FIKIT_INVALID_ARG;
  if (workspace_bytes < fikit_pairing_workspace_bytes(n_tasks)) return FIKIT_WORKSPACE_TOO_SMALL;
  if (n_tasks == 0) return FIKIT_OK;

  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (n_scenarios > 0 && !d_filled_ns) {   // (allowed if there are no gaps, which only the device knows)
    uint64_t n_gaps = 0;
    Reads r(st);
    if (int rc = r.add(&n_gaps, d_gap_offsets + n_scenarios, 8)) return rc;
    if (int rc = r.wait(false)) return rc;
    if (n_gaps > 0) return FIKIT_INVALID_ARG;
  }
  unsigned char* ws = static_cast<unsigned char*>(d_workspace);
  Carver c;
  Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + c.take(256));
  long long* top_filled = reinterpret_cast<long long*>(ws + c.take(static_cast<uint64_t>(n_tasks) * 8));
  unsigned long long* best_scenario = reinterpret_cast<unsigned long long*>(d_best_scenario);

  Tracer tr(st);
  tr.mark("pair_setup");
  FIKIT_COUNT_LAUNCH(k_pair_init, dim3(blocks_for(n_tasks, 256)), dim3(256), 0, st, n_tasks,
                     n_scenarios > 0 ? d_gap_offsets + n_scenarios : static_cast<const uint64_t*>(nullptr), top_filled, best_scenario,
                     d_best_lp, d_best_filled_ns, ctrl);
  if (n_scenarios > 0) {
    tr.mark("k_pair_sum");
    const bool waves = n_scenarios >= PAIR_WAVES;
    const uint64_t most = waves ? PAIR_STAY : n_scenarios;
    const uint64_t groups = waves ? (n_scenarios + PAIR_THREADS / WAVE - 1) / (PAIR_THREADS / WAVE) : n_scenarios;
    FIKIT_COUNT_LAUNCH(waves ? k_pair_sum<WAVE> : k_pair_sum<PAIR_THREADS>, dim3(static_cast<uint32_t>(groups < most ? groups : most)),
                       dim3(PAIR_THREADS), 0, st, d_hp_task, d_lp_task, static_cast<uint32_t>(n_scenarios), n_tasks, d_gap_offsets,
                       d_filled_ns, d_scenario_filled_ns, top_filled, ctrl);
    tr.mark("k_pair_pick");
    FIKIT_COUNT_LAUNCH(k_pair_pick, dim3(blocks_for(n_scenarios, PAIR_THREADS)), dim3(PAIR_THREADS), 0, st, d_hp_task, d_lp_task, n_scenarios,
                       n_tasks, d_scenario_filled_ns, d_lp_completion_ns, top_filled, best_scenario, d_best_lp, d_best_filled_ns, ctrl);
    if (n_tasks > PAIR_LAST_TASKS)
      FIKIT_COUNT_LAUNCH(k_pair_finish, dim3(blocks_for(n_tasks, PAIR_THREADS)), dim3(PAIR_THREADS), 0, st, n_tasks, d_lp_task,
                         d_scenario_filled_ns, best_scenario, d_best_lp, d_best_filled_ns, ctrl);
  }
  FIKIT_HIP(hipGetLastError());
  tr.mark("host_sync");
  Ctrl h{};
  if (int rc = read_ctrl(ctrl, &h, st)) return rc;
  return status_from_bits(h.status);
}

size_t fikit_profile_merge_workspace_bytes(uint32_t n_tasks) {
  Carver c;
  c.take(256);
  c.take((static_cast<uint64_t>(n_tasks) + 1) * 4);
  c.take(((static_cast<uint64_t>(n_tasks) + 1) / SCAN_TILE + 2) * 4);
  return static_cast<size_t>(c.at);
}

int fikit_profile_merge(const fikit_row* d_rows_a, const uint64_t* d_task_row_offsets_a, const fikit_row* d_rows_b,
                        const uint64_t* d_task_row_offsets_b, uint32_t n_tasks, fikit_row* d_rows_out, uint64_t row_capacity,
                        uint64_t* d_task_row_offsets_out, uint64_t* h_n_rows, void* d_workspace, size_t workspace_bytes,
                        void* hip_stream) {
  if (h_n_rows) *h_n_rows = 0;
  if (!h_n_rows || !d_task_row_offsets_a || !d_task_row_offsets_b || !d_task_row_offsets_out || !d_workspace || n_tasks == 0)
    return FIKIT_INVALID_ARG;
  if (row_capacity > 0 && !d_rows_out) return FIKIT_INVALID_ARG;
  if (!aligned(d_rows_a, 16) || !aligned(d_rows_b, 16) || !aligned(d_rows_out, 16) || !aligned(d_task_row_offsets_a, 8) ||
      !aligned(d_task_row_offsets_b, 8) || !aligned(d_task_row_offsets_out, 8) || !aligned(d_workspace, 256))
    return FIKIT_INVALID_ARG;
  if (workspace_bytes < fikit_profile_merge_workspace_bytes(n_tasks)) return FIKIT_WORKSPACE_TOO_SMALL;

  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  // The numbers of rows live on the device, whose first kernel looks at them; the host only waits for them where a table may be
  // missing.
  if (!d_rows_a || !d_rows_b) {
    uint64_t na = 0, nb = 0;
    Reads counts(st);
    if (int rc = counts.add(&na, d_task_row_offsets_a + n_tasks, 8)) return rc;
    if (int rc = counts.add(&nb, d_task_row_offsets_b + n_tasks, 8)) return rc;
    if (int rc = counts.wait(false)) return rc;
    if ((na > 0 && !d_rows_a) || (nb > 0 && !d_rows_b)) return FIKIT_INVALID_ARG;
  }

  unsigned char* ws = static_cast<unsigned char*>(d_workspace);
  Carver c;
  Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + c.take(256));
  uint32_t* dcount = reinterpret_cast<uint32_t*>(ws + c.take((static_cast<uint64_t>(n_tasks) + 1) * 4));
  uint32_t* sums = reinterpret_cast<uint32_t*>(ws + c.take(((static_cast<uint64_t>(n_tasks) + 1) / SCAN_TILE + 2) * 4));

  Tracer tr(st);
  tr.mark("merge_count");
  const uint32_t grid = n_tasks < 65536u ? n_tasks : 65536u;
  // The kernel with the small LDS tables takes every task, and puts those that do not fit them on a list for the one with the
  // larger tables; or that one takes all (k_merge_begin).  (The list lives where nothing else does at that time: in the row
  // offsets before they exist, in the row counts after.)
  const uint32_t large_grid = n_tasks < MERGE_LARGE_WORKGROUPS ? n_tasks : MERGE_LARGE_WORKGROUPS;
  auto pass = [&](auto small, auto large, uint32_t* list) {
    FIKIT_COUNT_LAUNCH(small, dim3(grid), dim3(MERGE_THREADS), 0, st, d_rows_a, d_task_row_offsets_a, d_rows_b, d_task_row_offsets_b,
                       n_tasks, dcount, d_task_row_offsets_out, d_rows_out, row_capacity, list, ctrl);
    FIKIT_COUNT_LAUNCH(large, dim3(large_grid), dim3(MERGE_THREADS), 0, st, d_rows_a, d_task_row_offsets_a, d_rows_b, d_task_row_offsets_b,
                       n_tasks, dcount, d_task_row_offsets_out, d_rows_out, row_capacity, list, ctrl);
  };
  FIKIT_COUNT_LAUNCH(k_merge_begin, dim3(1), dim3(64), 0, st, d_task_row_offsets_a + n_tasks, d_task_row_offsets_b + n_tasks, n_tasks, MAX_ELEMS, ctrl);
  pass(k_merge<0, MERGE_IDS_SMALL, false>, k_merge<0, MERGE_IDS, true>, reinterpret_cast<uint32_t*>(d_task_row_offsets_out));
  if (int rc = row_offsets_enqueue(dcount, static_cast<uint64_t>(n_tasks) + 1, sums, d_task_row_offsets_out, ctrl, st)) return rc;
  tr.mark("k_merge_rows");   // (does nothing if a check failed or the rows are too many)
  pass(k_merge<1, MERGE_IDS_SMALL, false>, k_merge<1, MERGE_IDS, true>, dcount);
  FIKIT_HIP(hipGetLastError());
  tr.mark("host_sync");
  Ctrl h{};
  if (int rc = read_ctrl(ctrl, &h, st)) return rc;
  if (int rc = status_from_bits(h.status)) return rc;
  *h_n_rows = h.n_rows;
  return h.n_rows > row_capacity ? FIKIT_ROW_CAPACITY : FIKIT_OK;
}

}  // extern "C"
