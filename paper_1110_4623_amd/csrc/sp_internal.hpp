// Host-side internals of libsp.so shared by the translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "sp.h"
#include "sp/atomics.hpp"

struct sp_default_entry {
  uint32_t kind;
  sp_params p;
  bool builtin;  // the library's own entry: its kind may give way to another by size
};

struct sp_ctx {
  // Objects created from the context (barriers, mutexes, semaphores, graphs) hold a
  // reference: sp_fini releases the context's device resources at once, but the struct
  // itself lives until the last object is destroyed, so an object destroyed after
  // sp_fini (as a garbage-collecting caller may do at exit) touches no freed memory.
  int refs = 0;
  bool closed = false;
  int device = 0;
  hipDeviceProp_t prop{};
  int last_hip = 0;
  uint32_t cu_count = 0;
  uint32_t xcd_count = 0;
  uint32_t xcc_mask = 0;  // XCC ids seen at sp_init (bit i = id i)
  uint32_t wall_khz = 100000;
  uint32_t* d_err = nullptr;   // watchdog word, own 256-byte block
  uint32_t* h_err = nullptr;   // pinned: the watchdog word as a run's last kernel found it
  // pinned staging of sp_buffer_read_strided, made by its first call
  uint32_t* h_stage = nullptr;
  unsigned long long* d_sums = nullptr;  // kSumSlots partial sums, one per 128-byte line
  // occupancy of the library's kernels, asked of the runtime once per kernel and size
  struct Occupancy { const void* kern; uint32_t lanes, per_cu; };
  std::vector<Occupancy> occupancy;
  uint32_t* d_scratch = nullptr;  // small staging area (4 KiB) for state readback
  // the allocation-free entry point's fixed workspace on this device (a file-scope device
  // array; its address is looked up once per device at sp_init)
  uint32_t* static_scratch = nullptr;
  uint64_t static_scratch_words = 0;
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  hipStream_t capture_stream = nullptr;
  hipStream_t setup_stream = nullptr;  // work done while creating objects (not the caller's)
  sp_default_entry defaults[3][2];
};

namespace spi {

// Looks up (once per device) the address of the allocation-free entry point's fixed
// workspace and records it in the context.  The context's device must be current.
int static_scratch_setup(sp_ctx* ctx);


// Records a failing HIP call in the context and returns SP_E_HIP from the caller.
#define SP_HIP(ctx, call)                                      \
  do {                                                         \
    hipError_t e_ = (call);                                    \
    if (e_ != hipSuccess) {                                    \
      if (ctx) (ctx)->last_hip = (int)e_;                      \
      return SP_E_HIP;                                         \
    }                                                          \
  } while (0)

#define SP_CHECK(expr)                  \
  do {                                  \
    int rc_ = (expr);                   \
    if (rc_ != SP_OK) return rc_;       \
  } while (0)

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

// A context that can still run work (not NULL, not finalized).
inline bool usable(const sp_ctx* ctx) { return ctx && !ctx->closed; }
// Object lifetime: every create that succeeds takes a reference, every destroy drops it;
// the last drop after sp_fini deletes the context.
inline void ctx_ref(sp_ctx* ctx) { ++ctx->refs; }
inline void ctx_unref(sp_ctx* ctx) {
  if (--ctx->refs == 0 && ctx->closed) delete ctx;
}

// Normalized parameters (defaults filled, ranges clamped); returns SP_E_INVAL on bad
// values.
int normalize(const sp_ctx* ctx, const sp_params* in, sp_params* out);

inline uint32_t stride_words(const sp_params& p) { return std::max<uint32_t>(1, p.pad_bytes / 4); }

inline uint64_t timeout_ticks(const sp_ctx* ctx, const sp_params& p) {
  return (uint64_t)p.timeout_ms * ctx->wall_khz;
}

inline sp::BackoffCfg backoff_cfg(const sp_params& p, uint32_t* private_word) {
  sp::BackoffCfg c;
  c.kind = p.backoff;
  c.imin = p.backoff_min;
  c.imax = p.backoff_max;
  c.unit = p.backoff_unit;
  c.private_word = private_word;
  return c;
}

// Up to kMax ranges of uint32 words set by one kernel (no memset nodes, so launches stay
// capturable): what a run has to reset costs one launch, not one per array.  A range too many
// is counted but not kept, and the reset refuses the list.
struct Resets {
  static constexpr uint32_t kMax = 8;
  struct Range {
    uint32_t* p;
    uint64_t words;
    uint32_t value;
  } r[kMax];
  uint32_t n = 0;
  void add(void* p, uint64_t words, uint32_t value = 0) {
    if (!words) return;
    if (n < kMax) r[n] = Range{static_cast<uint32_t*>(p), words, value};
    ++n;
  }
};
int reset(sp_ctx* ctx, const Resets& z, hipStream_t s);
// One range.
int fill_u32(sp_ctx* ctx, uint32_t* d, uint64_t words, uint32_t value, hipStream_t s);

// True while `s` is being captured into a HIP graph (sp_graph_begin): run calls then
// record their kernels and skip timing, host waits and host readbacks.
bool capturing(hipStream_t s);

// Around a run's main kernel.  begin_timed resets `z` and the watchdog word and records
// ev0; mark_end records ev1; the run's last kernel (its own, or end_timed's) copies the
// watchdog word into h_err (report_error); wait_done waits for the stream once, reads the
// time and h_err and fills st.  Under capture nothing is timed, awaited or read: the graph's
// launcher does that, and clears the watchdog word, once per replay.
// What bounds a small run is the number of launches and waits around its kernel: on an
// MI355X a mutex run of 24 workgroups took 135-137 us from call to words with a fill kernel
// per array, a copy of the watchdog word and a second wait for the gather, 115 us with one
// reset kernel, the watchdog word in pinned memory and one wait.
int begin_timed(sp_ctx* ctx, hipStream_t s, Resets z = Resets());
int mark_end(sp_ctx* ctx, hipStream_t s);
int wait_done(sp_ctx* ctx, hipStream_t s, sp_stats* st, uint32_t nwg, uint32_t lanes,
              uint32_t resident_per_cu, uint64_t ops);
int end_timed(sp_ctx* ctx, hipStream_t s, sp_stats* st, uint32_t nwg, uint32_t lanes,
              uint32_t resident_per_cu, uint64_t ops);
__device__ __forceinline__ void report_error(const uint32_t* err, uint32_t* h_err) {
  __hip_atomic_store(h_err, __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Where the workgroups of a microbenchmark add their sums.  One word takes atomics 12 ns
// apart, so the sums of 8192 workgroups took 104 us behind a 64 MiB read of 14 us: workgroup
// b adds to slot b mod kSumSlots, each on its own line, and the call's last kernel adds the
// slots to the output.  The slots are the context's, so a recorded call, which may be
// replayed beside others, adds to the output itself (mask 0).
constexpr uint32_t kSumSlots = 256, kSumStride = 16;
struct Sums {
  unsigned long long* p;
  uint32_t mask;
  __device__ unsigned long long* slot(uint32_t b) const { return p + (b & mask) * kSumStride; }
};
// The sums of a call on `s`; what they need reset is added to z.
Sums sums_for(sp_ctx* ctx, unsigned long long* out, hipStream_t s, Resets* z);

// A kernel that reports the watchdog word and adds the slots (if any) to `out`, then
// wait_done.  end_timed: mark_end, then this without sums.
int finish(sp_ctx* ctx, hipStream_t s, sp_stats* st, uint32_t nwg, uint32_t lanes,
           uint32_t resident_per_cu, uint64_t ops, const Sums& sums, unsigned long long* out);

// Workgroups of `kern` (launched with `lanes` threads) that fit on one CU at once: the
// runtime's occupancy figure checked against the kernel's own VGPR and LDS use
// (sp_resident_per_cu).
int resident_per_cu(sp_ctx* ctx, const void* kern, uint32_t lanes, uint32_t* per_cu);

inline bool lanes_ok(uint32_t lanes) { return lanes >= 64 && lanes <= 1024 && lanes % 64 == 0; }

// Device memory owned for the duration of one call; the caller synchronizes the stream
// before it goes out of scope.
struct DeviceScratch {
  void* p = nullptr;
  DeviceScratch() = default;
  DeviceScratch(const DeviceScratch&) = delete;
  DeviceScratch& operator=(const DeviceScratch&) = delete;
  ~DeviceScratch() {
    if (p) (void)hipFree(p);
  }
  template <typename T>
  T* as() const {
    return static_cast<T*>(p);
  }
};

inline uint32_t bucket_of(uint32_t contenders) { return contenders >= 64 ? 1u : 0u; }
// Barriers: every workgroup is a contender.  Us per round, central counter / per-XCD, 256
// lanes: plain data, 16 workgroups 1.69 / 2.35, 32 2.35 / 2.34, 40 2.65 / 2.36, 48 2.98 /
// 2.42, 64 3.50 / 2.51; agent-scope data 1.23 / 1.96, 1.53 / 1.95, 1.53 / 1.96, 1.62 / 1.96,
// 1.78 / 2.00.  The two meet at 32 for plain data and above 64 for agent-scope data; one line
// serves both, and the high bucket starts at 40.
inline uint32_t barrier_bucket_of(uint32_t nwg) { return nwg >= 40 ? 1u : 0u; }
// A default mutex whose bucket names the CU-cohort lock runs it only where a lock has
// enough contenders per CU; below that few hand-overs stay within a CU and the XCD-cohort
// lock is faster.  M acquisitions/s, CU-cohort / XCD-cohort, 16 words: plain data, one lock,
// 512 workgroups 0.93 / 1.02, 640 1.17 / 1.02, 1024 1.66 / 1.02; 2048 workgroups on 2
// locks 2.57 / 2.05, 3 3.53 / 3.15, 4 4.43 / 4.23, 8 7.81 / 8.56: from 2.5 per CU and lock
// (2 per CU go either way).  Coherent data, whose sections go to memory
// whatever the hand-over: 2048 on one lock 1.12 / 1.03, on 2 2.11 / 2.06, on 3 3.07 / 3.11,
// on 4 4.03 / 4.16: from 5, where the gain is sure.
inline bool cu_cohort_pays(uint64_t nwg, uint64_t nlocks, uint64_t cu_count, bool coherent) {
  return 2 * nwg >= (coherent ? 10 : 5) * nlocks * cu_count;
}
// The K = 1 semaphore's line between one chain and the CU-cohort lock.  M pairs/s, lock /
// chain, holds U[0, 2000] clocks: plain data, 256 workgroups 0.61 / 0.74, 384 0.74 / 0.72, 512
// 0.84 / 0.72, 2048 0.99 / 0.66; coherent 384 0.89 / 0.93, 512 0.96 / 0.91, 2048 0.95 / 0.84.
inline bool cu_lock_pays(uint64_t nwg, uint64_t cu_count) { return nwg >= 2 * cu_count; }
// A default mutex whose low bucket is the library's own (the spin lock with the paper's
// backoff) runs the XCD-cohort lock where a lock has enough contenders that some of them
// share an XCD.  M acquisitions/s, spin / XCD-cohort, 16 words: plain data, 64 workgroups
// on 16 locks 9.4 / 9.0, 96 10.1 / 10.3, 128 10.2 / 11.2, 256 10.6 / 13.2; 600 on 100 39.5
// / 43.0; 2048 on 256 53.9 / 62.9, on 64 28 / 48; 8 on one
// lock 0.80 / 0.62 (one per XCD), 24 on 3 2.24 / 2.27: from six per lock and three per XCD.
// Coherent data, where there is no writeback to save: 128 on 16 locks 14.0 / 13.5, 256 14.5
// / 14.4, 2048 on 128 102 / 106, on 64 38 / 59: from 16 per lock.
inline bool cohort_pays(uint64_t nwg, uint64_t nlocks, uint64_t xcds, bool coherent) {
  return nwg >= (coherent ? 16 : 6) * nlocks && nwg >= 3 * xcds;
}

}  // namespace spi
