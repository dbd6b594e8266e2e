// Host stand-in for include/sp/atomics.hpp: the device headers that build on it compile with
// it for the CPU, one thread per workgroup of one lane.  Agent and workgroup scope are both
// sequentially consistent atomics here (caches are the model checker's business); the
// watchdog is the device's, on the steady clock in microseconds.
#pragma once

#include <sched.h>
#include <stdint.h>

#include <algorithm>
#include <chrono>

#include "sp.h"

#define __device__
#define __forceinline__ inline
#define __shared__ static thread_local

struct Dim { uint32_t x; };
inline thread_local Dim threadIdx{0}, blockIdx{0};
inline Dim blockDim{1};
inline void __syncthreads() {}

namespace sp {

// Where this thread's workgroup runs.
inline thread_local uint32_t host_xcc = 0, host_cu = 0;
inline uint32_t xcc_id() { return host_xcc; }
inline uint32_t cu_in_xcc() { return host_cu; }

template <class T>
inline T ld(const T* p) { return __atomic_load_n(p, __ATOMIC_SEQ_CST); }
template <class T>
inline void st(T* p, T v) { __atomic_store_n(p, v, __ATOMIC_SEQ_CST); }
inline uint32_t ld_relaxed(const uint32_t* p) { return ld(p); }
inline void st_relaxed(uint32_t* p, uint32_t v) { st(p, v); }
inline uint32_t ld_cu(const uint32_t* p) { return ld(p); }
inline void st_cu(uint32_t* p, uint32_t v) { st(p, v); }
inline uint64_t ld_relaxed64(const uint64_t* p) { return ld(p); }
inline void st_relaxed64(uint64_t* p, uint64_t v) { st(p, v); }
inline uint64_t ld_xcd64(const uint64_t* p) { return ld(p); }
inline void st_xcd64(uint64_t* p, uint64_t v) { st(p, v); }
inline uint32_t add_relaxed(uint32_t* p, uint32_t v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
inline uint32_t exch_relaxed(uint32_t* p, uint32_t v) { return __atomic_exchange_n(p, v, __ATOMIC_SEQ_CST); }
inline uint32_t cas_relaxed(uint32_t* p, uint32_t e, uint32_t d) {
  __atomic_compare_exchange_n(p, &e, d, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
  return e;
}
// The device reads these 16 bytes in one access.  Here word 0 (the grant) is read first: what
// was stored before it is then seen, and the caller drops the rest unless it is its turn.
struct u32x4 { uint32_t x, y, z, w; };
inline u32x4 ld_cu128(const uint32_t* p) {
  u32x4 v;
  v.x = ld(p);
  v.y = ld(p + 1);
  const uint64_t r = ld(reinterpret_cast<const uint64_t*>(p + 2));
  v.z = (uint32_t)r;
  v.w = (uint32_t)(r >> 32);
  return v;
}
template <class T>
inline T uniform(T v) { return v; }
template <class T>
inline T* uniform_ptr(T* p) { return p; }
inline void wave_stores_complete() {}
inline void stores_complete_before_release(bool) {}
inline void fence_acquire() {}
inline void fence_release() {}
inline void st_release(uint32_t* p, uint32_t v) { st(p, v); }
inline bool reached(uint32_t a, uint32_t b) { return (int32_t)(a - b) >= 0; }
inline bool is_leader() { return threadIdx.x == 0; }
inline uint64_t wall_clock() {
  return std::chrono::duration_cast<std::chrono::microseconds>(
             std::chrono::steady_clock::now().time_since_epoch()).count();
}
inline void sleep_units(uint32_t) { sched_yield(); }

enum : uint32_t { DEV_OK = 0, DEV_TIMEOUT = 1, DEV_PARITY = 2 };
struct Ctl {
  uint32_t* err;
  uint64_t deadline;
};
struct Wait {
  Ctl ctl;
  uint32_t poll_sleep, n = 0;
  Wait(const Ctl& c, uint32_t ps) : ctl(c), poll_sleep(ps) {}
  bool tick() {
    sleep_units(poll_sleep);
    if ((++n & 63) != 0) return true;
    if (ld(ctl.err) != DEV_OK) return false;
    if (wall_clock() <= ctl.deadline) return true;
    cas_relaxed(ctl.err, DEV_OK, DEV_TIMEOUT);
    return false;
  }
};
template <class Seen>
inline bool poll(Wait& w, Seen seen) {
  while (!seen())
    if (!w.tick()) return false;
  return true;
}

struct BackoffCfg {
  uint32_t kind, imin, imax, unit;
  uint32_t* private_word;
};
struct Backoff {
  explicit Backoff(const BackoffCfg&) {}
  void operator()(const BackoffCfg&) { sched_yield(); }
};

}  // namespace sp
