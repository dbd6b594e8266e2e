// The per-XCD barrier in a caller's own kernel, with placement tables of the caller's choice:
// groups or arrival blocks too small for the run, which sp_barrier_create never makes, send
// every round to the counter tree.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "sp/barrier.hpp"

namespace {

template <bool COHERENT>
__global__ SP_FULL_OCCUPANCY void k_rounds(sp::BarrierState s, uint32_t rounds, uint32_t seed,
                                           uint32_t* slots, uint32_t* out, uint32_t* err,
                                           uint64_t timeout) {
  const sp::Ctl ctl{err, sp::wall_clock() + timeout};
  const uint32_t b = blockIdx.x, N = s.nwg;
  uint32_t chk = 0;
  for (uint32_t r = 0; r < rounds; ++r) {
    uint32_t* half = slots + (r & 1) * N;
    if (threadIdx.x == blockDim.x - 1) {
      const uint32_t v = sp::sm32(seed ^ (b << 16) ^ r);
      if constexpr (COHERENT) sp::st_relaxed(half + b, v);
      else half[b] = v;
    }
    if (!sp::barrier_wait<SP_BARRIER_XCD>(s, r, ctl)) return;
    if (threadIdx.x == 64 % blockDim.x) {
      const uint32_t* p = half + (b + r) % N;
      if constexpr (COHERENT) chk ^= sp::ld_relaxed(p);
      else chk ^= *p;
    }
  }
  if (threadIdx.x == 64 % blockDim.x) out[b] = chk;
}

}  // namespace

// Runs `rounds` rounds of nwg x lanes with `groups` XCD groups (1-16) whose arrival blocks are
// said to take `xblock` members (the memory takes all of them); out_host: nwg checksums;
// info[0] = registrations that did not fit, info[1] = the watchdog word.
extern "C" int sp_test_barrier_fallback(uint32_t nwg, uint32_t lanes, uint32_t rounds,
                                        uint32_t seed, uint32_t coherent, uint32_t groups,
                                        uint32_t xblock, uint32_t* out_host, uint32_t* info) {
  if (nwg == 0 || nwg > 1024 || lanes == 0 || lanes > 256 || lanes % 64 || groups == 0 ||
      groups > 16 || xblock == 0 || xblock > nwg || !out_host || !info)
    return -1;
  constexpr uint32_t kStride = 32, kCopies = 64;
  const uint64_t block = (nwg + 127) / 128 * 32;  // words of one byte per workgroup
  const uint64_t words = (6 + 3ull * groups) * kStride + groups * block +
                         (uint64_t)groups * sp::kCuLines * kStride + groups * 256ull * 2 +
                         (2ull * groups + 31) / 32 * 32 + (uint64_t)kCopies * kStride +
                         2ull * nwg + nwg;
  uint32_t* base = nullptr;
  if (hipMalloc(&base, words * 4) != hipSuccess) return -2;
  uint32_t* next = base;
  const auto take = [&](uint64_t n) {
    uint32_t* p = next;
    next += n;
    return p;
  };
  sp::BarrierState s{};
  s.nwg = nwg;
  s.stride = kStride;
  s.groups = groups;
  s.tgroups = groups < nwg ? groups : nwg;
  s.flag_stride = 1;
  s.xblock = xblock;
  s.fenced = !coherent;
  s.xcopies = kCopies % groups ? 0 : kCopies;
  s.xmstride = kStride;
  s.xmstep = groups * kStride;
  for (uint32_t x = 0; x < groups; ++x) {
    s.xoff[x] = (uint32_t)(x * block);
    s.moff[x] = x * kStride;
    s.roff[x] = x * sp::kCuLines * kStride;
  }
  s.cnt = take(kStride);
  s.gen = take(kStride);
  s.top = take(kStride);
  s.topgen = take(kStride);
  s.mismatch = take(kStride);
  s.overflow = take(kStride);
  uint32_t* err = s.overflow + 1;
  s.gcnt = take(groups * kStride);
  s.ggen = take(groups * kStride);
  s.xarrive = take(groups * kStride);
  s.larrive = take(groups * block);
  s.lrelease = take((uint64_t)groups * sp::kCuLines * kStride);
  s.cu_count = take(groups * 256);
  s.cu_rank = take(groups * 256);
  s.xcount = take((2ull * groups + 31) / 32 * 32);
  s.xcu = s.xcount + groups;
  s.xmail = take((uint64_t)kCopies * kStride);
  uint32_t* slots = take(2ull * nwg);
  uint32_t* out = take(nwg);
  int khz = 100000;
  (void)hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, 0);
  const uint64_t timeout = 5000ull * (uint64_t)khz;
  bool ok = next == base + words && hipMemset(base, 0, words * 4) == hipSuccess;
  if (ok) {
    if (coherent) k_rounds<true><<<nwg, lanes>>>(s, rounds, seed, slots, out, err, timeout);
    else k_rounds<false><<<nwg, lanes>>>(s, rounds, seed, slots, out, err, timeout);
    ok = hipGetLastError() == hipSuccess && hipDeviceSynchronize() == hipSuccess &&
         hipMemcpy(out_host, out, nwg * 4, hipMemcpyDeviceToHost) == hipSuccess &&
         hipMemcpy(info, s.overflow, 8, hipMemcpyDeviceToHost) == hipSuccess;
  }
  (void)hipFree(base);
  return ok ? 0 : -2;
}
