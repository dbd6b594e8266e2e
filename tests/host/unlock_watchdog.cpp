// A CU-cohort unlock whose predecessor on the CU gave up: it has to end with the watchdog.
// Argument: "unlock" (mutex_unlock without a control block) or "cond" (cond_wait).
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "sp/cond.hpp"

using namespace sp;

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  constexpr uint32_t kStride = 4;
  std::vector<uint32_t> lockw(3 * kStride);
  std::vector<uint32_t> lines(kStride * (kXccSlots * kCohortLines + kXccSlots * kCuIds * kCuLines) + 4);
  uint32_t err = DEV_OK, cv_words[2] = {0, 0};
  MutexState s{};
  s.stride = kStride;
  s.lockw = lockw.data();
  s.ticket = lockw.data() + kStride;
  s.turn = lockw.data() + 2 * kStride;
  s.queue = reinterpret_cast<uint32_t*>((reinterpret_cast<uintptr_t>(lines.data()) + 15) & ~(uintptr_t)15);
  s.qlen = 1;
  s.qstride = kStride;
  s.cohort_bound = 64;
  s.cuq = s.queue + kXccSlots * kCohortLines * kStride;
  const Ctl ctl{&err, wall_clock() + 10'000'000};

  MutexHold first{}, second{};
  if (!mutex_lock<SP_MUTEX_CU_COHORT>(s, 0, ctl, &first)) return 3;
  uint32_t* announced = cu_line(s, 0, 0, 0, 1) + 1;
  std::thread next([&] {
    if (!mutex_lock<SP_MUTEX_CU_COHORT>(s, 0, ctl, &second)) std::_Exit(4);
  });
  while (ld(announced) != 2) sched_yield();
  mutex_unlock<SP_MUTEX_CU_COHORT>(s, 0, &first, &ctl);  // passes within the CU
  next.join();
  if (second.cu_session != 1) return 5;
  // The first holder as if the watchdog had taken it ahead of its count.
  uint32_t* done = cu_line(s, 0, 0, 0, 2);
  if (ld(done) != 1) return 6;
  st(done, 0u);
  st(&err, (uint32_t)DEV_TIMEOUT);
  if (!strcmp(argv[1], "unlock")) {
    mutex_unlock<SP_MUTEX_CU_COHORT>(s, 0, &second);
  } else {
    const CondState cv{&cv_words[0], &cv_words[1], 1};
    if (cond_wait<SP_MUTEX_CU_COHORT>(cv, s, 0, &second, ctl)) return 7;
  }
  printf("ended\n");
  return 0;
}
