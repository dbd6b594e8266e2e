// One range more than a reset takes: refused by the reset, and nothing written past the list.
#include <cstdio>

#include "sp_internal.hpp"

int main() {
  struct {
    spi::Resets z;
    uint32_t guard[16];
  } s;
  for (uint32_t& g : s.guard) g = 0xA5A5A5A5u;
  uint32_t word = 0;
  for (uint32_t i = 0; i < spi::Resets::kMax + 1; ++i) s.z.add(&word, 1, 0x11111111u * i);
  for (const uint32_t& g : s.guard)
    if (const_cast<const volatile uint32_t&>(g) != 0xA5A5A5A5u) return 3;
  if (s.z.r[spi::Resets::kMax - 1].value != 0x77777777u) return 4;
  if (spi::reset(nullptr, s.z, nullptr) != SP_E_INVAL) return 5;  // before any use of the GPU
  printf("refused\n");
  return 0;
}
