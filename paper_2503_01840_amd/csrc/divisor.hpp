// Division by multiplication (host part; common.hpp has the device's).
#pragma once
#include <cstdint>

// Division by a size of the launch, exact for 0 <= n < 2^31: three instructions.  What the compiler makes of n / d are some thirty that depend on each
// other, 0.1 to 0.2 us in front of a workgroup's first load (four of them: 0.5 us of every many-row product).
struct Divisor {
  uint32_t mul, shift;
  int d;
};
inline Divisor divisor(int d) {
  uint32_t s = 0;
  while ((1ull << s) < (uint64_t)d) ++s;
  return {(uint32_t)((((1ull << s) - (uint64_t)d) << 32) / (uint64_t)d + 1), s, d};
}
