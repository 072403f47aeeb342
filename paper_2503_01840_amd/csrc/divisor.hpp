// Division by multiplication, on the host and in kernels (Granlund and Montgomery, "Division by invariant integers using multiplication").
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define HOST_AND_DEVICE __host__ __device__ __forceinline__
#else
#define HOST_AND_DEVICE inline
#endif

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
HOST_AND_DEVICE int operator/(int n, const Divisor& by) {
  return (int)(((uint32_t)((uint64_t)(uint32_t)n * by.mul >> 32) + (uint32_t)n) >> by.shift);
}
HOST_AND_DEVICE int operator%(int n, const Divisor& by) { return n - n / by * by.d; }
