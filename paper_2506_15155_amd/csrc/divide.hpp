// Division by a number that is known before a launch, as a multiplication and a shift: the compiler's division of two
// run-time integers goes through the vector unit's reciprocal, 25 dependent instructions, and a wave has three or four of
// them ahead of its first request for K.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define ELLM_BOTH __host__ __device__
#else
#define ELLM_BOTH
#endif

namespace ellm {

struct Divisor { uint32_t mul, shift; };

// d >= 1. With shift = 31 + c, 2^(c-1) < d <= 2^c, and mul = ceil(2^shift / d) < 2^32, n * mul / 2^shift is n / d plus less than
// n / 2^31 / d: its floor is that of n / d for every n < 2^31.
inline Divisor divisor(int32_t d) {
  uint32_t c = 0;
  while (((uint64_t)1 << c) < (uint64_t)d) c++;
  const uint32_t shift = 31 + c;
  return {(uint32_t)((((uint64_t)1 << shift) + (uint64_t)d - 1) / (uint64_t)d), shift};
}

// n / d, n >= 0
ELLM_BOTH inline int32_t divide(int32_t n, Divisor by) { return (int32_t)(((uint64_t)(uint32_t)n * by.mul) >> by.shift); }

}  // namespace ellm
