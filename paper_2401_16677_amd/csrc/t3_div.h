// Division by a number the host knows.  Plain C++ on the host side.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define T3_HOST_DEVICE __host__ __device__
#else
#define T3_HOST_DEVICE
#endif

namespace t3k {

// Division of numbers below 2^31 by one that the host knows, without dividing (the kernels decode a grid
// position between two tiles, where the matrix cores wait for it): with 2^(s - 1) < d <= 2^s and
// m = floor(2^32 (2^s - d) / d) + 1, n / d = (high word of m n + n) >> s.  (m n / 2^32 + n exceeds
// 2^s n / d by less than 2^s / d, n <= 2^31 - 1 keeps the sum in 32 bits.)
struct FastDiv {
  uint32_t m, s, d;
};
T3_HOST_DEVICE inline FastDiv fast_div(uint32_t d) {
  uint32_t s = 0;
  while ((1u << s) < d) ++s;
  return FastDiv{(uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << s) - d)) / d + 1u), s, d};
}
T3_HOST_DEVICE inline uint32_t div_by(uint32_t n, const FastDiv &f) {
#if defined(__HIP_DEVICE_COMPILE__)
  return (__umulhi(f.m, n) + n) >> f.s;
#else
  return ((uint32_t)(((uint64_t)f.m * n) >> 32) + n) >> f.s;
#endif
}

}  // namespace t3k
