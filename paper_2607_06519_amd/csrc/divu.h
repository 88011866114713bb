// Division by a divisor that the host knows before a launch.
//
// floor(n / d) = (n mul) >> shift for every n < 2^31 and 1 <= d < 2^31, with
// 2^shift = 2^31 2^s, s = ceil(log2 d), mul = ceil(2^shift / d): mul is below
// 2^32, and with e = mul d - 2^shift < d <= 2^s, n mul = (n 2^shift + n e) / d
// where n e < 2^shift, so the quotient is exact.  (On the device: one 32 x 32
// product and a shift, where a division by an unknown number is some twenty
// scalar instructions.)  Plain C++, usable on the host.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define FDKV_DIVU_HD __host__ __device__ __forceinline__
#else
#define FDKV_DIVU_HD inline
#endif

namespace fdkv {

struct DivU {
  uint32_t mul, shift;
  void set(uint32_t d) {
    uint32_t s = 0;
    while ((1ull << s) < d) ++s;
    shift = 31 + s;
    mul = (uint32_t)(((1ull << shift) + d - 1) / d);
  }
  FDKV_DIVU_HD uint32_t div(uint32_t n) const { return (uint32_t)(((uint64_t)n * mul) >> shift); }
};

}  // namespace fdkv
