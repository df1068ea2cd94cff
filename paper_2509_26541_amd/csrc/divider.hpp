// Division of a non-negative 32-bit integer by a divisor known to the host: a multiplication and a shift.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace tasp {

// m / g = (m mul) >> (31 + shift) with shift = ceil(log2 g) and mul = ceil(2^(31 + shift) / g).  mul exceeds the
// true factor by less than 1 (in units of 2^-(31 + shift)), so the product is too large by less than
// m / 2^(31 + shift) < 1 / g for m < 2^31: exact there for every g in [1, 2^30].  mul fits 32 bits.
struct Divider {
  uint32_t mul, shift;
};

inline Divider make_divider(uint32_t g) {
  uint32_t shift = 0;
  while ((uint64_t{1} << shift) < g) ++shift;
  return Divider{static_cast<uint32_t>(((uint64_t{1} << (31 + shift)) + g - 1) / g), shift};
}

__host__ __device__ inline uint32_t divide(uint32_t m, Divider d) {      // m < 2^31
  return static_cast<uint32_t>(static_cast<uint64_t>(m << 1) * d.mul >> 32) >> d.shift;
}

}  // namespace tasp
