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

// Which work item a workgroup has, as xcd_balanced (gfx950.hpp) says, but as (unit, item of the unit) and with every division prepared: a
// division by a number that only the launch knows is some forty dependent instructions, and a kernel's first load is behind them.
struct XcdMap {
  int32_t per_unit, window, units, len, shared;      // items of a unit; units met together; units and items of a group of XCDs; XCDs of a group (a power of two)
  Divider by_window, by_full, by_rest;               // by the items of a window; by the units of a full one and of the last one
};

inline XcdMap make_xcd_map(int32_t n_units, int32_t per_unit, int32_t window) {
  XcdMap m{};
  const int32_t g = n_units & -n_units;
  m.shared = g >= 8 ? 1 : 8 / g;
  m.per_unit = per_unit;
  m.units = n_units / (8 / m.shared);
  m.len = m.units * per_unit;
  m.window = window < m.units ? window : m.units;
  m.by_window = make_divider(static_cast<uint32_t>(m.window) * per_unit);
  m.by_full = make_divider(static_cast<uint32_t>(m.window));
  m.by_rest = make_divider(static_cast<uint32_t>(m.units % m.window != 0 ? m.units % m.window : 1));
  return m;
}

// false: no item for this workgroup.
__host__ __device__ inline bool xcd_item(const XcdMap& m, int block, int& unit, int& item) {
  const int xcd = block & 7, j = (block >> 3) * m.shared + (xcd & (m.shared - 1));
  if (j >= m.len) return false;
  const int w0 = static_cast<int>(divide(j, m.by_window)) * m.window, left = m.units - w0, wn = left < m.window ? left : m.window, jj = j - w0 * m.per_unit;
  item = static_cast<int>(divide(jj, wn == m.window ? m.by_full : m.by_rest));
  int group = xcd;
  for (int k = m.shared; k > 1; k >>= 1) group >>= 1;
  unit = group * m.units + w0 + jj - item * wn;
  return true;
}

}  // namespace tasp
