"""The division by the number of query heads of a group that the fp32 backward kernel finds its rows with
(csrc/divider.hpp), compiled for the host: equal to m / g for every kind of m below 2^31.  CPU only."""
import os
import shutil
import subprocess

import pytest

from tests import asm_checks

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")

PROGRAM = r"""
#include "divider.hpp"
#include <cstdio>
int main() {
  long long bad = 0;
  auto check = [&](uint32_t m, uint32_t g, tasp::Divider d) {
    const uint32_t q = tasp::divide(m, d);
    if (q != m / g && bad++ < 5) std::printf("m=%u g=%u: %u, not %u\n", m, g, q, m / g);
  };
  for (uint32_t g = 1; g <= 64; ++g) {
    const tasp::Divider d = tasp::make_divider(g);
    for (uint32_t m = 0; m < 4096; ++m) check(m, g, d);
    for (uint32_t m = 2147483647u; m > 2147483647u - 4096; --m) check(m, g, d);
    for (uint64_t m = 0; m < (1ull << 31); m += 9973) check(static_cast<uint32_t>(m), g, d);
    // both sides of multiples of g, where a quotient that is off by one shows
    for (uint64_t q = 0; q * g < (1ull << 31); q += (1u << 31) / g / 20000 + 1) {
      const uint32_t m = static_cast<uint32_t>(q * g);
      check(m, g, d);
      if (m > 0) check(m - 1, g, d);
    }
  }
  for (uint32_t g : {65u, 127u, 1000u, 65535u, 65536u, 65537u, 16777215u, 1073741823u, 1073741824u}) {
    const tasp::Divider d = tasp::make_divider(g);
    for (uint64_t q = 0; q * g < (1ull << 31); q += (1u << 31) / g / 20000 + 1) {
      const uint32_t m = static_cast<uint32_t>(q * g);
      check(m, g, d);
      if (m > 0) check(m - 1, g, d);
    }
    check(2147483647u, g, d);
  }
  // rows at which an estimate in 32-bit floating point with one correction is wrong
  for (uint32_t g : {1u, 3u, 7u, 12u})
    for (uint32_t m : {33554434u, 33554438u, 58721438u, 134217752u}) check(m, g, tasp::make_divider(g));
  return bad != 0;
}
"""


def test_divider_is_exact_below_2_31(tmp_path):
    src, exe = tmp_path / "divider.cpp", tmp_path / "divider"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-I" + asm_checks.CSRC, "-x", "hip", str(src),
                    "-o", str(exe)], check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout


def test_fp32_backward_rows_are_found_by_it():
    """The kernel forms no such quotient in floating point."""
    with open(os.path.join(asm_checks.CSRC, "attn_bwd_fp32.hip")) as f:
        text = f.read()
    assert "divide(static_cast<uint32_t>(m), group)" in text and "inv_g" not in text
