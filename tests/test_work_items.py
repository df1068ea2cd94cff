"""Which work item a workgroup has (XcdMap in csrc/divider.hpp), compiled for the host: over the grid that is launched every item of every
unit comes exactly once, each group of XCDs keeps to its own units, and inside a window the items come by their number.  CPU only."""
import os
import shutil
import subprocess

import pytest

from tests import asm_checks

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")

PROGRAM = r"""
#include "gfx950.hpp"
#include "divider.hpp"
#include <cstdio>
#include <vector>
int main() {
  for (int units : {1, 2, 3, 4, 5, 6, 8, 12, 20, 24, 31, 64, 65, 160, 2560})
    for (int per_unit : {1, 2, 3, 7, 24, 32, 33, 97, 1000})
      for (int window : {1, 2, 5, 32, 96}) {
        if (static_cast<long long>(units) * per_unit > 300000) continue;
        const tasp::XcdMap m = tasp::make_xcd_map(units, per_unit, window);
        const int g = (units & -units) >= 8 ? 8 : units & -units;      // groups of XCDs
        std::vector<char> seen(static_cast<size_t>(units) * per_unit);
        std::vector<int> unit_group(units, -1), last_window(8, -1), last_item(8, -1);
        long long n = 0;
        const long long blocks = tasp::xcd_balanced_blocks(units, per_unit);
        for (long long b = 0; b < blocks; ++b) {
          int u = -1, i = -1;
          if (!tasp::xcd_item(m, static_cast<int>(b), u, i)) continue;
          if (u < 0 || u >= units || i < 0 || i >= per_unit || seen[static_cast<size_t>(u) * per_unit + i]++) return 2;
          ++n;
          const int group = static_cast<int>(b & 7) / (8 / g);
          if (unit_group[u] >= 0 && unit_group[u] != group) return 3;
          unit_group[u] = group;
          const int w = (u - group * (units / g)) / m.window;
          if (w < last_window[group] || (w == last_window[group] && i < last_item[group])) return 4;
          last_window[group] = w; last_item[group] = i;
        }
        if (n != static_cast<long long>(units) * per_unit) { std::printf("%d units of %d, window %d: %lld items\n", units, per_unit, window, n); return 5; }
      }
  return 0;
}
"""


def test_every_item_once(tmp_path):
    src, exe = tmp_path / "items.cpp", tmp_path / "items"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I" + asm_checks.CSRC, "-x", "hip", str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stdout)
