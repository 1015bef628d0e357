"""Order of the resident-rows forward's workgroups (xcd_slot in csrc/grid.hpp).

Workgroup wg runs on XCD wg mod 8.  Its slot must be a permutation of the
grid, whatever the grid's size, that gives each XCD one contiguous range, so
that an XCD serves as few column groups as the grid allows.  Built with hipcc
and run on the host; nothing launches on a GPU.
"""

import subprocess

import pytest

from test_layout import ROOT, _hipcc

SRC = r"""
#include "grid.hpp"
#include <cstdio>
#include <vector>
int main() {
  for (uint32_t n = 1; n <= 320; ++n) {
    std::vector<int> hit(n, 0);
    for (uint32_t x = 0; x < 8; ++x)
      for (uint32_t wg = x; wg < n; wg += 8) {
        const uint32_t t = infcl::xcd_slot(wg, n);
        if (t >= n || hit[t]++) return printf("n %u wg %u: slot %u out of range or taken\n", n, wg, t), 1;
        if (wg >= 8 && t != infcl::xcd_slot(wg - 8, n) + 1) return printf("n %u wg %u: not contiguous\n", n, wg), 1;
      }
  }
  puts("order ok");
}
"""


def test_slots_are_a_permutation_contiguous_per_xcd(tmp_path):
    cc = _hipcc()
    if cc is None:
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "order.hip", str(tmp_path / "order")
    src.write_text(SRC)
    r = subprocess.run([cc, "--offload-arch=gfx950", "-O1", "-std=c++17",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", f"{ROOT}/paper_2410_17243_amd/csrc", str(src), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "order ok" in r.stdout, r.stdout
