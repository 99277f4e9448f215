"""CPU: which wave of a decode launch starts with which slot-space range.  Every
range has one wave, and few ranges keep to workgroups that run at once, at most
one more in any of them than in another.  Compiled from the library's own header
by the host compiler."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "dmc_internal.h"
int main() {
  int nranges, grid, waves, workgroups;
  while (std::scanf("%d %d %d %d", &nranges, &grid, &waves, &workgroups) == 4) {
    for (int b = 0; b < grid; ++b)
      for (int w = 0; w < waves; ++w) std::printf("%d ", dmc::first_range(nranges, grid, waves, workgroups, b, w));
    std::printf("\n");
  }
}
"""
# grid, waves per workgroup, workgroups that run at once
LAUNCHES = [(256, 8, 256), (512, 4, 256), (256, 4, 256), (512, 4, 512), (64, 4, 256), (608, 4, 304), (6, 4, 2)]


def test_first_ranges(tmp_path):
    cxx = shutil.which("g++")
    hip = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    if cxx is None or not os.path.isdir(hip):
        pytest.skip("no host compiler")
    (tmp_path / "ranges.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", hip, "-I",
                    os.path.join(ROOT, "paper_2403_09636_amd", "csrc"), "-o", str(tmp_path / "ranges"),
                    str(tmp_path / "ranges.cpp")], check=True)
    cases = [(n, g, w, m) for g, w, m in LAUNCHES
             for n in (1, 2, 5, 63, 64, 65, 255, 256, 257, 732, 920, 1023, 1024, 1025, 2048, 5000)]
    res = subprocess.run([str(tmp_path / "ranges")], input="\n".join(" ".join(map(str, c)) for c in cases),
                         capture_output=True, text=True, check=True)
    lines = res.stdout.strip().split("\n")
    assert len(lines) == len(cases)
    for (n, grid, waves, most), line in zip(cases, lines):
        first = [int(x) for x in line.split()]
        runs = [r for f in first for r in range(f, n, grid * waves)]   # as the kernel steps through them
        assert sorted(runs) == list(range(n)), (n, grid, waves, most)
        if 2 * n <= grid * waves and n <= min(grid, most) * waves:
            held = [sum(f < n for f in first[b * waves:(b + 1) * waves]) for b in range(grid)]
            assert not any(held[most:]) and max(held) <= min(held[:most]) + 1, (n, grid, waves, most)
