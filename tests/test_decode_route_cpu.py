"""CPU: which decode steps run as one workgroup per unit.  The rule is compiled
from the library's own header by the host compiler."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "dmc_internal.h"
int main() {
  int es, d, group, vt, split;
  long long units, slots;
  while (std::scanf("%d %d %d %d %lld %lld %d", &es, &d, &group, &vt, &units, &slots, &split) == 7)
    std::printf("%d\n", int(dmc::decode_one_launch(es, d, group, vt != 0, units, slots, split)));
}
"""

# elem bytes, d, group, matrix cores, units, slots at capacity, split_tile -> one launch
CASES = [
    ((2, 128, 8, 1, 64, 1024, 0), 1), ((2, 128, 8, 1, 64, 1025, 0), 0), ((2, 128, 4, 1, 63, 1024, 0), 0),
    ((2, 64, 4, 1, 256, 2048, 0), 1), ((2, 128, 4, 1, 257, 100, 0), 0), ((2, 128, 8, 1, 8, 512, 0), 1),
    ((2, 128, 8, 1, 64, 1 << 24, 0), 0), ((2, 128, 8, 1, 64, 100, 1), 0),
    # groups of 4 and 8 without transposed value pages (vector ALUs)
    ((2, 128, 4, 0, 64, 256, 0), 1), ((2, 128, 4, 0, 64, 257, 0), 0), ((2, 64, 4, 0, 128, 257, 0), 0),
    ((2, 128, 4, 0, 192, 512, 0), 1), ((2, 64, 4, 0, 192, 513, 0), 0), ((2, 128, 4, 0, 256, 1024, 0), 1),
    ((2, 64, 4, 0, 256, 1025, 0), 0), ((2, 128, 8, 0, 64, 513, 0), 0), ((2, 128, 8, 0, 64, 512, 0), 1),
    ((2, 64, 8, 0, 64, 768, 0), 1), ((2, 64, 8, 0, 64, 769, 0), 0), ((2, 128, 8, 0, 128, 1024, 0), 1),
    ((2, 64, 8, 0, 256, 2049, 0), 0),
    # one and two heads, fp32
    ((2, 128, 1, 0, 64, 512, 0), 1), ((2, 128, 2, 0, 64, 513, 0), 0), ((2, 64, 1, 0, 1, 1024, 0), 1),
    ((4, 128, 8, 0, 128, 256, 0), 1), ((4, 128, 8, 0, 128, 257, 0), 0), ((4, 128, 4, 0, 8, 256, 0), 1),
    ((4, 64, 4, 0, 64, 512, 0), 1), ((4, 64, 1, 0, 4, 513, 0), 0),
]


def test_one_launch_rule(tmp_path):
    cxx = shutil.which("g++")
    hip = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    if cxx is None or not os.path.isdir(hip):
        pytest.skip("no host compiler")
    (tmp_path / "rule.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", hip, "-I",
                    os.path.join(ROOT, "paper_2403_09636_amd", "csrc"), "-o", str(tmp_path / "rule"),
                    str(tmp_path / "rule.cpp")], check=True)
    res = subprocess.run([str(tmp_path / "rule")], input="\n".join(" ".join(map(str, c)) for c, _ in CASES),
                         capture_output=True, text=True, check=True)
    assert [int(x) for x in res.stdout.split()] == [w for _, w in CASES]
