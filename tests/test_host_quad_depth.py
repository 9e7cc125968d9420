"""CPU check of how deep a model's groups of few pixels go by fours (quad_limit in
nx_kernels.hpp, compiled here for the host): with 16 channels up to 4 blocks,
with 32 and 64 whatever their number. The lines lie where the timings beside
the rule cross.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2201_05213_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "nx_kernels.hpp"
int main() {
  for (int C : {16, 32, 64})
    for (int nb = 0; nb <= 40; ++nb) printf("%d %d %d\n", C, nb, nx::quad_limit(C, nb));
}
"""


def test_quads_by_depth(tmp_path):
    src, exe = tmp_path / "depth.cpp", tmp_path / "depth"
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("host build of nx_kernels.hpp failed:\n" + r.stderr[-2000:])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout
    for line in out.splitlines():
        C, nb, limit = (int(v) for v in line.split())
        assert limit == {16: 4 if nb <= 4 else 0, 32: 8, 64: 12}[C], (C, nb)
