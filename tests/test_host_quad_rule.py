"""CPU check of the rule that sends a group of few pixels to the network by
fours instead of a tile of 16 (quad_limit in nx_kernels.hpp, compiled here for
the host): for every model size the kernels are built for, the largest group
taken by fours has less matrix work so than as a tile. A tile is a 32-cycle
instruction for 16 outputs by 4 inputs, four pixels an 8-cycle one for 64
outputs by one input; a tenth is left for what the fours do besides.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2201_05213_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "nx_kernels.hpp"
using namespace nx;
int main() {
  const int sizes[][2] = {{3, 64}, {3, 32}, {3, 16}, {2, 64}, {2, 32}, {2, 16}, {1, 32}, {1, 16}};
  for (auto& s : sizes)
    for (int nb = 1; nb <= 4; ++nb) {
      const int C = s[1], mt = C / 16, kc = conv_chunks(s[0]);
      const int tile = 32 * (mt * kc + 2 * nb * mt * mt * 4 + HEAD_TILES * mt * 4);
      const int four = 8 * (4 * kc + 2 * nb * C + 2 * C);
      printf("%d %d %d %d %d %d\n", s[0], C, nb, quad_limit(C), tile, four);
    }
}
"""


def test_fours_have_less_matrix_work_than_a_tile(tmp_path):
    src, exe = tmp_path / "quad.cpp", tmp_path / "quad"
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("host build of nx_kernels.hpp failed:\n" + r.stderr[-2000:])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout
    rows = [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    assert len(rows) == 32
    for h, C, nb, limit, tile, four in rows:
        assert limit % 4 == 0 and limit >= 4, (h, C, nb)
        assert limit // 4 * four <= 0.9 * tile, (h, C, nb, limit)
        # by fours as far as that: the next size up would not hold, but for the 12 pixels' table
        assert limit == 12 or (limit // 4 + 1) * four > 0.9 * tile, (h, C, nb, limit)
