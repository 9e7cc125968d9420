"""CPU check of the rule that gives a lane to a team of waves (team_count in
nx_kernels.hpp, compiled here for the host): the waves it counts as having
pixels are those that team_row gives any; one team per CU whatever the step; two
where at most two waves have pixels, and else as far as the model's depth pays
for them beside the timings at the rule; and plans that do not know their step's
rows are taken for full groups.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2201_05213_amd", "csrc")

DRIVER = r"""
#include <cstddef>
#include <cstdio>
#include "nx_kernels.hpp"
#include "nx_window.hpp"
#include "nellox.h"
using namespace nx;
int main() {
  for (int K : {0, 1, 2, 4, 8, 16})
    for (int rows = 0; rows <= 64; ++rows) {
      const int group = rows < 1 || rows > 16 ? 16 : rows;
      int busy = 0;
      for (int w = 0; w < 4; ++w) {
        bool some = false;
        for (int q = 0; q < 4; ++q) some = some || team_row(w, q, K == 8) < group;
        busy += some;
      }
      printf("busy %d %d %d %d\n", K, rows, team_busy(K, rows), busy);
    }
  for (int C : {16, 32, 64})
    for (int nb : {0, 1, 2, 4, 5, 8, 9, 24})
      for (int K : {0, 1, 2, 4, 8, 16})
        for (int rows : {0, 1, 4, 5, 8, 9, 16, 64})
          for (int lanes : {0, 1, 256, 257, 512, 513})
            printf("rule %d %d %d %d %d %d\n", C, nb, K, rows, lanes, team_count(C, nb, K, lanes, rows, 256));
  // the field lies where the structure had padding
  printf("plan %d %d\n", (int)offsetof(nellox_decode_plan, step_rows), (int)offsetof(nellox_decode_plan, n_lanes));
}
"""


def test_team_rule(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
                        os.path.join(ROOT, "include"), "-I", "/opt/rocm/include", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("host build of nx_kernels.hpp failed:\n" + r.stderr[-2000:])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout
    busy = {}
    for line in out.splitlines():
        kind, *v = line.split()
        v = [int(a) for a in v]
        if kind == "busy":
            K, rows, said, counted = v
            assert said == counted, v
            busy[K, rows] = said
        elif kind == "rule":
            C, nb, K, rows, lanes, teams = v
            if lanes in (0, 513) or (C == 16 and nb > 8 and K == 4):
                assert teams == 0, v
            elif lanes <= 256:
                assert teams == 1, v
            else:
                two = K == 2 or busy[K, rows] <= 2 or nb <= {16: 0, 32: 4, 64: 99}[C]
                assert teams == (2 if two else 0), v
        else:
            assert v == [20, 24]
