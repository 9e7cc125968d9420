"""CPU check of the order in which the waves of a team use their context
window: between two barriers no place of it is written or cleared by one wave
and read or written by another, and every pixel's context holds the pixels of
its lane, 0 outside.

The driver runs the kernel's own group walk and places (nx_window.hpp,
compiled here for the host) for each of a team's waves and sorts their reads,
pixels and clears by the barrier they come after; for h = 1 .. 3, a stream per
row or per two rows of a group (16 and 8 streams), both teams of a workgroup,
and lanes of one row, one column, fewer than h + 1 columns, patches and
thumbnails. (Fewer streams add barriers between a group's reads and its pixels;
they take the same places.)
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2201_05213_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <utility>
#include <vector>
#include "nx_window.hpp"
using namespace nx;

struct Use {                // of one wave between two barriers
  std::vector<int> reads;
  std::vector<std::pair<int, int>> writes;           // place, value
  std::vector<std::pair<int, int>> want;             // place read for a pixel, its value
};

// a pixel's value of channel c: never 0, as 2x - 255
static int value(int i, int j, int c, int Wl) { return 1 + 3 * (i * Wl + j) + c; }

template <int H_>
static int lane(int Hl, int Wl, bool pairs, int team, const char** what) {
  const int o = H_ + 1, T = Wl + o * (Hl - 1), KC = 4 * conv_chunks(H_);
  const int rows = (int)ring_rows_for(Hl, H_);
  int total = 0;
  for (int t = 0; t < T; ++t) total += team_groups_at(t, Hl, Wl, o);
  std::vector<std::vector<Use>> use(total + 1, std::vector<Use>(4));
  for (int w4 = 0; w4 < 4; ++w4) {
    const int v4 = (w4 + 2 * team) & 3;
    int at = 0;  // barriers passed
    TeamGroup G = TEAM_START;
    auto put = [&](int t, int c, int r, int v) {
      const int p = win_place(rows, t, c, r);
      use[at][w4].writes.push_back({p, v});
      use[at][w4].writes.push_back({p + win_copy(rows), v});
    };
    for (int it = 0; it < total; ++it) {
      team_next<H_>(G, Hl, Wl, [&] { ++at; }, [&] {
        for (int l = 0; w4 == 3 && l < 64; ++l) {
          const int r = team_clear_row<H_>(G, Hl, l);
          for (int c = 0; r >= 0 && c < 3; ++c) put(G.step, c, H_ + r, 0);
        }
      });
      const int na = nx_min(16, G.last - G.ts + 1);
      bool some = false;
      for (int q = 0; q < 4; ++q) some = some || team_row(v4, q, pairs) < na;
      if (!some) continue;
      for (int l = 0; l < 64; ++l) {
        const int row = team_row(v4, l & 3, pairs), i = nx_min(G.ts + row, Hl - 1), j = G.step - o * i;
        for (int n = 0; 16 * n < KC; ++n) {
          const int p = win_origin<H_>(rows, G.step, i) + win_tap<H_>(rows, n, l);
          if (p < 0 || p >= WIN_PLANES * rows) { *what = "place"; return 1; }
          use[at][w4].reads.push_back(p);
          int k, dy, ty, tx;
          quad_tap<H_>(n, l, k, dy);
          tap_of(H_, k / 3, ty, tx);
          if (ty != dy) { *what = "tap"; return 1; }
          const int y = i - H_ + ty, x = j - H_ + tx;
          if (row < na)
            use[at][w4].want.push_back({p, y >= 0 && y < Hl && x >= 0 && x < Wl ? value(y, x, k % 3, Wl) : 0});
        }
      }
      for (int q = 0; q < 4; ++q) {
        const int row = team_row(v4, q, pairs), i = G.ts + row;
        for (int c = 0; row < na && c < 3; ++c) put(G.step, c, H_ + i, value(i, G.step - o * i, c, Wl));
      }
    }
    if (G.step != T - 1 || G.ts + 15 < G.last) { *what = "groups"; return 1; }
  }
  std::vector<int> window(WIN_PLANES * rows, 0), writer(WIN_PLANES * rows, -1), mark(WIN_PLANES * rows, -1);
  for (int at = 0; at <= total; ++at) {
    for (int w4 = 0; w4 < 4; ++w4)
      for (auto& u : use[at][w4].writes) {
        if (mark[u.first] == at) { *what = "two writes"; return 1; }
        mark[u.first] = at;
        writer[u.first] = w4;
      }
    for (int w4 = 0; w4 < 4; ++w4)
      for (int p : use[at][w4].reads)
        if (mark[p] == at && writer[p] != w4) { *what = "a read beside another wave's write"; return 1; }
    for (int w4 = 0; w4 < 4; ++w4)
      for (auto& u : use[at][w4].want)
        if (window[u.first] != u.second) { *what = "context"; return 1; }
    for (int w4 = 0; w4 < 4; ++w4)
      for (auto& u : use[at][w4].writes) window[u.first] = u.second;
  }
  return 0;
}

int main() {
  const int shapes[][2] = {{1, 1}, {1, 20}, {20, 1}, {5, 2}, {40, 3}, {3, 70}, {9, 14}, {23, 90},
                           {17, 16}, {32, 32}, {64, 64}, {82, 64}, {64, 37}};
  int cases = 0, bad = 0;
  for (auto& s : shapes)
    for (int h = 1; h <= 3; ++h)
      for (int pairs = 0; pairs < 2; ++pairs)
        for (int team = 0; team < 2; ++team) {
          const char* what = "";
          const int b = h == 1 ? lane<1>(s[0], s[1], pairs, team, &what)
                      : h == 2 ? lane<2>(s[0], s[1], pairs, team, &what) : lane<3>(s[0], s[1], pairs, team, &what);
          if (b) printf("%s: h %d lane %dx%d streams %d team %d\n", what, h, s[0], s[1], pairs ? 8 : 16, team);
          ++cases;
          bad += b;
        }
  printf("%d cases %d bad\n", cases, bad);
  return bad != 0;
}
"""


def test_no_place_is_written_beside_another_waves_read(tmp_path):
    src, exe = tmp_path / "window.cpp", tmp_path / "window"
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("host build of nx_window.hpp failed:\n" + r.stderr[-2000:])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and " 0 bad" in r.stdout, r.stdout[-3000:]
