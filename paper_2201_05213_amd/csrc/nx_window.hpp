// nx_window.hpp -- the context window of a team of waves (nx_team.hip), shared
// by the host (tests) and the kernels: where a context's inputs lie in it,
// which groups of rows a team decodes one after the other, and what of the
// window it clears, and when.
#pragma once
#include "nx_order.hpp"

namespace nx {

// The sheared window of nx_layout.hpp in LDS: the last 16 wavefront steps
// (columns) of the team's rows, int16 numerators 2x - 255, 0 off the lane,
// planes [column][channel][row] with H_ rows on top. Input k of a pixel at
// step t (window row dy) is plane 3 (t - H_(H_+2)) + k - 3 H_ dy (mod 48),
// row i + dy; every column is held twice, 48 planes apart, so a step's planes
// follow each other without a wrap.
constexpr int WIN_PLANES = 2 * 3 * RING_COLS;

// (column t, channel ch, window row r): its first copy, and how far the second is
NXHD int win_place(int rows, int t, int ch, int r) { return (3 * (t & (RING_COLS - 1)) + ch) * rows + r; }
NXHD int win_copy(int rows) { return 3 * RING_COLS * rows; }

// Value j of lane l is input k = 16 j + l / 4 of its pixel, window row dy
template <int H_>
NXHD void quad_tap(int j, int lane, int& k, int& dy) {
  k = nx_min(16 * j + (lane >> 2), 4 * conv_chunks(H_) - 1);
  dy = nx_min(k / (3 * (2 * H_ + 1)), H_);
}
// input k's place is that of the step and the pixel's row plus that of the tap
template <int H_>
NXHD int win_origin(int rows, int t, int i) {
  return 3 * ((t - H_ * (H_ + 2)) & (RING_COLS - 1)) * rows + i;
}
template <int H_>
NXHD int win_tap(int rows, int j, int lane) {
  int k, dy;
  quad_tap<H_>(j, lane, k, dy);
  return (k - 3 * H_ * dy) * rows + dy;
}

// Pixel q of a wave's four: the row of the group it is. Four in a row, so that
// a group of few rows leaves whole waves free; where rows r and r + 8 share a
// stream (pairs), both are the wave's.
NXHD int team_row(int wave, int q, bool pairs) { return pairs ? 2 * wave + (q & 1) + 8 * (q >> 1) : 4 * wave + q; }

// A team's group: rows ts .. min(ts + 15, last) of wavefront step `step`. A
// step without a pixel (a lane narrower than h + 1 columns has them) is a
// group without rows.
struct TeamGroup {
  int step, ts, last;
};
constexpr TeamGroup TEAM_START = {-1, 0, -1};

NXHD int team_groups_at(int t, int Hl, int Wl, int o) {
  int a, b;
  step_rows(t, Hl, Wl, o, a, b);
  return a <= b ? (b - a) / 16 + 1 : 1;
}

// The next group, which starts with a barrier (sync): the reads and writes of
// the group before are in front of it. A step's column is cleared (clear)
// behind the barrier of its first group: its place in the window is that of 16
// steps before, which for H_ = 3 the step before still reads, and a wave
// without a pixel comes here as soon as that step has begun. The step itself
// does not read its own column, its pixels go to other rows than those cleared,
// and the next step's reads are behind another barrier.
template <int H_, class Sync, class Clear>
NXHD void team_next(TeamGroup& G, int Hl, int Wl, Sync sync, Clear clear) {
  G.ts += 16;
  const bool first = G.ts > G.last;
  if (first) {
    ++G.step;
    step_rows(G.step, Hl, Wl, H_ + 1, G.ts, G.last);
  }
  sync();
  if (first) clear();
}

// The row of the step's column that lane `lane` clears, or -1: the step's rows
// are written as they decode; of the others those that a later read can reach
// (see decode_lane). G is the step's first group.
template <int H_>
NXHD int team_clear_row(const TeamGroup& G, int Hl, int lane) {
  const bool some = G.ts <= G.last;
  const int r = some && lane >= H_ ? G.last + 1 + (lane - H_) : G.ts - H_ + lane;
  const int n = some ? 2 * H_ + 1 : 2 * H_ + 1 + (G.last + 1 - G.ts);
  return lane < n && r >= 0 && r < Hl ? r : -1;
}

}  // namespace nx
