// Rules of the pivoted LU's panels (lupiv.hip) that need no device: which rows a
// panel's moves may name.
#pragma once

namespace trsm {

constexpr int kPw = 32;               // panel width

// Where the rows a panel exchanged came from and went to (panel-relative):
// the row at position i < w after the panel was row src[i] before it, and the
// row that was at i is at dst[i] now.
struct Moves {
  int src[kPw];
  int dst[kPw];
};

// The position exchanged with position j of a panel of h rows, p having been chosen
// from the candidates.  A p outside j .. h-1 can only come from candidates read
// after a wait gave up; j then, so that every row goes back to a row of the panel.
constexpr int pivot_position(int p, int j, int h) { return p < j || p >= h ? j : p; }

// A row that the moves name for position i, kept inside the panel.  After a wait gave
// up, workgroups may have chosen different positions for a step; then no row writes
// that step's src, and what is read there is whatever the workspace held.
constexpr int moved_row(int row, int i, int h) { return (unsigned)row < (unsigned)h ? row : i; }

}  // namespace trsm
