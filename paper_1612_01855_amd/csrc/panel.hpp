// Rules of the pivoted LU's panels (lupiv.hip) that need no device: which rows a
// panel's moves may name, and how many workgroups may wait for each other in an
// ordinary launch.
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

constexpr int kPanelThreads = 512;    // threads per panel workgroup
constexpr int kMaxRpt = 2;            // panel rows per thread: 1 or 2
constexpr int kMaxPanelRows = 65536;  // positions fit a slot's tags
constexpr int kMaxGroups = kMaxPanelRows / (kPanelThreads * kMaxRpt);   // workgroups of a panel

// The most workgroups of one row per thread that a panel may have in an ordinary
// launch, on a device (or partition) with room for `places` of them at once.  They
// wait for each other, so all of them have to find a place although others wait too:
// kPanelsAtOnce panels of this size (one for each of a process's hardware queues,
// 4 by default, times eight) and one cooperative launch of kMaxGroups workgroups, two
// rows per thread, each taking the room of two.  All 256 compute units have 512 places:
// 8 workgroups, 4096 rows, 256 + 128 places at the most; 32 compute units have 64, and
// every panel of several workgroups is launched cooperatively.
constexpr int kPanelsAtOnce = 32;
constexpr int kMaxPlainGroups = 8;    // one candidate to wait for per wave
constexpr int plain_groups(int places) {
  const int g = (places - 2 * kMaxGroups) / kPanelsAtOnce;
  return g < 0 ? 0 : g > kMaxPlainGroups ? kMaxPlainGroups : g;
}

}  // namespace trsm
