"""Host tests of the rules of the pivoted LU's panels (csrc/panel.hpp), compiled
with g++: the indexes a panel's moves may name, whatever its workgroups chose."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1612_01855_amd", "csrc")


def run_program(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include <vector>\n'
                   '#include "panel.hpp"\nusing namespace trsm;\n' + body)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout


# One panel as piv_panel_kernel keeps it: every workgroup's rows with their
# positions, each step's position chosen by each workgroup for itself.
PANEL = r"""
static unsigned long long seed = 12345;
static int rnd(int n) {
  seed = seed * 6364136223846793005ull + 1442695040888963407ull;
  return (int)((seed >> 33) % (unsigned long long)n);
}
int main() {
  const int kRows = 8;
  int stale = 0, lost = 0;
  for (int t = 0; t < 4000; ++t) {
    const int w = 1 + rnd(kPw), h = w + rnd(60);
    const int groups = (h + kRows - 1) / kRows;
    std::vector<int> pos(h);
    std::vector<char> act(h, 1);
    for (int r = 0; r < h; ++r) pos[r] = r;
    // what an earlier, taller panel left, or uninitialised memory
    Moves mv;
    for (int i = 0; i < kPw; ++i) {
      const int kind = rnd(3);
      mv.src[i] = mv.dst[i] = kind == 0 ? h + rnd(32) : kind == 1 ? -1 - rnd(1 << 30) : 0x7FFFFFFF;
    }
    for (int j = 0; j < w; ++j) {
      const int common = j + rnd(h - j);
      for (int g = 0; g < groups; ++g) {
        // agreeing, or torn candidates: any position, also outside the panel
        const int kind = DISAGREE ? rnd(4) : 0;
        const int raw = kind == 0 ? common : kind == 1 ? rnd(h) : kind == 2 ? (1 << 20) - 1 : rnd(1 << 20);
        const int p = pivot_position(raw, j, h);
        if (p < j || p >= h) return 1;
        for (int r = g * kRows; r < h && r < (g + 1) * kRows; ++r) {
          if (act[r] && pos[r] == p) {
            act[r] = 0;
            pos[r] = j;
            mv.src[j] = r;
            if (r < w) mv.dst[r] = j;
          }
          if (act[r] && pos[r] == j) pos[r] = p;
        }
      }
    }
    for (int r = 0; r < h; ++r) {
      if (pos[r] < 0 || pos[r] >= h) return 2;
      if (act[r] && r < w) mv.dst[r] = pos[r];
    }
    for (int i = 0; i < w; ++i) {
      if (mv.src[i] < 0 || mv.src[i] >= h) ++stale;
      const int s = moved_row(mv.src[i], i, h), d = moved_row(mv.dst[i], i, h);
      if (s < 0 || s >= h || d < 0 || d >= h) return 3;
      if (!DISAGREE && (s != mv.src[i] || d != mv.dst[i])) ++lost;
    }
  }
  printf("%d %d\n", stale, lost);
}
"""


@pytest.mark.parametrize("disagree", [False, True])
def test_moves_stay_inside_the_panel(tmp_path, disagree):
    stale, lost = map(int, run_program(tmp_path, f"#define DISAGREE {int(disagree)}\n" + PANEL)
                      .split())
    # agreeing workgroups name every row themselves; disagreeing ones leave some
    # unwritten, which is what the rule is for
    assert lost == 0
    assert (stale > 0) == disagree


def test_waiting_panels_find_their_places(tmp_path):
    # kPanelsAtOnce ordinary panels and the largest cooperative one (two rows per
    # thread: the room of two) fit the device at once, whatever its size; the
    # largest device keeps panels of 4096 rows out of the cooperative launch
    out = run_program(tmp_path, r"""
int main() {
  for (int places = 0; places <= 4096; ++places) {
    const int g = plain_groups(places);
    if (g < 0 || g > kMaxPlainGroups) return 1;
    if (g > 0 && kPanelsAtOnce * g + 2 * kMaxGroups > places) return 2;
  }
  printf("%d %d %d %d\n", plain_groups(512) * kPanelThreads, plain_groups(256) * kPanelThreads,
         plain_groups(64), plain_groups(0));
}
""")
    assert out.split() == ["4096", "2048", "0", "0"]
