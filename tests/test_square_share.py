"""Host test of how threads share a square inverted in LDS (csrc/square.hpp),
compiled with g++."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <vector>
#include "square.hpp"
using namespace trsm;
int main() {
  for (int ts = 1; ts <= kInvRows; ts *= 2) {
    std::vector<int> seen(ts * ts);
    for (int t = 0; t < kInvThreads; ++t) {
      const SquareShare s = square_share(t, ts);
      for (int q = 0; q < s.most; ++q) {
        const int line = square_line(s, q, ts);
        // read inside the square, so inside the tiles that LDS holds
        if (line < 0 || line >= ts || s.fast < 0 || s.fast >= ts) return 1;
        if (s.s0 + q * s.ds < ts) ++seen[line * ts + s.fast];
      }
    }
    for (int n : seen)
      if (n != 1) return 2;
    // the largest square's lines are shared evenly, without a check
    if (ts == kInvRows)
      for (int t = 0; t < kInvThreads; ++t) {
        const SquareShare s = square_share(t, ts);
        if (s.most != kInvRows * kInvRows / kInvThreads || s.s0 + (s.most - 1) * s.ds >= ts) return 3;
      }
  }
  return 0;
}
"""


def test_every_element_of_a_square_is_one_threads(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1612_01855_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    assert subprocess.run([str(exe)]).returncode == 0
