// How a workgroup's threads share the square of a diagonal block that it inverts in
// LDS (block_inverse_kernel); needs no device.
#pragma once

namespace trsm {

// Rows of the squares inverted in LDS, and threads of a workgroup: a wave for each
// tile of the largest combine.
constexpr int kInvRows = 128;
constexpr int kInvThreads = 1024;

// The elements of a square of ts rows (a power of two, at most kInvRows) that a thread
// carries: `fast` along the rows in memory, in the lines s0 + q ds below ts, q < most
// (most is the same for all threads; a small square leaves some of them without a line).
struct SquareShare {
  int fast, s0, ds, most;
};
constexpr SquareShare square_share(int tid, int ts) {
  const int lg = 31 - __builtin_clz((unsigned)ts), ds = kInvThreads >> lg;
  return {tid & (ts - 1), tid >> lg, ds, ts > ds ? ts >> (31 - __builtin_clz((unsigned)ds)) : 1};
}

// The line to read for index q: inside the square also where there is none to write.
constexpr int square_line(const SquareShare& s, int q, int ts) {
  return s.s0 + q * s.ds < ts ? s.s0 + q * s.ds : ts - 1;
}

}  // namespace trsm
