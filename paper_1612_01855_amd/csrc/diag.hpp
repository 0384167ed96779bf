// Operations of one workgroup on a diagonal block held in LDS: the base cases of
// Alg. RecTriInv and of the blocked factorizations.
//
// A block lies in LDS as 16 x 16 tiles (row stride kTld; a lower triangle keeps
// only its lower tiles) that the matrix cores read directly.  All functions are
// called by the whole workgroup unless stated.
//
// What bounds these blocks is the chain of their columns, not their work (a
// 128-row inversion is 0.7 MFLOP, 2.3 us of one compute unit's matrix cores), so
// the chain is kept inside one launch and as few of its steps as possible are
// serial: 64 columns one after the other took 27 us (Cholesky), 34 us (LU) and 40
// us (inversion) per 64-row block, and the products between such blocks 4 to 7 us
// a launch.  Straight-line code that runs once is itself part of that time: an
// instruction line of 64 bytes that is not in the cache costs about 145 cycles, so
// the steps are short loops.
#pragma once

#include "common.hpp"

namespace trsm {
namespace diag {

constexpr int kTld = 18;              // row stride of a tile (rows 16-byte aligned, 36 banks apart)
constexpr int kTile = 16 * kTld;      // elements of a tile

// Tile (i, j) of a block: the lower tiles row by row.
struct LowerTiles {
  static __device__ __forceinline__ double* at(double* S, int i, int j) {
    return S + (i * (i + 1) / 2 + j) * kTile;
  }
  static constexpr int count(int nt) { return nt * (nt + 1) / 2; }
};
__device__ __forceinline__ void tile_store(double* c, const d4& v, double s = 1.0) {
  const int lane = threadIdx.x & 63, gi = lane & 15, g = lane >> 4;
#pragma unroll
  for (int r = 0; r < 4; ++r) c[(4 * r + g) * kTld + gi] = s * v[r];
}

// One wave: the triangle of a diagonal tile becomes its own inverse (UNIT: the
// diagonal is one, whatever is stored there, and stays as it is; the other
// triangle is not touched).  Alg. RecTriInv inside the tile: the four 4 x 4
// diagonal blocks by substitution, one column a lane, then the combine for 4 and
// 8 rows, as products of the whole tile with the blocks that take no part masked
// to zero.
template <bool UPPER, bool UNIT>
__device__ __forceinline__ void invert_tile(double* x) {
  const int lane = threadIdx.x & 63, gi = lane & 15, g = lane >> 4;
  if (lane < 16) {
    // in reversed coordinates an upper block is a lower one
    const int b = lane >> 2, c = lane & 3;
    auto at = [&](int i, int p) {
      return UPPER ? (4 * b + 3 - i) * kTld + 4 * b + 3 - p : (4 * b + i) * kTld + 4 * b + p;
    };
    double v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double t = i == c ? 1.0 : 0.0;
#pragma unroll
      for (int q = 0; q < i; ++q) t = fma(-x[at(i, q)], v[q], t);
      v[i] = UNIT ? t : t / x[at(i, i)];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (UNIT ? i > c : i >= c) x[at(i, c)] = v[i];
  }
#pragma unroll 1
  for (int h = 4; h < 16; h *= 2) {
    // (i, j) in an inverted diagonal block / in the block to be combined
    auto inv = [&](int i, int j, double v) {
      const bool same = (i & -h) == (j & -h);
      if (UNIT && i == j) return 1.0;
      return same && (UPPER ? j >= i : j <= i) ? v : 0.0;
    };
    auto off = [&](int i, int j) {
      return (i & -(2 * h)) == (j & -(2 * h)) && (UPPER ? (j & h) > (i & h) : (i & h) > (j & h));
    };
#pragma unroll 1
    for (int step = 0; step < 2; ++step) {   // the inverse from the left, then from the right
      double va[4], vb[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 4 * q + g;
        const double a = x[gi * kTld + k], b = x[k * kTld + gi];
        const double ai = inv(gi, k, a), ao = off(gi, k) ? -a : 0.0;
        const double bi = inv(k, gi, b), bo = off(k, gi) ? b : 0.0;
        va[q] = step ? ao : ai;
        vb[q] = step ? bi : bo;
      }
      d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 4; ++q) acc = Mfma<double>::mma(va[q], vb[q], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (off(4 * r + g, gi)) x[(4 * r + g) * kTld + gi] = acc[r];
    }
  }
}

// Alg. RecTriInv's combine for all pairs of blocks along the diagonal of an NT-tile
// block (nt of them in use) whose diagonal tiles are already inverted, for Q =
// 1, 2, ... tiles:
//   lower: A21 := -(A22^{-1} A21) A11^{-1},  upper: A12 := -(A11^{-1} A12) A22^{-1},
// both products through registers, so no scratch is needed and the other
// triangle is not touched.  UNIT as above.  One wave a tile: (NT / 2)^2 waves.
// One copy of the code serves all levels: a workgroup runs it once, so the time
// to fetch an instruction counts as much as the time to run it.
template <typename Map, int NT, bool UPPER, bool UNIT>
__device__ __forceinline__ void combine(double* S, int nt) {
  const int lane = threadIdx.x & 63, gi = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll 1
  for (int lq = 0; (1 << lq) < nt; ++lq) {
    const int Q = 1 << lq, o = 2 * Q * (wave >> (2 * lq));
    const int hi = (wave >> lq) & (Q - 1), lo = wave & (Q - 1);
#pragma unroll 1
    for (int step = 0; step < 2; ++step) {   // the inverse from the left, then from the right
      // the coordinate that sets the cost varies over the waves of a SIMD
      const int i = step ? lo : hi, j = step ? hi : lo;
      auto tile = [&](int r, int c) {
        return UPPER ? Map::at(S, o + r, o + Q + c) : Map::at(S, o + Q + r, o + c);
      };
      const bool in = wave < NT * Q / 2 && o + Q + (UPPER ? j : i) < nt;
      d4 acc = {0.0, 0.0, 0.0, 0.0};
      if (in) {
        const int f = (step == 0) != UPPER ? o + Q : o;   // the diagonal block that multiplies
        // its tiles (d, k) or (k, d), and the diagonal one of them, k = d
        const int d = step ? j : i;
        const bool up = UPPER != (step == 1);             // k runs from d up, or from 0 to d
        const int k0 = up ? d : 0;
        int k1 = up ? Q : d + 1;
        if (UPPER == false && step == 0) k1 = min(k1, nt - o - Q);
#pragma unroll 1
        for (int k = k0; k < k1; ++k) {
          const double* a = step ? tile(i, k) : Map::at(S, f + d, f + k);
          const double* b = step ? Map::at(S, f + k, f + d) : tile(k, j);
          double va[4], vb[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            va[q] = a[gi * kTld + 4 * q + g];
            vb[q] = b[(4 * q + g) * kTld + gi];
          }
          if (k == d) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int r = step ? 4 * q + g : gi, c = step ? gi : 4 * q + g;
              double& v = step ? vb[q] : va[q];
              v = UNIT && r == c ? 1.0 : (UPPER ? c >= r : c <= r) ? v : 0.0;
            }
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) acc = Mfma<double>::mma(va[q], vb[q], acc);
        }
      }
      __syncthreads();
      if (in) tile_store(tile(i, j), acc, step ? -1.0 : 1.0);
      __syncthreads();
    }
  }
}

}  // namespace diag
}  // namespace trsm
