// Operations of one workgroup on a diagonal block held in LDS: the base cases of
// Alg. RecTriInv and of the blocked factorizations.
//
// A block lies in LDS as 16 x 16 tiles (row stride kTld; a lower triangle keeps
// only its lower tiles).  A factorization's 16 columns are worked on by waves with a
// row a lane in registers (values of other lanes by readlane), everything else by
// the matrix cores straight from LDS.  All functions are called by the whole
// workgroup unless stated.
//
// What bounds these blocks is the chain of their columns, not their work (a
// 128-row inversion is 0.7 MFLOP, 2.3 us of one compute unit's matrix cores), so
// the chain is kept inside one launch and as few of its steps as possible are
// serial: 64 columns one after the other took 27 us (Cholesky), 34 us (LU) and 40
// us (inversion) per 64-row block, and the products between such blocks 4 to 7 us
// a launch.  Straight-line code that runs once is itself part of that time: an
// instruction line of 64 bytes that is not in the cache costs about 145 cycles, so
// the steps are short loops, or run through once by all waves while the block is
// still on its way from memory (chol_columns).
#pragma once

#include <type_traits>

#include "common.hpp"

namespace trsm {
namespace diag {

constexpr int kTld = 18;              // row stride of a tile (rows 16-byte aligned, 36 banks apart)
constexpr int kTile = 16 * kTld;      // elements of a tile

// Tile (i, j) of a block: the lower tiles row by row, or all NT x NT of them.
struct LowerTiles {
  static __device__ __forceinline__ double* at(double* S, int i, int j) {
    return S + (i * (i + 1) / 2 + j) * kTile;
  }
  static constexpr int count(int nt) { return nt * (nt + 1) / 2; }
};
template <int NT>
struct AllTiles {
  static __device__ __forceinline__ double* at(double* S, int i, int j) {
    return S + (i * NT + j) * kTile;
  }
  static constexpr int count(int) { return NT * NT; }
};

typedef double D2 __attribute__((ext_vector_type(2)));

// Value of lane `lane` (a wave-uniform constant) for every lane.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// The lane's number as a value the compiler cannot see through: addresses and
// masks made from it are computed where they are used, not ahead of a loop, where
// they would take the registers that the columns need.
__device__ __forceinline__ int fresh_lane() {
  int t = threadIdx.x & 63;
  asm volatile("" : "+v"(t));
  return t;
}

// a / d given r = 1 / d to working precision: one correction step, which
// gives the rounded quotient wherever no intermediate leaves the normal range.
__device__ __forceinline__ double quotient(double a, double d, double r) {
  const double q = a * r;
  return fma(fma(-d, q, a), r, q);
}

// One wave: C -= A B for tiles A, B, C; BT: B is given as its transpose.
template <bool BT>
__device__ __forceinline__ void tile_update(double* c, const double* a, const double* b) {
  const int lane = fresh_lane(), gi = lane & 15, g = lane >> 4;
  double va[4], vb[4];
  d4 acc;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = 4 * q + g;
    va[q] = -a[gi * kTld + k];
    vb[q] = BT ? b[gi * kTld + k] : b[k * kTld + gi];
    acc[q] = c[k * kTld + gi];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) acc = Mfma<double>::mma(va[q], vb[q], acc);
#pragma unroll
  for (int r = 0; r < 4; ++r) c[(4 * r + g) * kTld + gi] = acc[r];
}

// A lane's row of a tile.
__device__ __forceinline__ void row_load(double (&a)[16], const double* p) {
#pragma unroll
  for (int i = 0; i < 16; i += 2) {
    const D2 v = *reinterpret_cast<const D2*>(p + i);
    a[i] = v.x;
    a[i + 1] = v.y;
  }
}

__device__ __forceinline__ void row_store(const double (&a)[16], double* p) {
#pragma unroll
  for (int i = 0; i < 16; i += 2) *reinterpret_cast<D2*>(p + i) = D2{a[i], a[i + 1]};
}

// f(std::integral_constant<int, I>()) for I = B, ..., E - 1: register arrays stay in
// registers whatever the unroller decides.
template <int B, int E, typename F>
__device__ __forceinline__ void steps(F f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>());
    steps<B + 1, E>(f);
  }
}

// Pivots for which the reciprocals below stay in the normal range.
__device__ __forceinline__ bool ordinary(double p) { return p > 0x1p-900 && p < 0x1p900; }

// One wave: 16 columns of a Cholesky factorization, row i of the diagonal tile in
// lane i < 16, rows below it in the others, right-looking: l_jj = sqrt(a_jj),
// l_ij = a_ij / l_jj, a_ic -= l_ij l_cj (c > j; entries above the diagonal are
// updated too, nothing reads them).  FAST: roots and quotients from the hardware's
// estimates, refined to working precision; returns whether a pivot was not
// `ordinary`, and the caller then repeats the columns with FAST off, where a pivot
// that is not positive (or NaN) sets `bad` to its first column and counts as 1.
// Four columns for each bit of `mask`: a column is 60 to 130 instructions, run once
// for each 16 columns of a block, and the first time through takes 6 us for the
// cache misses alone; so before the first step the waves run a quarter each on
// whatever their registers hold.
template <bool FAST>
__device__ __forceinline__ bool chol_columns(double (&a)[16], int mask, int* bad) {
  const int lane = threadIdx.x & 63;
  bool odd = false;
  steps<0, 4>([&](auto g) {
    if (!(mask >> g() & 1)) return;
    steps<4 * g(), 4 * g() + 4>([&](auto jc) {
      constexpr int j = jc();
      double piv = lane_value(a[j], j), l;
      if (FAST) {
        odd |= !ordinary(piv);
        double y = __builtin_amdgcn_rsq(piv);
        y = fma(0.5 * y, fma(-(piv * y), y, 1.0), y);
        double d = piv * y;
        d = fma(fma(-d, d, piv), 0.5 * y, d);
        const double r = fma(fma(-d, y, 1.0), y, y);
        l = lane == j ? d : quotient(a[j], d, r);
      } else {
        const bool ok = piv > 0.0;
        if (!ok && *bad > j) *bad = j;
        piv = ok ? piv : 1.0;
        const double d = sqrt(piv);
        l = lane == j ? d : a[j] / d;
      }
      a[j] = l;
      steps<j + 1, 16>([&](auto c) { a[c()] = fma(-l, lane_value(l, c()), a[c()]); });
    });
  });
  return odd;
}

// One wave: 16 columns of an LU factorization without row exchanges, rows in the
// lanes as in chol_columns; b: lane c's column of the rows right of the diagonal
// tile, which takes the same steps (b_i -= l_ij b_j).  l_ij = a_ij / u_jj, a_ic -=
// l_ij u_jc.  FAST and mask as in chol_columns; a zero or non-finite pivot sets
// `bad` and counts as 1.
template <bool FAST>
__device__ __forceinline__ bool lu_columns(double (&a)[16], double (&b)[16], int mask, int* bad) {
  const int lane = threadIdx.x & 63;
  bool odd = false;
  steps<0, 4>([&](auto g) {
    if (!(mask >> g() & 1)) return;
    steps<4 * g(), 4 * g() + 4>([&](auto jc) {
      constexpr int j = jc();
      double piv = lane_value(a[j], j), l;
      if (FAST) {
        odd |= !ordinary(fabs(piv));
        double y = __builtin_amdgcn_rcp(piv);
        y = fma(fma(-piv, y, 1.0), y, y);
        y = fma(fma(-piv, y, 1.0), y, y);
        l = quotient(a[j], piv, y);
      } else {
        const bool ok = piv != 0.0 && isfinite(piv);
        if (!ok && *bad > j) *bad = j;
        l = a[j] / (ok ? piv : 1.0);
      }
      a[j] = lane > j ? l : a[j];
      l = lane > j ? l : 0.0;
      steps<j + 1, 16>([&](auto c) {
        a[c()] = fma(-l, lane_value(a[c()], j), a[c()]);
        b[c()] = fma(-lane_value(l, c()), b[j], b[c()]);
      });
    });
  });
  return odd;
}

__device__ __forceinline__ void tile_store(double* c, const d4& v, double s = 1.0) {
  const int lane = threadIdx.x & 63, gi = lane & 15, g = lane >> 4;
#pragma unroll
  for (int r = 0; r < 4; ++r) c[(4 * r + g) * kTld + gi] = s * v[r];
}

// One wave: the triangle of a diagonal tile becomes its own inverse (unit: the
// diagonal is one, whatever is stored there, and stays as it is; the other
// triangle is not touched).  Alg. RecTriInv inside the tile: the four 4 x 4
// diagonal blocks by substitution, one column a lane, then the combine for 4 and
// 8 rows (in the order of `combine`), as products of the whole tile with the blocks
// that take no part masked to zero.
__device__ __forceinline__ void invert_tile(double* x, bool upper, bool unit) {
  const int lane = fresh_lane(), gi = lane & 15, g = lane >> 4;
  if (lane < 16) {
    // in reversed coordinates an upper block is a lower one
    const int b = lane >> 2, c = lane & 3;
    auto at = [&](int i, int p) {
      return upper ? (4 * b + 3 - i) * kTld + 4 * b + 3 - p : (4 * b + i) * kTld + 4 * b + p;
    };
    double v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double t = i == c ? 1.0 : 0.0;
#pragma unroll
      for (int q = 0; q < i; ++q) t = fma(-x[at(i, q)], v[q], t);
      v[i] = unit ? t : t / x[at(i, i)];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (unit ? i > c : i >= c) x[at(i, c)] = v[i];
  }
#pragma unroll 1
  for (int h = 4; h < 16; h *= 2) {
    // (i, j) in an inverted diagonal block / in the block to be combined
    auto inv = [&](int i, int j, double v) {
      const bool same = (i & -h) == (j & -h);
      if (unit && i == j) return 1.0;
      return same && (upper ? j >= i : j <= i) ? v : 0.0;
    };
    auto off = [&](int i, int j) {
      return (i & -(2 * h)) == (j & -(2 * h)) && (upper ? (j & h) > (i & h) : (i & h) > (j & h));
    };
#pragma unroll 1
    for (int step = 0; step < 2; ++step) {   // the inverse from the right, then from the left
      double va[4], vb[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 4 * q + g;
        const double a = x[gi * kTld + k], b = x[k * kTld + gi];
        const double ai = inv(gi, k, a), ao = off(gi, k) ? -a : 0.0;
        const double bi = inv(k, gi, b), bo = off(k, gi) ? b : 0.0;
        va[q] = step ? ai : ao;
        vb[q] = step ? bo : bi;
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
//   lower: A21 := -A22^{-1} A21 A11^{-1},  upper: A12 := -A11^{-1} A12 A22^{-1},
// both products through registers, so no scratch is needed and the other
// triangle is not touched.  Within 64 rows the product with the inverse on the right
// comes first: its terms are those of a substitution, so that columns of any
// scale stay in range (the other order overflows once two columns differ by more than
// about 2^1023); above, the left one, as in the levels of larger blocks.
// unit as above.  One wave a tile: (NT / 2)^2 waves.
// One copy of the code serves all levels: a workgroup runs it once, so the time
// to fetch an instruction counts as much as the time to run it.
template <typename Map, int NT>
__device__ __forceinline__ void combine(double* S, int nt, bool upper, bool unit) {
  const int lane = threadIdx.x & 63, gi = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll 1
  for (int lq = 0; (1 << lq) < nt; ++lq) {
    const int Q = 1 << lq, o = 2 * Q * (wave >> (2 * lq));
    const int hi = (wave >> lq) & (Q - 1), lo = wave & (Q - 1);
#pragma unroll 1
    for (int step = 0; step < 2; ++step) {
      const bool right = (step == 0) == (lq < 2);   // the inverse from the right
      // the coordinate that sets the cost varies over the waves of a SIMD
      const int i = right ? lo : hi, j = right ? hi : lo;
      auto tile = [&](int r, int c) {
        return upper ? Map::at(S, o + r, o + Q + c) : Map::at(S, o + Q + r, o + c);
      };
      const bool in = wave < NT * Q / 2 && o + Q + (upper ? j : i) < nt;
      d4 acc = {0.0, 0.0, 0.0, 0.0};
      if (in) {
        const int f = right == upper ? o + Q : o;   // the diagonal block that multiplies
        // its tiles (d, k) or (k, d), and the diagonal one of them, k = d
        const int d = right ? j : i;
        const bool up = upper != right;             // k runs from d up, or from 0 to d
        const int k0 = up ? d : 0;
        int k1 = up ? Q : d + 1;
        if (!upper && !right) k1 = min(k1, nt - o - Q);
#pragma unroll 1
        for (int k = k0; k < k1; ++k) {
          const double* a = right ? tile(i, k) : Map::at(S, f + d, f + k);
          const double* b = right ? Map::at(S, f + k, f + d) : tile(k, j);
          double va[4], vb[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            va[q] = a[gi * kTld + 4 * q + g];
            vb[q] = b[(4 * q + g) * kTld + gi];
          }
          if (k == d) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int r = right ? 4 * q + g : gi, c = right ? gi : 4 * q + g;
              double& v = right ? vb[q] : va[q];
              v = unit && r == c ? 1.0 : (upper ? c >= r : c <= r) ? v : 0.0;
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
