// Blocked factorizations whose panel steps are the triangular solve of Alg.
// It-Inv-TRSM with whole inverted diagonal blocks: Cholesky A = L L^T (C ABI
// trsm_chol_*) and LU without row exchanges A = L U (trsm_lu_*), both binary64
// (see include/trsm.h).
//
// The abstract and Sec. I name Cholesky as a factorization whose main
// subroutine is TRSM.  Right-looking, block size nb:
//
//   for each diagonal block S_j (nb rows, the last one ragged):
//     factor A(S_j, S_j) = L_jj L_jj^T and form Linv_jj = L_jj^{-1}
//     L(T_j, S_j) = A(T_j, S_j) Linv_jj^T          (the panel solve)
//     A(T_j, T_j) -= L(T_j, S_j) L(T_j, S_j)^T      (lower triangle only)
//
// The panel solve X L_jj^T = A(T_j, S_j) has nb columns of L and n - (j+1) nb
// rows of right-hand sides: the one-large-dimension regime of Sec. VIII,
// where the rule takes n0 equal to the whole triangle (here nb), so it is a
// single product with the inverted block.  The diagonal block is factored
// recursively: halves h and s - h,
//
//   factor D11 -> L11, Linv11;   L21 = D21 Linv11^T;   D22 -= L21 L21^T;
//   factor D22 -> L22, Linv22;   Linv21 = -(Linv22 L21) Linv11,
//
// the last line being Alg. RecTriInv's combine, so the inverse of the block
// is built along the way; leaves of 64 or 128 rows are factored and inverted in LDS.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "../../include/trsm.h"
#include "common.hpp"
#include "diag.hpp"
#include "gemm.hpp"
#include "kernels.hpp"

namespace trsm {

namespace {

constexpr int kLeaf = 64;
constexpr int64_t kDefaultNb = 512;
constexpr int64_t kLargeN = 12288;
constexpr int64_t kMidN = 6144;
constexpr int64_t kMaxNb = 4096;
constexpr size_t kCholSplitBytes = (size_t)32 << 20;
constexpr size_t kAl = 256;
inline size_t al(size_t v) { return (v + kAl - 1) / kAl * kAl; }

inline int64_t pow2_at_least(int64_t v) {
  int64_t p = 1;
  while (p < v) p <<= 1;
  return p;
}

// The elements of a 16 NT-row block that a thread of T carries between global
// memory and LDS: column c of rows r0, r0 + kStep, ...
template <int NT, int T>
struct Carry {
  static constexpr int kRows = 16 * NT, kStep = T / kRows, kEach = kRows / kStep;
  int c, r0;
  __device__ __forceinline__ Carry() {
    int t = threadIdx.x;
    // each use computes its addresses anew: kept from one to the next they would
    // take the registers that the columns need
    asm volatile("" : "+v"(t));
    c = t % kRows;
    r0 = t / kRows;
  }
  // f(row, column, q, offset of the element in a matrix of leading dimension ld)
  template <typename F>
  __device__ __forceinline__ void each(int64_t ld, F f) const {
    const int64_t o = r0 * ld + c, step = kStep * ld;
#pragma unroll
    for (int q = 0; q < kEach; ++q) f(r0 + q * kStep, c, q, o + q * step);
  }
};

// Leaf: the s x s diagonal block D (s <= 16 NT, lower triangle read) is factored
// and inverted in LDS, 16 columns a step: the columns by waves with a row a lane
// (chol_columns; with more than 48 rows below them the diagonal tile's rows are
// worked on by every wave that needs them), the rest of the block by the matrix
// cores, while wave 3 stores and inverts the last step's diagonal tile in place.
// Then the inverse is completed as in Alg. RecTriInv (combine).  Positions past s hold
// the identity.  L goes to D's lower triangle (the strict upper triangle is not
// written), the inverse to V (ld ldv, nothing above the diagonal).  A pivot that is
// not positive (or NaN) records its global row in *bad (the smallest one wins) and is
// replaced by 1 so that the arithmetic goes on.
//
// Bound by the chain of columns.  64 rows take 22.5 us alone (one wave for 64 columns
// one after the other, one for the inverse a step behind: 27.4, 49 beside the trailing
// products); 128 rows 50 us, 55 beside them, where two such leaves and the four
// products between them took 95.
template <int NT>
constexpr int kCholThreads = NT <= 4 ? 256 : 1024;

template <int NT>
__global__ __launch_bounds__(kCholThreads<NT>, 4) void chol_leaf_kernel(
    double* __restrict__ D, int64_t ldd, int s, double* __restrict__ V, int64_t ldv, int64_t row0,
    unsigned long long* bad) {
  using namespace diag;
  using Map = LowerTiles;
  constexpr int T = kCholThreads<NT>, kWaves = T / 64;
  constexpr bool kShared = NT > 4;   // the diagonal tile's rows in several waves
  using C = Carry<NT, T>;
  __shared__ __attribute__((aligned(16))) double S[Map::count(NT) * kTile];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __builtin_amdgcn_s_setprio(3);   // before the trailing products' waves beside it
  const int nt = (s + 15) >> 4;
  auto at = [&](int r, int c) {
    return Map::at(S, r >> 4, min(c >> 4, r >> 4)) + (r & 15) * kTld + (c & 15);
  };
  double v[C::kEach];
  C().each(ldd, [&](int r, int c, int q, int64_t o) { v[q] = D[r < s && c <= r ? o : 0]; });
  int first = C::kRows;
#pragma unroll 1
  for (int p = -1; p <= nt; ++p) {
    // p < 0: the run through the code; p = nt: only the last tile's inversion
    const bool panel = p < nt && (p < 0 || wave == 0 || p + 1 + 3 * wave < nt);
    const int i = lane < 16 ? p : p + 3 * wave + (lane >> 4);   // this lane's tile row
    double* row = Map::at(S, min(max(i, 0), nt - 1), max(p, 0)) + (lane & 15) * kTld;
    double a[16];
    if (panel) row_load(a, row);
    if (kShared) __syncthreads();
    if (panel) {
      int b = 16;
      const bool odd = chol_columns<true>(a, p < 0 ? 1 << (wave & 3) : 15, &b);
      if (odd && p >= 0) {
        row_load(a, row);
        chol_columns<false>(a, 15, &b);
        if (b < 16) first = min(first, 16 * p + b);
      }
    } else if (wave == 3 && p >= 1) {
      double* x = Map::at(S, p - 1, p - 1);
      const int o = 16 * (p - 1), gi = lane & 15, g = lane >> 4;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = 4 * q + g;
        if (gi <= r && o + r < s) D[(o + r) * ldd + o + gi] = x[r * kTld + gi];
      }
      invert_tile(x, false, false);
    }
    if (kShared) __syncthreads();
    if (p < 0) {
      C().each(0, [&](int r, int c, int q, int64_t) {
        if (c >> 4 <= r >> 4) *at(r, c) = r < s && c <= r ? v[q] : r == c ? 1.0 : 0.0;
      });
    } else if (panel && (lane < 16 ? wave == 0 : i < nt)) {
      row_store(a, row);
    }
    __syncthreads();
    if (p < 0) continue;
    int e = wave;
    for (int ti = p + 1; ti < nt; ++ti) {
      for (; e <= ti - p - 1; e += kWaves)
        tile_update<true>(Map::at(S, ti, p + 1 + e), Map::at(S, ti, p), Map::at(S, p + 1 + e, p));
      e -= ti - p;
    }
    __syncthreads();
  }
  if (tid == 0 && first < s) atomicMin(bad, (unsigned long long)(row0 + first));
  C().each(ldd, [&](int r, int c, int, int64_t o) {
    const double x = *at(r, c);
    if (r < s && c >> 4 < r >> 4) D[o] = x;
  });
  __syncthreads();
  combine<Map, NT>(S, nt, false, false);
  C().each(ldv, [&](int r, int c, int, int64_t o) {
    const double x = *at(r, c);
    if (r < s && c <= r) V[o] = x;
  });
}

// Linv blocks: zero everywhere except the identity on the padded diagonal of
// the ragged last block; the status word starts at "no failure".
__global__ void chol_init_kernel(double* __restrict__ V, int64_t n, int64_t nb, int64_t m,
                                 unsigned long long* bad) {
  const int64_t per = nb * nb, total = per * m;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid == 0) *bad = ~0ull;
  for (int64_t idx = tid; idx < total; idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = idx / per, e = idx % per, i = e / nb, j = e % nb;
    V[idx] = (i == j && b * nb + i >= n) ? 1.0 : 0.0;
  }
}

// LU leaf: the s x s (s <= 64) diagonal block D is factored without row exchanges
// and both factors are inverted in LDS, as in chol_leaf_kernel: 16 columns of L and
// the 16 rows of U beside them by wave 0 (lu_columns), the rest of the block by the
// matrix cores, the last step's diagonal tile inverted in place by waves 2 (L) and 3
// (U), and the inverses completed by combine.  Positions past s hold the identity.
// L (strictly lower) and U go back to D, the inverses to VL (unit lower, diagonal
// stored) and VU (upper), ld ldv, nothing written on their other side.  A zero or
// non-finite pivot records its global row in *bad (the smallest one wins) and is
// replaced by 1 in the divisions of L.
//
// Four waves, 37 KB: the size of one workgroup of the trailing products, whose place
// it takes when it runs beside them.  Bound by the chain of columns: 36.5 us alone (four
// waves exchanging 64 columns one after the other through LDS: 35, but 8 % more for the
// factorization of 8192 rows).  Beside the trailing products of 8192 rows it takes 67 us
// on average and up to 130, as their matrix instructions use the same binary64 units;
// more LDS, to keep their workgroups off the compute unit, made it wait longer for its
// place than it gained (15.4 ms then; 96 or 129 KB 16.5).
constexpr int kLuTiles = kLeaf / 16;

__global__ __launch_bounds__(256, 4) void lu_leaf_kernel(double* __restrict__ D, int64_t ldd, int s,
                                                      double* __restrict__ VL,
                                                      double* __restrict__ VU, int64_t ldv,
                                                      int64_t row0, unsigned long long* bad) {
  using namespace diag;
  using Map = AllTiles<kLuTiles>;
  using C = Carry<kLuTiles, 256>;
  __shared__ __attribute__((aligned(16))) double S[Map::count(kLuTiles) * kTile];
  const int tid = threadIdx.x, lane = tid & 63, gi = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __builtin_amdgcn_s_setprio(3);   // before the trailing products' waves beside it
  const int nt = (s + 15) >> 4;
  auto at = [&](int r, int c) { return Map::at(S, r >> 4, c >> 4) + (r & 15) * kTld + (c & 15); };
  // a quarter of the block is on its way during the run through the code, the rest
  // follows: all of it would take the registers that the columns need (28 spilled, and
  // 64 rows 44.2 us instead of 42.5)
  constexpr int kEarly = C::kEach / 4;
  double early[kEarly];
  C().each(ldd, [&](int r, int c, int q, int64_t o) {
    if (q < kEarly) early[q] = D[r < s && c < s ? o : 0];
  });
  int first = C::kRows;
#pragma unroll 1
  for (int p = -1; p <= nt; ++p) {
    // p < 0: the run through the code; p = nt: only the last tile's inversions
    if (p < nt && (p < 0 || wave == 0)) {
      // lanes 0 to 15 the diagonal tile's rows, lane group t the rows of the t-th tile
      // below and the columns of the t-th tile to the right
      const int pp = max(p, 0), other = min(pp + g, nt - 1);
      double* row = Map::at(S, other, pp) + gi * kTld;
      double* col = Map::at(S, pp, other) + gi;
      double a[16], b[16];
      auto load = [&] {
        row_load(a, row);
#pragma unroll
        for (int k = 0; k < 16; ++k) b[k] = col[k * kTld];
      };
      load();
      int f = 16;
      const bool odd = lu_columns<true>(a, b, p < 0 ? 1 << wave : 15, &f);
      if (p >= 0) {
        if (odd) {
          load();
          lu_columns<false>(a, b, 15, &f);
          if (f < 16) first = min(first, 16 * p + f);
        }
        if (p + g < nt) row_store(a, row);
        if (g > 0 && p + g < nt) {
#pragma unroll
          for (int k = 0; k < 16; ++k) col[k * kTld] = b[k];
        }
      }
    } else if (wave >= 2 && p >= 1) {
      double* x = Map::at(S, p - 1, p - 1);
      const int o = 16 * (p - 1);
      const bool upper = wave == 3;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = 4 * q + g;
        if ((upper ? gi >= r : gi < r) && o + r < s && o + gi < s)
          D[(o + r) * ldd + o + gi] = x[r * kTld + gi];
      }
      invert_tile(x, upper, !upper);
    }
    if (p < 0) {
      double v[C::kEach];
      C().each(ldd, [&](int r, int c, int q, int64_t o) {
        if (q >= kEarly) v[q] = D[r < s && c < s ? o : 0];
      });
      C().each(0, [&](int r, int c, int q, int64_t) {
        const double x = q < kEarly ? early[q < kEarly ? q : 0] : v[q];
        *at(r, c) = r < s && c < s ? x : r == c ? 1.0 : 0.0;
      });
    }
    __syncthreads();
    if (p < 0) continue;
    int e = wave;
    for (int ti = p + 1; ti < nt; ++ti) {
      for (; e < nt - p - 1; e += 4)
        tile_update<false>(Map::at(S, ti, p + 1 + e), Map::at(S, ti, p), Map::at(S, p, p + 1 + e));
      e -= nt - p - 1;
    }
    __syncthreads();
  }
  if (tid == 0 && first < s) atomicMin(bad, (unsigned long long)(row0 + first));
  C().each(ldd, [&](int r, int c, int, int64_t o) {
    const double x = *at(r, c);
    if (r < s && c < s && c >> 4 != r >> 4) D[o] = x;
  });
  __syncthreads();
#pragma unroll 1
  for (int u = 0; u < 2; ++u) combine<Map, kLuTiles>(S, nt, u, !u);
  C().each(ldv, [&](int r, int c, int, int64_t o) {
    const double x = *at(r, c);
    if (r < s && c <= r) VL[o] = c == r ? 1.0 : x;
    if (r <= c && c < s) VU[o] = x;
  });
}

struct Ctx {
  double* A;
  int64_t lda, n, nb;
  double* V = nullptr;      // m inverted diagonal blocks, nb x nb each (LU: of L)
  double* VU = nullptr;     // LU: m inverted diagonal blocks of U
  double* W = nullptr;      // nb x nb: the diagonal block's panel and combine
  double* W2[2] = {};       // (n - nb) x nb each: the outer panel L(T_j, S_j), by parity of j
  double* WU[2] = {};       // LU: nb x (n - nb) each: the outer panel U(S_j, T_j)
  void* split;    // split-K scratch
  size_t split_bytes;
  unsigned long long* bad;
  hipStream_t s;
};

// C = alpha * A op(B) (+ C when accumulate); op(B) = B^T stored as N x K rows
// when BT.  Small products take 64 x 64 tiles (small_tile) and split K when
// those are few, if `split`: the products inside a diagonal block are too small
// for the finishing pass to pay off.
GemmParams<double, double, double, float> prod_params(const Ctx& c, const double* A, int64_t lda,
                                                      const double* B, int64_t ldb, double* C,
                                                      int64_t ldc, int64_t M, int64_t N, int64_t K,
                                                      double alpha, bool accumulate,
                                                      uint32_t flags, bool split) {
  auto p = gemm_params<double, double, double, float>();
  p.A = A; p.lda = lda;
  p.B = B; p.ldb = ldb;
  p.Cout = C; p.ldco = ldc;
  if (accumulate) {
    p.Cin = C;
    p.ldci = ldc;
    p.beta = 1.0;
    flags |= G_BETA;
  }
  p.M = (int)M; p.N = (int)N; p.K = (int)K;
  p.alpha = alpha;
  p.flags = flags;
  p.part = split ? c.split : nullptr;
  p.part_bytes = split ? (int64_t)c.split_bytes : 0;
  return p;
}

template <bool BT>
hipError_t prod(const Ctx& c, const double* A, int64_t lda, const double* B, int64_t ldb,
                double* C, int64_t ldc, int64_t M, int64_t N, int64_t K, double alpha,
                bool accumulate, uint32_t flags, bool split = true) {
  const auto p = prod_params(c, A, lda, B, ldb, C, ldc, M, N, K, alpha, accumulate, flags, split);
  return small_tile<double>(p, 1)
             ? launch_gemm<double, double, double, float, 64, 64, 2, 2, BT>(p, 1, c.s)
             : launch_gemm<double, double, double, float, 128, 128, 2, 2, BT>(p, 1, c.s);
}

#define CHOL_HIP(...)                                           \
  do {                                                          \
    hipError_t e_ = (__VA_ARGS__);                              \
    if (e_ != hipSuccess) return (trsm_status)note_hip_error(e_); \
  } while (0)

#define CHOL_TRY(...)                 \
  do {                                \
    trsm_status s_ = (__VA_ARGS__);   \
    if (s_ != TRSM_OK) return s_;     \
  } while (0)

// Factor the s x s diagonal block at global row r0 and write its inverse at V
// (ld nb).
trsm_status factor_diag(const Ctx& c, int64_t r0, int64_t s, double* V) {
  const int64_t lda = c.lda, nb = c.nb;
  double* D = c.A + r0 * lda + r0;
  // 128 rows at once only where they are a whole block: their 83 KB and 16 waves
  // do not find a place beside the trailing products, and a block's first leaf
  // starts before those
  if (s <= kLeaf || (s <= 2 * kLeaf && nb <= 2 * kLeaf)) {
    if (s <= kLeaf)
      chol_leaf_kernel<4><<<1, kCholThreads<4>, 0, c.s>>>(D, lda, (int)s, V, nb, r0, c.bad);
    else
      chol_leaf_kernel<8><<<1, kCholThreads<8>, 0, c.s>>>(D, lda, (int)s, V, nb, r0, c.bad);
    CHOL_HIP(hipGetLastError());
    return TRSM_OK;
  }
  const int64_t h = kLeaf * ((s + 2 * kLeaf - 1) / (2 * kLeaf));
  const int64_t t = s - h;
  double* D21 = D + h * lda;
  double* D22 = D21 + h;
  double* V21 = V + h * nb;
  double* V22 = V21 + h;
  CHOL_TRY(factor_diag(c, r0, h, V));
  // L21 = D21 Linv11^T.  With h <= 64 the product has one column tile, so
  // each workgroup reads its rows of D21 in full before it writes them and
  // the product runs in place; otherwise it goes through W.
  const double* L21 = D21;
  int64_t ld21 = lda;
  if (h <= kLeaf) {
    CHOL_HIP(prod<true>(c, D21, lda, V, nb, D21, lda, t, h, h, 1.0, false, 0u, false));
  } else {
    CHOL_HIP(prod<true>(c, D21, lda, V, nb, c.W, nb, t, h, h, 1.0, false, 0u, false));
    CHOL_HIP(launch_copy2d<double, double>(c.W, nb, D21, lda, t, h, 1.0, c.s));
    L21 = c.W;
    ld21 = nb;
  }
  // D22 -= L21 L21^T, lower triangle
  CHOL_HIP(prod<true>(c, L21, ld21, L21, ld21, D22, lda, t, t, h, -1.0, true, G_C_LOWER, false));
  CHOL_TRY(factor_diag(c, r0 + h, t, V22));
  // Linv21 = -(Linv22 L21) Linv11
  CHOL_HIP(prod<false>(c, V22, nb, D21, lda, c.W, nb, t, h, t, 1.0, false,
                       G_A_LOWER | G_A_ZERO_UPPER, false));
  CHOL_HIP(prod<false>(c, c.W, nb, V, nb, V21, nb, t, h, h, -1.0, false, G_B_LOWER, false));
  return TRSM_OK;
}

// The library's second stream and its events, per device: the lookahead
// runs the bulk of each trailing update there.  Enqueueing is serialised by
// the mutex (the events are reused from one step to the next: a wait takes
// the event's state at the moment it is enqueued).
struct Side {
  std::mutex mu;
  hipStream_t s2 = nullptr;
  hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
};
constexpr int kMaxDevices = 64;
Side g_side[kMaxDevices];

// The device's side stream and events, created on first use (under the
// device's mutex, which the caller then keeps while it enqueues); they live
// until the process ends.
trsm_status side_for(Side** out, std::unique_lock<std::mutex>* lock) {
  int dev = 0;
  CHOL_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return TRSM_EINVAL;
  Side& sd = g_side[dev];
  *lock = std::unique_lock<std::mutex>(sd.mu);
  if (!sd.s2) {
    hipStream_t s2 = nullptr;
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
    CHOL_HIP(hipStreamCreateWithFlags(&s2, hipStreamNonBlocking));
    for (auto& e : ev) CHOL_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    for (int i = 0; i < 3; ++i) sd.ev[i] = ev[i];
    sd.s2 = s2;
  }
  *out = &sd;
  return TRSM_OK;
}

trsm_status init(const Ctx& c, int64_t m) {
  const int64_t total = m * c.nb * c.nb;
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, 4096));
  chol_init_kernel<<<g, 256, 0, c.s>>>(c.V, c.n, c.nb, m, c.bad);
  CHOL_HIP(hipGetLastError());
  return TRSM_OK;
}

// One stream: diagonal block, panel, trailing update, in order.
trsm_status factor_serial(const Ctx& c) {
  const int64_t n = c.n, nb = c.nb, m = (n + nb - 1) / nb, lda = c.lda;
  CHOL_TRY(init(c, m));
  for (int64_t j = 0; j < m; ++j) {
    const int64_t r0 = j * nb, s = std::min(nb, n - r0), t = n - r0 - s;
    double* Vj = c.V + j * nb * nb;
    CHOL_TRY(factor_diag(c, r0, s, Vj));
    if (t <= 0) break;
    double* A21 = c.A + (r0 + s) * lda + r0;
    double* A22 = A21 + s;
    // L(T_j, S_j) = A(T_j, S_j) Linv_jj^T
    CHOL_HIP(prod<true>(c, A21, lda, Vj, nb, c.W2[0], nb, t, s, s, 1.0, false, 0u));
    CHOL_HIP(launch_copy2d<double, double>(c.W2[0], nb, A21, lda, t, s, 1.0, c.s));
    // A(T_j, T_j) -= L(T_j, S_j) L(T_j, S_j)^T, lower triangle
    CHOL_HIP(prod<true>(c, c.W2[0], nb, c.W2[0], nb, A22, lda, t, t, s, -1.0, true, G_C_LOWER));
  }
  return TRSM_OK;
}

// Lookahead over two streams.  Update j, A(T_j, T_j) -= P_j P_j^T, is split
// into the next diagonal block A(S_{j+1}, S_{j+1}) (on the caller's stream,
// the critical chain) and everything below it, A(T_{j+1}, S_{j+1} u T_{j+1})
// (on the side stream).  The side part of update j runs while the chain
// factors diagonal block j+1, whose inputs are complete once the chain's own
// part of update j is done (the side parts of earlier updates, which also
// touched that block, were finished before panel j).  Panel j+1 then waits
// for the side part of update j (event 2), which wrote the rows it reads;
// the side part of update j+1 waits for panel j+1 (event 1).  Panels
// alternate between two buffers, so panel j+1 never overwrites the one the
// side stream may still be reading.
trsm_status factor_lookahead(const Ctx& c, Side& sd) {
  const int64_t n = c.n, nb = c.nb, m = (n + nb - 1) / nb, lda = c.lda;
  hipStream_t s2 = sd.s2;
  Ctx c2 = c;
  c2.s = s2;
  c2.split = nullptr;
  c2.split_bytes = 0;
  CHOL_TRY(init(c, m));
  CHOL_HIP(hipEventRecord(sd.ev[0], c.s));
  CHOL_HIP(hipStreamWaitEvent(s2, sd.ev[0], 0));
  bool pending = false;
  for (int64_t j = 0; j < m; ++j) {
    const int64_t r0 = j * nb, s = std::min(nb, n - r0), t = n - r0 - s;
    double* Vj = c.V + j * nb * nb;
    CHOL_TRY(factor_diag(c, r0, s, Vj));
    if (t <= 0) break;
    double* P = c.W2[j & 1];
    double* A21 = c.A + (r0 + s) * lda + r0;
    double* A22 = A21 + s;
    if (pending) CHOL_HIP(hipStreamWaitEvent(c.s, sd.ev[2], 0));
    CHOL_HIP(prod<true>(c, A21, lda, Vj, nb, P, nb, t, s, s, 1.0, false, 0u));
    const int64_t s1 = std::min(nb, t);
    // the next diagonal block, lower triangle, on the chain
    CHOL_HIP(prod<true>(c, P, nb, P, nb, A22, lda, s1, s1, s, -1.0, true, G_C_LOWER));
    if (t > s1) {
      CHOL_HIP(hipEventRecord(sd.ev[1], c.s));
      CHOL_HIP(hipStreamWaitEvent(s2, sd.ev[1], 0));
      // rows T_{j+1}: block column S_{j+1}, then the lower triangle of T_{j+1}
      CHOL_HIP(prod<true>(c2, P + s1 * nb, nb, P, nb, A22 + s1 * lda, lda, t - s1, s1, s, -1.0,
                          true, 0u));
      CHOL_HIP(prod<true>(c2, P + s1 * nb, nb, P + s1 * nb, nb, A22 + s1 * lda + s1, lda,
                          t - s1, t - s1, s, -1.0, true, G_C_LOWER));
      CHOL_HIP(hipEventRecord(sd.ev[2], s2));
      pending = true;
    } else {
      pending = false;
    }
    // the panel into A, off the chain: nothing reads it there before the end
    CHOL_HIP(launch_copy2d<double, double>(P, nb, A21, lda, t, s, 1.0, t > s1 ? s2 : c.s));
  }
  // join: the caller's stream sees the side stream's work
  CHOL_HIP(hipEventRecord(sd.ev[2], s2));
  CHOL_HIP(hipStreamWaitEvent(c.s, sd.ev[2], 0));
  return TRSM_OK;
}

// ---------------------------------------------------------------------------
// LU without row exchanges.  Diagonal block of s rows at global row r0, its
// inverses at VL / VU (ld nb): halves h and s - h,
//   factor D11 -> L11, U11, Linv11, Uinv11;
//   L21 = D21 Uinv11;  U12 = Linv11 D12;  D22 -= L21 U12;
//   factor D22 -> L22, U22, Linv22, Uinv22;
//   Linv21 = -(Linv22 L21) Linv11;  Uinv12 = -(Uinv11 U12) Uinv22,
// the last two being Alg. RecTriInv's combine for the lower and the upper
// factor.
trsm_status lu_factor_diag(const Ctx& c, int64_t r0, int64_t s, double* VL, double* VU) {
  const int64_t lda = c.lda, nb = c.nb;
  double* D = c.A + r0 * lda + r0;
  if (s <= kLeaf) {
    lu_leaf_kernel<<<1, 256, 0, c.s>>>(D, lda, (int)s, VL, VU, nb, r0, c.bad);
    CHOL_HIP(hipGetLastError());
    return TRSM_OK;
  }
  const int64_t h = kLeaf * ((s + 2 * kLeaf - 1) / (2 * kLeaf));
  const int64_t t = s - h;
  double* D12 = D + h;
  double* D21 = D + h * lda;
  double* D22 = D21 + h;
  CHOL_TRY(lu_factor_diag(c, r0, h, VL, VU));
  // L21 = D21 Uinv11 and U12 = Linv11 D12, in one launch.  With h <= 64 each product
  // has few enough columns (L21) or rows (U12) to run in place (launch_strips);
  // otherwise they go through W (L21 in its first t rows, U12 below).
  double* W1 = c.W + t * nb;
  const double *L21 = D21, *U12 = D12;
  int64_t ld21 = lda, ld12 = lda;
  const uint32_t lower = G_A_LOWER | G_A_ZERO_UPPER;
  if (h <= kLeaf) {
    CHOL_HIP(launch_strips<double>(
        prod_params(c, D21, lda, VU, nb, D21, lda, t, h, h, 1.0, false, 0u, false),
        prod_params(c, VL, nb, D12, lda, D12, lda, h, t, h, 1.0, false, lower, false), c.s));
  } else {
    CHOL_HIP(launch_pair<double>(
        prod_params(c, D21, lda, VU, nb, c.W, nb, t, h, h, 1.0, false, 0u, false),
        prod_params(c, VL, nb, D12, lda, W1, nb, h, t, h, 1.0, false, lower, false), c.s));
    CHOL_HIP(launch_copy2d<double, double>(c.W, nb, D21, lda, t, h, 1.0, c.s));
    CHOL_HIP(launch_copy2d<double, double>(W1, nb, D12, lda, h, t, 1.0, c.s));
    L21 = c.W;
    U12 = W1;
    ld21 = ld12 = nb;
  }
  // D22 -= L21 U12
  CHOL_HIP(prod<false>(c, L21, ld21, U12, ld12, D22, lda, t, t, h, -1.0, true, 0u, false));
  CHOL_TRY(lu_factor_diag(c, r0 + h, t, VL + h * nb + h, VU + h * nb + h));
  // Linv21 = -(Linv22 L21) Linv11 and Uinv12 = -(Uinv11 U12) Uinv22, side by side
  CHOL_HIP(launch_pair<double>(
      prod_params(c, VL + h * nb + h, nb, D21, lda, c.W, nb, t, h, t, 1.0, false, lower, false),
      prod_params(c, VU, nb, D12, lda, W1, nb, h, t, h, 1.0, false, G_A_UPPER, false), c.s));
  CHOL_HIP(launch_pair<double>(
      prod_params(c, c.W, nb, VL, nb, VL + h * nb, nb, t, h, h, -1.0, false, G_B_LOWER, false),
      prod_params(c, W1, nb, VU + h * nb + h, nb, VU + h, nb, h, t, t, -1.0, false, 0u, false),
      c.s));
  return TRSM_OK;
}

trsm_status lu_init(const Ctx& c, int64_t m) {
  CHOL_TRY(init(c, m));
  Ctx cu = c;
  cu.V = c.VU;
  return init(cu, m);
}

// The panels L(T_j, S_j) = A(T_j, S_j) Uinv_jj into PL (ld nb) and U(S_j, T_j) =
// Linv_jj A(S_j, T_j) into PU (ld n - nb): t rows and columns, in one launch.  7168 rows
// and columns, K = 256: 38 us, one after the other 50.
trsm_status lu_panels(const Ctx& c, const double* A21, const double* A12, const double* VL,
                      const double* VU, double* PL, double* PU, int64_t s, int64_t t) {
  const int64_t nb = c.nb, ldu = c.n - nb;
  const auto pl = prod_params(c, A21, c.lda, VU, nb, PL, nb, t, s, s, 1.0, false, 0u, true);
  const auto pu = prod_params(c, VL, nb, A12, c.lda, PU, ldu, s, t, s, 1.0, false,
                              G_A_LOWER | G_A_ZERO_UPPER, true);
  CHOL_HIP(launch_pair<double>(pl, pu, c.s));
  return TRSM_OK;
}

// One stream: diagonal block, both panels, trailing update, in order.
trsm_status lu_factor_serial(const Ctx& c) {
  const int64_t n = c.n, nb = c.nb, m = (n + nb - 1) / nb, lda = c.lda;
  CHOL_TRY(lu_init(c, m));
  for (int64_t j = 0; j < m; ++j) {
    const int64_t r0 = j * nb, s = std::min(nb, n - r0), t = n - r0 - s;
    double* VLj = c.V + j * nb * nb;
    double* VUj = c.VU + j * nb * nb;
    CHOL_TRY(lu_factor_diag(c, r0, s, VLj, VUj));
    if (t <= 0) break;
    double* A12 = c.A + r0 * lda + r0 + s;
    double* A21 = c.A + (r0 + s) * lda + r0;
    double* A22 = A21 + s;
    const int64_t ldu = n - nb;
    // L(T_j, S_j) = A(T_j, S_j) Uinv_jj;  U(S_j, T_j) = Linv_jj A(S_j, T_j)
    CHOL_TRY(lu_panels(c, A21, A12, VLj, VUj, c.W2[0], c.WU[0], s, t));
    CHOL_HIP(launch_copy2d<double, double>(c.W2[0], nb, A21, lda, t, s, 1.0, c.s));
    CHOL_HIP(launch_copy2d<double, double>(c.WU[0], ldu, A12, lda, s, t, 1.0, c.s));
    // A(T_j, T_j) -= L(T_j, S_j) U(S_j, T_j)
    CHOL_HIP(prod<false>(c, c.W2[0], nb, c.WU[0], ldu, A22, lda, t, t, s, -1.0, true, 0u));
  }
  return TRSM_OK;
}

// Lookahead over two streams, as for Cholesky: update j is split into the
// next diagonal block (on the caller's stream) and the rest, the rows below
// it and the columns right of it (on the side stream), which overlaps the
// factorization of diagonal block j+1; panels j+1 wait for it.
trsm_status lu_factor_lookahead(const Ctx& c, Side& sd) {
  const int64_t n = c.n, nb = c.nb, m = (n + nb - 1) / nb, lda = c.lda;
  const int64_t ldu = n - nb;
  hipStream_t s2 = sd.s2;
  Ctx c2 = c;
  c2.s = s2;
  c2.split = nullptr;
  c2.split_bytes = 0;
  CHOL_TRY(lu_init(c, m));
  CHOL_HIP(hipEventRecord(sd.ev[0], c.s));
  CHOL_HIP(hipStreamWaitEvent(s2, sd.ev[0], 0));
  bool pending = false;
  for (int64_t j = 0; j < m; ++j) {
    const int64_t r0 = j * nb, s = std::min(nb, n - r0), t = n - r0 - s;
    double* VLj = c.V + j * nb * nb;
    double* VUj = c.VU + j * nb * nb;
    CHOL_TRY(lu_factor_diag(c, r0, s, VLj, VUj));
    if (t <= 0) break;
    double* PL = c.W2[j & 1];
    double* PU = c.WU[j & 1];
    double* A12 = c.A + r0 * lda + r0 + s;
    double* A21 = c.A + (r0 + s) * lda + r0;
    double* A22 = A21 + s;
    if (pending) CHOL_HIP(hipStreamWaitEvent(c.s, sd.ev[2], 0));
    CHOL_TRY(lu_panels(c, A21, A12, VLj, VUj, PL, PU, s, t));
    const int64_t s1 = std::min(nb, t);
    // the next diagonal block on the chain
    CHOL_HIP(prod<false>(c, PL, nb, PU, ldu, A22, lda, s1, s1, s, -1.0, true, 0u));
    if (t > s1) {
      CHOL_HIP(hipEventRecord(sd.ev[1], c.s));
      CHOL_HIP(hipStreamWaitEvent(s2, sd.ev[1], 0));
      // rows of S_{j+1} right of its diagonal block, then all rows below it
      CHOL_HIP(prod<false>(c2, PL, nb, PU + s1, ldu, A22 + s1, lda, s1, t - s1, s, -1.0, true,
                           0u));
      CHOL_HIP(prod<false>(c2, PL + s1 * nb, nb, PU, ldu, A22 + s1 * lda, lda, t - s1, t, s,
                           -1.0, true, 0u));
      CHOL_HIP(hipEventRecord(sd.ev[2], s2));
      pending = true;
    } else {
      pending = false;
    }
    // the panels into A, off the chain: nothing reads them there before the end
    const hipStream_t sc = t > s1 ? s2 : c.s;
    CHOL_HIP(launch_copy2d<double, double>(PL, nb, A21, lda, t, s, 1.0, sc));
    CHOL_HIP(launch_copy2d<double, double>(PU, ldu, A12, lda, s, t, 1.0, sc));
  }
  CHOL_HIP(hipEventRecord(sd.ev[2], s2));
  CHOL_HIP(hipStreamWaitEvent(c.s, sd.ev[2], 0));
  return TRSM_OK;
}

struct Sizes {
  int64_t nb;
  size_t linv, off_w, off_w2, w2_bytes, off_split, ws;
  size_t off_wu = 0;   // LU only: two nb x (n - nb) panels of U after the split scratch
};

trsm_status sizes_for(int64_t n, int64_t nb, Sizes* z, bool lu = false) {
  if (n < 0 || nb < 0) return TRSM_EINVAL;
  // measured: 128-row blocks are the fastest up to n = 4096, 256-row ones at
  // 8192 and 512-row ones at 16384
  if (nb == 0)
    nb = std::min<int64_t>(
        n >= kLargeN ? kDefaultNb : (n >= kMidN ? kDefaultNb / 2 : kDefaultNb / 4),
        pow2_at_least(std::max<int64_t>(n, kLeaf)));
  if (nb < kLeaf || nb > kMaxNb || (nb & (nb - 1))) return TRSM_EINVAL;
  if (n > (int64_t)1 << 20) return TRSM_EINVAL;
  // no block larger than the matrix rounded up to a power of two (the cap a
  // TRSM plan puts on n0), so that the inverted blocks keep a plan's layout
  nb = std::min<int64_t>(nb, pow2_at_least(std::max<int64_t>(n, kLeaf)));
  const int64_t m = n > 0 ? (n + nb - 1) / nb : 0;
  z->nb = nb;
  // a TRSM_F64 plan's Linv buffer with n0 = nb: the packed inverses, then
  // the 256 bytes of that plan's status word
  z->linv = al((size_t)m * nb * nb * 8) + al(8);
  size_t off = kAl;                                 // status word
  z->off_w = off;
  off += al((size_t)nb * nb * 8);
  z->off_w2 = off;
  z->w2_bytes = al((size_t)std::max<int64_t>(n - nb, 1) * nb * 8);
  off += 2 * al((size_t)std::max<int64_t>(n - nb, 1) * nb * 8);
  z->off_split = off;
  off += kCholSplitBytes;
  if (lu) {
    z->off_wu = off;
    off += 2 * z->w2_bytes;
  }
  z->ws = off;
  return TRSM_OK;
}

}  // namespace
}  // namespace trsm

using namespace trsm;

extern "C" {

trsm_status trsm_chol_sizes(int64_t n, int64_t nb, int64_t* nb_used, size_t* linv_bytes,
                            size_t* workspace_bytes) {
  Sizes z;
  CHOL_TRY(sizes_for(n, nb, &z));
  if (nb_used) *nb_used = z.nb;
  if (linv_bytes) *linv_bytes = z.linv;
  if (workspace_bytes) *workspace_bytes = z.ws;
  return TRSM_OK;
}

trsm_status trsm_chol_factor(int64_t n, double* A, int64_t lda, int64_t nb, double* Linv,
                             void* workspace, void* stream) {
  Sizes z;
  CHOL_TRY(sizes_for(n, nb, &z));
  if (!workspace || (n > 0 && (!A || !Linv)) || lda < std::max<int64_t>(n, 1))
    return TRSM_EINVAL;
  if (((uintptr_t)workspace & (kAl - 1)) || ((uintptr_t)Linv & 15)) return TRSM_EINVAL;
  Ctx c;
  c.A = A;
  c.lda = lda;
  c.n = n;
  c.nb = z.nb;
  c.V = Linv;
  char* w = static_cast<char*>(workspace);
  c.bad = reinterpret_cast<unsigned long long*>(w);
  c.W = reinterpret_cast<double*>(w + z.off_w);
  c.W2[0] = reinterpret_cast<double*>(w + z.off_w2);
  c.W2[1] = reinterpret_cast<double*>(w + z.off_w2 + z.w2_bytes);
  c.split = w + z.off_split;
  c.split_bytes = kCholSplitBytes;
  c.s = static_cast<hipStream_t>(stream);
  if (n == 0) {
    chol_init_kernel<<<1, 64, 0, c.s>>>(nullptr, 0, z.nb, 0, c.bad);
    CHOL_HIP(hipGetLastError());
    return TRSM_OK;
  }
  // the lookahead pays once there are a few blocks to overlap
  if ((n + z.nb - 1) / z.nb <= 2) return factor_serial(c);
  Side* sd = nullptr;
  std::unique_lock<std::mutex> lock;
  CHOL_TRY(side_for(&sd, &lock));
  return factor_lookahead(c, *sd);
}

trsm_status trsm_chol_check(const void* workspace, trsm_status* status, int64_t* index) {
  if (!workspace || !status || !index) return TRSM_EINVAL;
  unsigned long long v = 0;
  CHOL_HIP(hipDeviceSynchronize());
  CHOL_HIP(hipMemcpy(&v, workspace, sizeof(v), hipMemcpyDeviceToHost));
  if (v == ~0ull) {
    *status = TRSM_OK;
    *index = -1;
  } else {
    *status = TRSM_ESINGULAR;
    *index = (int64_t)v;
  }
  return TRSM_OK;
}

trsm_status trsm_lu_sizes(int64_t n, int64_t nb, int64_t* nb_used, size_t* inv_bytes,
                          size_t* workspace_bytes) {
  Sizes z;
  CHOL_TRY(sizes_for(n, nb, &z, true));
  if (nb_used) *nb_used = z.nb;
  if (inv_bytes) *inv_bytes = z.linv;
  if (workspace_bytes) *workspace_bytes = z.ws;
  return TRSM_OK;
}

trsm_status trsm_lu_factor(int64_t n, double* A, int64_t lda, int64_t nb, double* Linv,
                           double* Uinv, void* workspace, void* stream) {
  Sizes z;
  CHOL_TRY(sizes_for(n, nb, &z, true));
  if (!workspace || (n > 0 && (!A || !Linv || !Uinv)) || lda < std::max<int64_t>(n, 1))
    return TRSM_EINVAL;
  if (((uintptr_t)workspace & (kAl - 1)) || ((uintptr_t)Linv & 15) || ((uintptr_t)Uinv & 15))
    return TRSM_EINVAL;
  Ctx c;
  c.A = A;
  c.lda = lda;
  c.n = n;
  c.nb = z.nb;
  c.V = Linv;
  c.VU = Uinv;
  char* w = static_cast<char*>(workspace);
  c.bad = reinterpret_cast<unsigned long long*>(w);
  c.W = reinterpret_cast<double*>(w + z.off_w);
  c.W2[0] = reinterpret_cast<double*>(w + z.off_w2);
  c.W2[1] = reinterpret_cast<double*>(w + z.off_w2 + z.w2_bytes);
  c.WU[0] = reinterpret_cast<double*>(w + z.off_wu);
  c.WU[1] = reinterpret_cast<double*>(w + z.off_wu + z.w2_bytes);
  c.split = w + z.off_split;
  c.split_bytes = kCholSplitBytes;
  c.s = static_cast<hipStream_t>(stream);
  if (n == 0) {
    chol_init_kernel<<<1, 64, 0, c.s>>>(nullptr, 0, z.nb, 0, c.bad);
    CHOL_HIP(hipGetLastError());
    return TRSM_OK;
  }
  if ((n + z.nb - 1) / z.nb <= 2) return lu_factor_serial(c);
  Side* sd = nullptr;
  std::unique_lock<std::mutex> lock;
  CHOL_TRY(side_for(&sd, &lock));
  return lu_factor_lookahead(c, *sd);
}

trsm_status trsm_lu_check(const void* workspace, trsm_status* status, int64_t* index) {
  return trsm_chol_check(workspace, status, index);
}

}  // extern "C"

