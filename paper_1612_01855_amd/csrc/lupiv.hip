// LU factorization with partial pivoting, P A = L U (binary64), built on the
// triangular solve of Alg. It-Inv-TRSM (C ABI trsm_lu_piv_*, see
// include/trsm.h).  The abstract and Sec. I name LU as a factorization whose
// main subroutine is TRSM; the row exchanges make it apply to every
// nonsingular matrix.
//
// Right-looking with block columns of nb (a power of two), each factored in
// panels of kPw = 32 columns:
//
//   for each block column S_j = [c0, c0 + s):
//     for each panel [c, c + w) of it:
//       factor A(c:n, c:c+w) with row exchanges          (one launch)
//       exchange the same rows in all other columns
//       A(c:c+w, c+w:c0+s) = Lp^{-1} A(c:c+w, c+w:c0+s)  (unit lower, w x w)
//       A(c+w:n, c+w:c0+s) -= A(c+w:n, c:c+w) A(c:c+w, c+w:c0+s)
//     Linv_jj = L_jj^{-1}  (Alg. Diagonal-Inverter + RecTriInv on the unit
//       lower diagonal block, through trsm_invert_diag)
//     U(S_j, T_j) = Linv_jj A(S_j, T_j)         (the panel solve: one product)
//     A(T_j, T_j) -= L(T_j, S_j) U(S_j, T_j)
//
// The panel kernel keeps the panel in registers (kRpt rows per thread, kRows
// rows per workgroup).  A panel of at most kRows rows is one workgroup and
// needs no device-wide meeting; taller ones run on G co-resident workgroups
// (cooperative launch) that meet once per column: every workgroup publishes
// its best candidate (largest magnitude, the first position on ties, positions
// being the row order after the exchanges so far) together with that row's
// values, each picks the winner from the G candidates and eliminates its own
// rows with it.  A published word carries its own step number, so the meeting
// is one store and one load of the candidates (no counter, no fence).  The
// exchanges are kept as positions and applied when the panel is written back;
// the same positions drive one gather pass over the other columns.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/trsm.h"
#include "common.hpp"
#include "gemm.hpp"
#include "kernels.hpp"

namespace trsm {
namespace {

constexpr int kPw = 32;               // panel width
constexpr int kSub = 8;               // columns per unrolled group of steps
constexpr int kThreads = 512;         // threads per panel workgroup
constexpr int kWaves = kThreads / 64;
constexpr int kRpt = 2;               // panel rows per thread
constexpr int kRows = kThreads * kRpt;   // panel rows per workgroup
constexpr int64_t kMaxN = 65536;      // rows a panel may have (positions fit a slot's tags)
constexpr int kMaxGroups = (int)(kMaxN / kRows);   // workgroups of a panel
constexpr int kSlotWords = 2 * kPw;   // 8-byte words of a candidate slot
constexpr int kNoPos = (1 << 30) - 1; // position of "no candidate"
constexpr unsigned kSpinLimit = 1u << 22;
constexpr size_t kAl = 256;
constexpr size_t kSplitBytes = (size_t)32 << 20;
inline size_t al(size_t v) { return (v + kAl - 1) / kAl * kAl; }

// Status words at the start of the workspace.
struct Words {
  unsigned long long bad;   // smallest column with a zero or non-finite pivot
  unsigned unused;
  unsigned err;             // a wait for a candidate gave up
};

// Where the rows a panel exchanged came from and went to (panel-relative):
// the row at position i < w after the panel was row src[i] before it, and the
// row that was at i is at dst[i] now.
struct Moves {
  int src[kPw];
  int dst[kPw];
};

__device__ __forceinline__ bool better(double a, int pa, double b, int pb) {
  // larger magnitude first; on equal magnitudes the smaller position
  return a > b || (a == b && pa < pb);
}

// Rank of a row in the pivot search: its magnitude, NaN below every number.
__device__ __forceinline__ double pivot_key(double x) {
  x = fabs(x);
  return x >= 0.0 ? x : -0.5;
}

template <int CTRL>
__device__ __forceinline__ double dpp_max(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = (int)(unsigned)b, hi = (int)(unsigned)(b >> 32);
  const unsigned l2 = (unsigned)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false);
  const unsigned h2 = (unsigned)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false);
  return fmax(v, __builtin_bit_cast(double, ((unsigned long long)h2 << 32) | l2));
}

// Largest v of the wave (no NaN), in every lane: row shifts by 1, 2, 4, 8,
// then the two row broadcasts; lane 63 holds the maximum.
__device__ __forceinline__ double wave_max(double v) {
  v = dpp_max<0x111>(v);
  v = dpp_max<0x112>(v);
  v = dpp_max<0x114>(v);
  v = dpp_max<0x118>(v);
  v = dpp_max<0x142>(v);
  v = dpp_max<0x143>(v);
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, 63);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 63);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// The best of kWaves candidates (largest value, smallest position on ties):
// its value, position and index, all wave-uniform.
__device__ __forceinline__ void pick(const double* v, const int* p, double& best, int& bp, int& bi) {
  double m = v[0];
#pragma unroll
  for (int i = 1; i < kWaves; ++i) m = fmax(m, v[i]);
  int mp = INT32_MAX, mi = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    const int pi = v[i] == m ? p[i] : INT32_MAX;
    if (pi < mp) {
      mp = pi;
      mi = i;
    }
  }
  best = m;
  bp = __builtin_amdgcn_readfirstlane(mp);
  bi = __builtin_amdgcn_readfirstlane(mi);
}

// Panel A(r0:r0+h, c0:c0+w) (w <= kPw) factored with row exchanges by G =
// gridDim.x co-resident workgroups (MULTI) or by one; workgroup g owns rows
// g*kRows.. of the panel, thread t of it rows t, t + kThreads, ...  ipiv[c0 +
// j] receives the absolute row exchanged with row r0 + j, *mv the panel's net
// row moves.
//
// What bounds it is the chain of w steps, each a search over the whole column
// that needs the previous step's update, so the step is kept short:
//  * search: a wave reduces its column by DPP; its best lane puts its row into
//    LDS, and after the one barrier every wave picks the workgroup's best;
//  * meeting (MULTI): the winner's wave stores the row as 64 words of
//    {32 bits of data, step << 15 | 15 bits of the position}; 8-byte words
//    arrive whole, so a reader that sees the step number in a word has its
//    data, whatever the order of arrival.  Wave v waits for candidates v,
//    v + kWaves, ...; two slots per workgroup, by step parity, suffice: a
//    workgroup publishes step j + 1 only after it has seen everyone's step j,
//    and everyone publishes step j after reading all of step j - 1;
//  * update: the columns right of j by the winner's row from LDS.
// Steps are unrolled in groups of kSub so that registers are indexed
// statically; after a group the columns move down by kSub places (cyclically:
// after kPw / kSub groups they are back), and columns that already hold L are
// left out of the update.
// Measured: 3.5 us per column on two to four workgroups (panels of 1025 to
// 4096 rows, of which about 0.4 us is the panel's load and store), 2.0 us on
// one; 11 to 16 us with one device-wide arrival counter and fences a column
// and 256 rows a workgroup.
template <bool MULTI>
__global__ __launch_bounds__(kThreads) void piv_panel_kernel(
    double* __restrict__ A, int64_t lda, int64_t r0, int64_t c0, int h, int w,
    int64_t* __restrict__ ipiv, unsigned long long* __restrict__ slots, Words* __restrict__ words,
    Moves* __restrict__ mv) {
  typedef double D2 __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(16))) double wrow[2][kWaves][kPw];   // a wave's best row
  __shared__ double wv[2][kWaves];
  __shared__ int wp[2][kWaves];
  __shared__ __attribute__((aligned(16))) double grow[MULTI ? 2 : 1][kWaves][kPw];
  __shared__ double gv[2][kWaves];
  __shared__ int gp[2][kWaves];
  __shared__ int piv[kPw];
  const int G = MULTI ? (int)gridDim.x : 1, g = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double a[kRpt][kPw];
  int pos[kRpt];                          // position in the exchanged order
  bool act[kRpt];
  const bool vec = (lda & 1) == 0 && w == kPw;   // rows 16-byte aligned (c0 is even)
#pragma unroll
  for (int r = 0; r < kRpt; ++r) {
    const int lr = g * kRows + r * kThreads + tid;   // panel row (original order)
    pos[r] = lr;
    act[r] = lr < h;
    const double* src = A + (r0 + (act[r] ? lr : 0)) * lda + c0;
    if (vec) {
#pragma unroll
      for (int c = 0; c < kPw; c += 2) {
        const D2 v = *reinterpret_cast<const D2*>(src + c);
        a[r][c] = v.x;
        a[r][c + 1] = v.y;
      }
    } else {
#pragma unroll
      for (int c = 0; c < kPw; ++c) a[r][c] = c < w ? src[c] : 0.0;
    }
  }
  bool dead = false;                      // a wait gave up: later ones do not wait
  for (int q = 0; q < kPw / kSub; ++q) {
#pragma unroll
    for (int jj = 0; jj < kSub; ++jj) {
      const int j = q * kSub + jj;
      if (j < w) {
        const int par = jj & 1;           // kSub is even: the parity of j
        // the wave's candidate
        double v = -1.0;
        int pv = kNoPos, rv = 0;
#pragma unroll
        for (int r = 0; r < kRpt; ++r) {
          const double key = act[r] ? pivot_key(a[r][jj]) : -1.0;
          if (act[r] && better(key, pos[r], v, pv)) {
            v = key;
            pv = pos[r];
            rv = r;
          }
        }
        const double m = wave_max(v);
        unsigned long long mask = __ballot(v == m);
        if (__popcll(mask) > 1) {         // ties: the smallest position
          int pm = v == m ? pv : kNoPos;
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) pm = min(pm, __shfl_xor(pm, o, 64));
          const unsigned long long first = __ballot(v == m && pv == pm);
          if (first) mask = first;
        }
        if (lane == __ffsll(mask) - 1) {
          wv[par][wave] = v;
          wp[par][wave] = pv;
#pragma unroll
          for (int r = 0; r < kRpt; ++r)
            if (rv == r) {
#pragma unroll
              for (int c = 0; c < kPw; c += 2)
                *reinterpret_cast<D2*>(&wrow[par][wave][c]) = D2{a[r][c], a[r][c + 1]};
            }
        }
        __syncthreads();
        // the workgroup's candidate
        double best;
        int p, sw;
        pick(wv[par], wp[par], best, p, sw);
        const double* u = wrow[par][sw];
        if constexpr (MULTI) {
          const unsigned step = (unsigned)(c0 + j + 1);
          if (wave == sw) {
            const unsigned data = reinterpret_cast<const unsigned*>(&wrow[par][sw][0])[lane];
            const unsigned part = lane == 0 ? (unsigned)p & 0x7FFFu
                                            : lane == 1 ? (unsigned)p >> 15 : 0u;
            const unsigned long long word =
                ((unsigned long long)(step << 15 | part) << 32) | data;
            __hip_atomic_store(&slots[((size_t)par * G + g) * kSlotWords + lane], word,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          double cv = -1.0;
          int cp = kNoPos;
          for (int c = wave; c < G; c += kWaves) {
            const unsigned long long* sl = slots + ((size_t)par * G + c) * kSlotWords + lane;
            unsigned long long word =
                __hip_atomic_load(sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned spins = 0;
            while (!dead && __any((unsigned)(word >> 47) != step)) {
              if (++spins > kSpinLimit) {
                dead = true;
                if (lane == 0) atomicOr(&words->err, 1u);
              }
              word = __hip_atomic_load(sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            const unsigned tag = (unsigned)(word >> 32) & 0x7FFFu, data = (unsigned)word;
            const int pc = __builtin_amdgcn_readlane((int)tag, 0) |
                           __builtin_amdgcn_readlane((int)tag, 1) << 15;
            const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)data, 2 * jj);
            const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)data, 2 * jj + 1);
            const double x = __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
            const double key = pc == kNoPos ? -1.0 : pivot_key(x);
            if (better(key, pc, cv, cp)) {
              cv = key;
              cp = pc;
              reinterpret_cast<unsigned*>(&grow[par][wave][0])[lane] = data;
            }
          }
          if (lane == 0) {
            gv[par][wave] = cv;
            gp[par][wave] = cp;
          }
          __syncthreads();
          pick(gv[par], gp[par], best, p, sw);
          u = grow[par][sw];
        }
        // a position outside j .. h-1 can only come from candidates read after
        // a wait gave up (reported through the error word): fall back to j so
        // that every row still goes back to a row of the panel
        if (p < j || p >= h) {
          p = j;
          if (tid == 0) atomicOr(&words->err, 2u);
        }
        if (tid == 0) piv[j] = p;
        const bool zero = !(best > 0.0) || !(best <= 1.7976931348623157e308);
        if (zero && g == 0 && tid == 0) atomicMin(&words->bad, (unsigned long long)(c0 + j));
        // exchange positions j and p; the pivot row leaves the elimination
#pragma unroll
        for (int r = 0; r < kRpt; ++r) {
          if (act[r] && pos[r] == p) {
            pos[r] = j;
            act[r] = false;
          } else if (act[r] && pos[r] == j) {
            pos[r] = p;
          }
        }
        if (!zero) {
          double uc[kPw];
#pragma unroll
          for (int c = 0; c < kPw; c += 2) {
            const D2 v2 = *reinterpret_cast<const D2*>(u + c);
            uc[c] = v2.x;
            uc[c + 1] = v2.y;
          }
#pragma unroll
          for (int r = 0; r < kRpt; ++r) {
            if (!act[r]) continue;        // rows that left keep their values
            const double l = a[r][jj] / uc[jj];
            a[r][jj] = l;
#pragma unroll
            for (int c = jj + 1; c < kSub; ++c) a[r][c] = fma(-l, uc[c], a[r][c]);
#pragma unroll
            for (int b = 1; b < kPw / kSub; ++b)
              if (q + b < kPw / kSub) {
#pragma unroll
                for (int c = b * kSub; c < (b + 1) * kSub; ++c) a[r][c] = fma(-l, uc[c], a[r][c]);
              }
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kRpt; ++r) {
      double t[kSub];
#pragma unroll
      for (int c = 0; c < kSub; ++c) t[c] = a[r][c];
#pragma unroll
      for (int c = 0; c + kSub < kPw; ++c) a[r][c] = a[r][c + kSub];
#pragma unroll
      for (int c = 0; c < kSub; ++c) a[r][kPw - kSub + c] = t[c];
    }
  }
#pragma unroll
  for (int r = 0; r < kRpt; ++r) {
    const int lr = g * kRows + r * kThreads + tid;
    if (lr >= h) continue;
    double* dst = A + (r0 + pos[r]) * lda + c0;
    if (vec) {
#pragma unroll
      for (int c = 0; c < kPw; c += 2) *reinterpret_cast<D2*>(dst + c) = D2{a[r][c], a[r][c + 1]};
    } else {
#pragma unroll
      for (int c = 0; c < kPw; ++c)
        if (c < w) dst[c] = a[r][c];
    }
    if (pos[r] < w) mv->src[pos[r]] = lr;
    if (lr < w) mv->dst[lr] = pos[r];
  }
  __syncthreads();
  if (g == 0 && tid < w) ipiv[c0 + tid] = r0 + piv[tid];
}

// A panel's row exchanges in the columns outside it, and the panel's U rows in
// the block's remaining columns [c0 + w, e0): one thread per column gathers
// the (at most 2 w) rows the panel moved -- all loads before the first store
// -- and for those columns solves with the panel's unit lower triangle (x_i =
// b_i - sum_{p<i} l_ip x_p, i and p ascending) before it writes them.  One
// pass over at most 2 w rows of the matrix: 19 us at n = 4096; exchanging the
// rows one pair at a time was a chain of w dependent memory round trips (1 to
// 1.5 us each), once for the block's columns and once for all others.
constexpr int kMoveCols = 64;
__global__ __launch_bounds__(kMoveCols) void panel_apply_kernel(double* __restrict__ A,
                                                                int64_t lda, int64_t n,
                                                                int64_t c0, int w, int64_t e0,
                                                                const Moves* __restrict__ mv) {
  __shared__ __attribute__((aligned(16))) double Ls[kPw][kPw];
  const int64_t t = (int64_t)blockIdx.x * kMoveCols + threadIdx.x;
  const int64_t col = t < c0 ? t : t + w;
  const bool live = col < n;
  const bool inside = live && col >= c0 + w && col < e0;
  const bool any = __any(inside);
  if (any) {
    for (int e = threadIdx.x; e < kPw * kPw; e += kMoveCols) {
      const int i = e / kPw, p = e % kPw;
      Ls[i][p] = (i < w && p < i) ? A[(c0 + i) * lda + c0 + p] : 0.0;
    }
  }
  double* __restrict__ P = A + c0 * lda + (live ? col : 0);
  double x[kPw], y[kPw];
#pragma unroll
  for (int i = 0; i < kPw; ++i) x[i] = i < w ? P[(int64_t)mv->src[i] * lda] : 0.0;
#pragma unroll
  for (int i = 0; i < kPw; ++i) y[i] = i < w ? P[(int64_t)i * lda] : 0.0;
  __syncthreads();
  if (inside) {
#pragma unroll
    for (int i = 1; i < kPw; ++i) {
      double acc = x[i];
#pragma unroll
      for (int p = 0; p < i; ++p) acc = fma(-Ls[i][p], x[p], acc);
      x[i] = acc;
    }
  }
  if (!live) return;
#pragma unroll
  for (int i = 0; i < kPw; ++i)
    if (i < w) {
      if (inside || mv->src[i] != i) P[(int64_t)i * lda] = x[i];
      const int d = mv->dst[i];
      if (d >= w) P[(int64_t)d * lda] = y[i];
    }
}

// "Swap rows k and ipiv[k]" for k = k0 .. k1-1, in order, on the first ncols
// columns of B (one thread per column).  The exchanges are taken kPw at a
// time: the rows a group names are lane slots of each wave (slot i: row k + i;
// slot kPw + i: row ipiv[k + i] if it is outside the group and no earlier
// exchange of the group names it), the group's exchanges are done on the slot
// contents, and then every named row is loaded once and stored where its
// contents belong, all loads before the first store.  One memory round trip
// per group instead of one per exchange: 1000 exchanges on 10 columns take
// 0.26 ms.
constexpr int kSwapCols = 256;
__global__ __launch_bounds__(kSwapCols) void swap_rows_kernel(double* __restrict__ B, int64_t ldb,
                                                              const int64_t* __restrict__ ipiv,
                                                              int64_t k0, int64_t k1,
                                                              int64_t ncols) {
  const int64_t col = (int64_t)blockIdx.x * kSwapCols + threadIdx.x;
  const bool live = col < ncols;
  const int lane = threadIdx.x & 63;
  double* __restrict__ P = B + (live ? col : 0);
  for (int64_t k = k0; k < k1; k += kPw) {
    const int w = (int)(k1 - k < kPw ? k1 - k : kPw);
    // target of exchange `lane` (lanes 0 .. w-1), then slot contents: the
    // group's row numbers relative to k, targets as 32-bit offsets
    const int64_t q = lane < w ? ipiv[k + lane] : k;
    const int off = (int)(q - k);
    int owner = kPw + lane;                 // the slot of this exchange's target
    if (off >= 0 && off < w) owner = off;
    for (int i = 0; i < w; ++i) {
      const int oi = __builtin_amdgcn_readlane(off, i);
      if (lane > i && lane < w && oi == off && owner == kPw + lane) owner = kPw + i;
    }
    const int far = __shfl(off, lane - kPw, 64);
    const int fown = __shfl(owner, lane - kPw, 64);
    const bool used = lane < w || (lane >= kPw && lane - kPw < w && fown == lane);
    const int place = lane < kPw ? lane : far;
    int cur = place;                        // the row (relative to k) now in this slot
    for (int i = 0; i < w; ++i) {
      const int t = __builtin_amdgcn_readlane(owner, i);
      const int x = __builtin_amdgcn_readlane(cur, i), y = __builtin_amdgcn_readlane(cur, t);
      cur = lane == i ? y : (lane == t ? x : cur);
    }
    const int from = used ? cur : 0, to = used ? place : 0;
    double v[2 * kPw];
#pragma unroll
    for (int s = 0; s < 2 * kPw; ++s)
      v[s] = P[(k + __builtin_amdgcn_readlane(from, s)) * ldb];
    const bool moved = used && cur != place;
    const unsigned long long mm = __ballot(moved);
#pragma unroll
    for (int s = 0; s < 2 * kPw; ++s)
      if (((mm >> s) & 1) && live) P[(k + __builtin_amdgcn_readlane(to, s)) * ldb] = v[s];
  }
}

// W (nb x nb) = the unit lower triangle of the s x s block D: strictly lower
// part from D, ones on the diagonal, zeros above, identity past s.
__global__ __launch_bounds__(256) void unit_lower_copy_kernel(const double* __restrict__ D,
                                                              int64_t ldd, int64_t s,
                                                              double* __restrict__ W, int64_t nb) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= nb * nb) return;
  const int64_t i = e / nb, c = e % nb;
  W[e] = (c < i) ? ((i < s) ? D[i * ldd + c] : 0.0) : (c == i ? 1.0 : 0.0);
}

#define PIV_HIP(...)                                              \
  do {                                                            \
    hipError_t e_ = (__VA_ARGS__);                                \
    if (e_ != hipSuccess) return (trsm_status)note_hip_error(e_); \
  } while (0)

#define PIV_TRY(...)                 \
  do {                               \
    trsm_status s_ = (__VA_ARGS__);  \
    if (s_ != TRSM_OK) return s_;    \
  } while (0)

struct Layout {
  int64_t nb, m;
  size_t words, slots, w, winv, wu, split, total, inv_bytes, plan_linv;
};

int64_t default_nb(int64_t n) { return n <= 4096 ? 256 : 512; }

inline int64_t pow2_at_least(int64_t v) {
  int64_t p = 1;
  while (p < v) p <<= 1;
  return p;
}

trsm_status layout_for(int64_t n, int64_t nb, Layout* L) {
  if (n <= 0 || n > kMaxN) return TRSM_EINVAL;
  if (nb < 0 || (nb > 0 && (nb < kPw || (nb & (nb - 1))))) return TRSM_EINVAL;
  if (nb == 0) nb = default_nb(n);
  // a solve plan caps its block size at the next power of two >= n
  nb = std::max<int64_t>(kPw, std::min(nb, pow2_at_least(n)));
  L->nb = nb;
  L->m = (n + nb - 1) / nb;
  trsm_plan_t plan = nullptr;
  PIV_TRY(trsm_plan(nb, 1, TRSM_F64, nb, 0, &plan));
  trsm_plan_info pi;
  const trsm_status st = trsm_plan_get_info(plan, &pi);
  trsm_plan_destroy(plan);
  if (st != TRSM_OK) return st;
  L->plan_linv = pi.linv_bytes;
  L->words = al(sizeof(Words));
  L->slots = al((size_t)2 * kMaxGroups * kSlotWords * 8) + al(sizeof(Moves));
  L->w = al((size_t)nb * nb * 8);
  L->winv = al(pi.linv_bytes);
  L->wu = al((size_t)nb * std::max<int64_t>(n - nb, 1) * 8);
  L->split = kSplitBytes;
  L->total = L->words + L->slots + L->w + L->winv + L->wu + L->split;
  L->inv_bytes = (size_t)L->m * nb * nb * 8;
  return TRSM_OK;
}

// C = alpha A B (+ C): binary64 product on the solve path's kernel.
hipError_t prod(const double* A, int64_t lda, const double* B, int64_t ldb, double* C,
                int64_t ldc, int64_t M, int64_t N, int64_t K, double alpha, bool accumulate,
                uint32_t flags, void* split, size_t split_bytes, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
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
  p.part = split;
  p.part_bytes = (int64_t)split_bytes;
  const bool small = gemm_wgs(p.M, p.N, p.K, flags, 128, 128) < kSplitTarget;
  return small ? launch_gemm<double, double, double, float, 64, 64, 2, 2, false>(p, 1, s)
               : launch_gemm<double, double, double, float, 128, 128, 2, 2, false>(p, 1, s);
}

trsm_status factor(int64_t n, double* A, int64_t lda, const Layout& L, int64_t* ipiv,
                   double* Linv, char* ws, hipStream_t s) {
  const int64_t nb = L.nb;
  Words* words = (Words*)ws;
  char* q = ws + L.words;
  unsigned long long* slots = (unsigned long long*)q;
  Moves* mv = (Moves*)(q + al((size_t)2 * kMaxGroups * kSlotWords * 8));
  q += L.slots;
  double* W = (double*)q;      q += L.w;
  double* Winv = (double*)q;   q += L.winv;
  double* WU = (double*)q;     q += L.wu;
  void* split = q;
  // words: bad = all ones, err = 0; no slot carries a step number of this call
  PIV_HIP(launch_fill_u32((unsigned*)words, 2, 0xFFFFFFFFu, s));
  PIV_HIP(launch_fill_u32((unsigned*)words + 2, 2, 0u, s));
  if (n > kRows)
    PIV_HIP(launch_fill_u32((unsigned*)slots, (int64_t)4 * kMaxGroups * kSlotWords, 0u, s));
  trsm_plan_t plan = nullptr;
  PIV_TRY(trsm_plan(nb, 1, TRSM_F64, nb, 0, &plan));
  trsm_status st = TRSM_OK;
  for (int64_t j = 0; j < L.m && st == TRSM_OK; ++j) {
    const int64_t c0 = j * nb, sb = std::min(nb, n - c0), e0 = c0 + sb;
    hipError_t e = hipSuccess;
    for (int64_t c = c0; c < e0 && e == hipSuccess; c += kPw) {
      int w = (int)std::min<int64_t>(kPw, e0 - c);
      int h = (int)(n - c);
      const int G = (h + kRows - 1) / kRows;
      if (G == 1) {
        piv_panel_kernel<false><<<1, kThreads, 0, s>>>(A, lda, c, c, h, w, ipiv, slots, words, mv);
        e = hipGetLastError();
      } else {
        int64_t r0 = c, cc = c;
        void* args[] = {&A, &lda, &r0, &cc, &h, &w, &ipiv, &slots, &words, &mv};
        e = hipLaunchCooperativeKernel(reinterpret_cast<const void*>(piv_panel_kernel<true>),
                                       dim3(G), dim3(kThreads), args, 0, s);
      }
      // the panel's exchanges in all other columns, U of the panel rows in the
      // block's remaining columns, then the block's trailing rows
      if (e == hipSuccess && n > w) {
        panel_apply_kernel<<<(unsigned)ceil_div(n - w, kMoveCols), kMoveCols, 0, s>>>(
            A, lda, n, c, w, e0, mv);
        e = hipGetLastError();
      }
      if (e == hipSuccess && c + w < e0)
        e = prod(A + (c + w) * lda + c, lda, A + c * lda + c + w, lda, A + (c + w) * lda + c + w,
                 lda, n - (c + w), e0 - (c + w), w, -1.0, true, 0u, split, kSplitBytes, s);
    }
    // Linv_jj: the unit lower diagonal block, inverted by Alg.
    // Diagonal-Inverter + RecTriInv (one block of nb rows)
    if (e == hipSuccess) {
      unit_lower_copy_kernel<<<(unsigned)ceil_div(nb * nb, 256), 256, 0, s>>>(
          A + c0 * lda + c0, lda, sb, W, nb);
      e = hipGetLastError();
    }
    if (e != hipSuccess) {
      st = (trsm_status)note_hip_error(e);
      break;
    }
    st = trsm_invert_diag(plan, W, nb, Winv, s);
    if (st != TRSM_OK) break;
    e = launch_copy2d<double, double>(Winv, nb, Linv + j * nb * nb, nb, nb, nb, 1.0, s);
    const int64_t t = n - e0;
    if (e == hipSuccess && t > 0) {
      // U(S_j, T_j) = Linv_jj A(S_j, T_j), then the trailing update
      e = prod(Linv + j * nb * nb, nb, A + c0 * lda + e0, lda, WU, t, sb, t, sb, 1.0, false,
               G_A_LOWER | G_A_ZERO_UPPER, split, kSplitBytes, s);
      if (e == hipSuccess) e = launch_copy2d<double, double>(WU, t, A + c0 * lda + e0, lda, sb, t,
                                                             1.0, s);
      if (e == hipSuccess)
        e = prod(A + e0 * lda + c0, lda, A + c0 * lda + e0, lda, A + e0 * lda + e0, lda, t, t, sb,
                 -1.0, true, 0u, split, kSplitBytes, s);
    }
    if (e != hipSuccess) st = (trsm_status)note_hip_error(e);
  }
  trsm_plan_destroy(plan);
  return st;
}

}  // namespace
}  // namespace trsm

using namespace trsm;

extern "C" {

trsm_status trsm_lu_piv_sizes(int64_t n, int64_t nb, int64_t* nb_used, size_t* inv_bytes,
                              size_t* workspace_bytes) {
  Layout L;
  const trsm_status st = layout_for(n, nb, &L);
  if (st != TRSM_OK) return st;
  if (nb_used) *nb_used = L.nb;
  if (inv_bytes) *inv_bytes = L.inv_bytes;
  if (workspace_bytes) *workspace_bytes = L.total;
  return TRSM_OK;
}

trsm_status trsm_lu_piv_factor(int64_t n, double* A, int64_t lda, int64_t nb, int64_t* ipiv,
                               double* Linv, void* workspace, void* stream) {
  if (!A || !ipiv || !Linv || !workspace || lda < n) return TRSM_EINVAL;
  Layout L;
  const trsm_status st = layout_for(n, nb, &L);
  if (st != TRSM_OK) return st;
  if (((uintptr_t)workspace & 255) || ((uintptr_t)A & 15) || ((uintptr_t)Linv & 15))
    return TRSM_EINVAL;
  return factor(n, A, lda, L, ipiv, Linv, static_cast<char*>(workspace), (hipStream_t)stream);
}

trsm_status trsm_lu_piv_check(const void* workspace, trsm_status* status, int64_t* index) {
  if (!workspace || !status) return TRSM_EINVAL;
  Words w;
  if (hipMemcpy(&w, workspace, sizeof(w), hipMemcpyDeviceToHost) != hipSuccess)
    return (trsm_status)note_hip_error(hipGetLastError());
  if (w.err) {
    *status = TRSM_EHIP;
    if (index) *index = -1;
    return TRSM_OK;
  }
  const bool bad = w.bad != ~0ull;
  *status = bad ? TRSM_ESINGULAR : TRSM_OK;
  if (index) *index = bad ? (int64_t)w.bad : -1;
  return TRSM_OK;
}

trsm_status trsm_row_swaps(int64_t k0, int64_t k1, const int64_t* ipiv, double* B, int64_t ldb,
                           int64_t ncols, void* stream) {
  if (k0 < 0 || k1 < k0 || ncols < 0 || (k1 > k0 && (!ipiv || !B)) || ldb < ncols)
    return TRSM_EINVAL;
  if (k1 == k0 || ncols == 0) return TRSM_OK;
  swap_rows_kernel<<<(unsigned)ceil_div(ncols, kSwapCols), kSwapCols, 0, (hipStream_t)stream>>>(
      B, ldb, ipiv, k0, k1, ncols);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? TRSM_OK : (trsm_status)note_hip_error(e);
}

}  // extern "C"
