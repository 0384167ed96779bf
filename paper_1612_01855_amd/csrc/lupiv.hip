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
//       lower diagonal block)
//     U(S_j, T_j) = Linv_jj A(S_j, T_j)         (the panel solve: one product)
//     A(T_j, T_j) -= L(T_j, S_j) U(S_j, T_j)
//
// The panel kernel keeps the panel in registers (one or two rows per thread).
// A panel of at most 1024 rows is one workgroup and needs no device-wide
// meeting; taller ones run on G co-resident workgroups
// (launch_panel) that meet once per column: every workgroup publishes
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
#include <atomic>

#include "../../include/trsm.h"
#include "common.hpp"
#include "gemm.hpp"
#include "kernels.hpp"
#include "panel.hpp"

namespace trsm {
namespace {

constexpr int kSub = 8;               // columns per unrolled group of steps
constexpr int kThreads = kPanelThreads;
constexpr int kWaves = kThreads / 64;
constexpr int64_t kMaxN = kMaxPanelRows;
constexpr int kSlotWords = 2 * kPw;   // 8-byte words of a candidate slot
constexpr int kNoPos = (1 << 20) - 1; // position of "no candidate" (times kWaves fits an int)
// Polls of a wait before it gives up, about a microsecond each (more than ten
// seconds in all); after kSpinBusy of them the wave sleeps between two.
constexpr unsigned kSpinLimit = 1u << 24;
constexpr unsigned kSpinBusy = 1u << 10;
constexpr size_t kAl = 256;
constexpr size_t kSplitBytes = (size_t)32 << 20;
inline size_t al(size_t v) { return (v + kAl - 1) / kAl * kAl; }

// Status words at the start of the workspace.
struct Words {
  unsigned long long bad;   // smallest column with a zero or non-finite pivot
  unsigned err;             // a wait for a candidate gave up
};

// Rank of a row in the pivot search, as an integer so that the largest
// magnitude is the largest rank: 0 for no row, 1 for a NaN, else the bits of
// |x| (which order like the values) plus 2.
__device__ __forceinline__ unsigned long long pivot_rank(double x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x) & ~(1ull << 63);
  return x == x ? b + 2 : 1;
}

// A candidate for the pivot: its rank and position.
struct __attribute__((aligned(16))) Cand {
  unsigned hi, lo;   // the rank
  int pos, unused;
};

// Lane `lane`'s v (a wave-uniform lane), in scalar registers.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

template <int CTRL>
__device__ __forceinline__ unsigned dpp_max(unsigned v) {
  return max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, false));
}

// Largest v over lanes 0 .. LANES-1 (8 or 64), wave-uniform: row shifts by 1,
// 2, 4 (lane 7 then holds lanes 0-7's), 8 and the two row broadcasts.
template <int LANES>
__device__ __forceinline__ unsigned lanes_max(unsigned v) {
  v = dpp_max<0x111>(v);
  v = dpp_max<0x112>(v);
  v = dpp_max<0x114>(v);
  if (LANES == 64) {
    v = dpp_max<0x118>(v);
    v = dpp_max<0x142>(v);
    v = dpp_max<0x143>(v);
  }
  return (unsigned)__builtin_amdgcn_readlane((int)v, LANES - 1);
}

// The lane (of 0 .. LANES-1) with the best candidate: the largest rank, the
// smallest position on ties.  One pass over the high words decides unless
// several lanes share the largest one.
template <int LANES>
__device__ __forceinline__ int best_lane(const Cand& c) {
  const unsigned long long in = LANES == 64 ? ~0ull : (1ull << LANES) - 1;
  const unsigned mh = lanes_max<LANES>(c.hi);
  unsigned long long mask = __ballot(c.hi == mh) & in;
  if (mask & (mask - 1)) {
    const unsigned ml = lanes_max<LANES>(c.hi == mh ? c.lo : 0u);
    const bool top = c.hi == mh && c.lo == ml;
    const unsigned mp = lanes_max<LANES>(top ? ~(unsigned)c.pos : 0u);
    mask = __ballot(top && ~(unsigned)c.pos == mp) & in;
  }
  return __ffsll(mask) - 1;
}

// Panel A(r0:r0+h, c0:c0+w) (w <= kPw) factored with row exchanges by G =
// gridDim.x co-resident workgroups (MULTI) or by one; workgroup g owns
// kThreads RPT rows of the panel, thread t of it rows t, t + kThreads, ...
// ipiv[c0 + j] receives the absolute row exchanged with row r0 + j, *mv the
// panel's net row moves.
//
// What bounds it is the chain of w steps, each a search over the whole column
// that needs the previous step's update, so the step is kept short:
//  * search: a wave reduces its column's ranks by DPP and shows its best; after
//    a barrier every wave picks the workgroup's best from the kWaves shown, and
//    only that row goes through LDS, its columns from j on (a 16-byte LDS write
//    of one lane costs about 16 cycles of the unit's LDS, so eight waves
//    showing whole rows took longer than the second barrier);
//  * meeting (MULTI): the winner's wave stores the row as 64 words of
//    {32 bits of data, step << 15 | 15 bits of the position}; 8-byte words
//    arrive whole, so a reader that sees the step number in a word has its
//    data, whatever the order of arrival.  Wave v waits for candidates v,
//    v + kWaves, ...; two slots per workgroup, by step parity, suffice: a
//    workgroup publishes step j + 1 only after it has seen everyone's step j,
//    and everyone publishes step j after reading all of step j - 1;
//  * update: the columns right of j; every lane reads one element of the pivot
//    row and the rest comes by readlane (LDS broadcasts of the row to eight
//    waves cost more).  Not masked: a pivot row's U part is written back at its
//    step, and its L part, the columns before, is no longer touched.
// Steps are unrolled in groups of kSub so that registers are indexed
// statically (4 and 2 measured the same to 4 % slower); after a group the
// columns move down by kSub places (cyclically: after kPw / kSub groups they
// are back), and columns that already hold L are left out of the update.
// Measured per column: 1.3 us on one workgroup (1.75 with two rows a thread), 2.45 us
// on several (1.3 of it the store and load of the candidates); 11 to 16 us with one
// device-wide arrival counter and fences a column and 256 rows a workgroup.
template <int RPT, bool MULTI>
__global__ __launch_bounds__(kThreads) void piv_panel_kernel(
    double* __restrict__ A, int64_t lda, int64_t r0, int64_t c0, int h, int w,
    int64_t* __restrict__ ipiv, unsigned long long* __restrict__ slots, Words* __restrict__ words,
    Moves* __restrict__ mv) {
  typedef double D2 __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(16))) double row[2][kPw];   // the workgroup's best row
  __shared__ Cand wcand[2][kWaves];
  __shared__ __attribute__((aligned(16))) double grow[MULTI ? 2 : 1][kWaves][kPw];
  __shared__ Cand gcand[2][kWaves];
  __shared__ int piv[kPw];
  const int G = MULTI ? (int)gridDim.x : 1, g = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double a[RPT][kPw];
  int pos[RPT];                           // position in the exchanged order
  bool act[RPT];
  const bool vec = (lda & 1) == 0 && w == kPw;   // rows 16-byte aligned (c0 is even)
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int lr = g * (kThreads * RPT) + r * kThreads + tid;   // panel row (original order)
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
  // every row has arrived before anyone may write the panel back: the empty asm
  // uses the registers, so the loads are waited for here
#pragma unroll
  for (int r = 0; r < RPT; ++r)
#pragma unroll
    for (int c = 0; c < kPw; ++c) asm volatile("" : "+v"(a[r][c]));
  // the next step's candidate: the lane's best row, then the wave's best lane
  Cand mine;
  int rv, wl;
  auto search = [&](const double (&x)[RPT]) {
    unsigned long long k = act[0] ? pivot_rank(x[0]) : 0;
    int pk = act[0] ? pos[0] : kNoPos;
    rv = 0;
#pragma unroll
    for (int r = 1; r < RPT; ++r) {
      const unsigned long long kr = act[r] ? pivot_rank(x[r]) : 0;
      const int pr = act[r] ? pos[r] : kNoPos;
      const bool better = kr > k || (kr == k && pr < pk);
      k = better ? kr : k;
      pk = better ? pr : pk;
      rv = better ? r : rv;
    }
    mine.hi = (unsigned)(k >> 32);
    mine.lo = (unsigned)k;
    mine.pos = pk;
    wl = best_lane<64>(mine);
  };
  {
    double x[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) x[r] = a[r][0];
    search(x);
  }
  // a wait gave up, here or in an earlier panel: later ones do not wait
  bool dead = MULTI && __hip_atomic_load(&words->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int q = 0; q < kPw / kSub; ++q) {
#pragma unroll
    for (int jj = 0; jj < kSub; ++jj) {
      const int j = q * kSub + jj;
      if (j < w) {
        const int par = jj & 1;           // kSub is even: the parity of j
        if (lane == wl) wcand[par][wave] = mine;
        __syncthreads();
        // the workgroup's candidate; its thread shows the row's columns from j
        // on (columns before j, already L, stay in its registers)
        Cand k = wcand[par][lane & (kWaves - 1)];
        int sw = best_lane<kWaves>(k);
        unsigned bhi = (unsigned)__builtin_amdgcn_readlane((int)k.hi, sw);
        unsigned blo = (unsigned)__builtin_amdgcn_readlane((int)k.lo, sw);
        int p = __builtin_amdgcn_readlane(k.pos, sw);
        if (wave == sw && lane == wl) {
#pragma unroll
          for (int r = 0; r < RPT; ++r)
            if (RPT == 1 || rv == r) {
              auto show = [&](int cb, int ce) {
#pragma unroll
                for (int c = cb; c < ce; c += 2)
                  *reinterpret_cast<D2*>(&row[par][c]) = D2{a[r][c], a[r][c + 1]};
              };
              show(jj & ~1, kSub);
#pragma unroll
              for (int b = 1; b < kPw / kSub; ++b)
                if (q + b < kPw / kSub) show(b * kSub, (b + 1) * kSub);
            }
        }
        double u;                         // the pivot row, column `lane` of this group's order
        if constexpr (!MULTI) {
          __syncthreads();
          u = row[par][lane & (kPw - 1)];
        }
        if constexpr (MULTI) {
          const unsigned step = (unsigned)(c0 + j + 1);
          if (wave == sw) {
            const unsigned data = reinterpret_cast<const unsigned*>(&row[par][0])[lane];
            const unsigned part = lane == 0 ? (unsigned)p & 0x7FFFu
                                            : lane == 1 ? (unsigned)p >> 15 : 0u;
            const unsigned long long word =
                ((unsigned long long)(step << 15 | part) << 32) | data;
            __hip_atomic_store(&slots[((size_t)par * G + g) * kSlotWords + lane], word,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          unsigned long long ck = 0;      // this wave's best candidate
          int cp = kNoPos;
          for (int c = wave; c < G; c += kWaves) {
            const unsigned long long* sl = slots + ((size_t)par * G + c) * kSlotWords + lane;
            unsigned long long word =
                __hip_atomic_load(sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned spins = 0;
            while (!dead && __any((unsigned)(word >> 47) != step)) {
              if (++spins > kSpinBusy) __builtin_amdgcn_s_sleep(2);
              if (spins > kSpinLimit) {
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
            const unsigned long long key = pc == kNoPos ? 0 : pivot_rank(x);
            if (key > ck || (key == ck && pc < cp)) {
              ck = key;
              cp = pc;
              reinterpret_cast<unsigned*>(&grow[par][wave][0])[lane] = data;
            }
          }
          if (lane == 0) gcand[par][wave] = Cand{(unsigned)(ck >> 32), (unsigned)ck, cp, 0};
          __syncthreads();
          k = gcand[par][lane & (kWaves - 1)];
          sw = best_lane<kWaves>(k);
          bhi = (unsigned)__builtin_amdgcn_readlane((int)k.hi, sw);
          blo = (unsigned)__builtin_amdgcn_readlane((int)k.lo, sw);
          p = __builtin_amdgcn_readlane(k.pos, sw);
          u = grow[par][sw][lane & (kPw - 1)];
          const int chosen = pivot_position(p, j, h);
          if (chosen != p && tid == 0) atomicOr(&words->err, 2u);
          p = chosen;
        }
        const unsigned long long rank = (unsigned long long)bhi << 32 | blo;
        // a zero, infinite or NaN pivot: ranks 2, of infinity, and below 2
        const bool zero = rank <= 2 || rank - 2 >= 0x7FF0000000000000ull;
        if (tid == 0) piv[j] = p;
        if (zero && g == 0 && tid == 0) atomicMin(&words->bad, (unsigned long long)(c0 + j));
        // exchange positions j and p; the pivot row leaves the elimination and
        // its U part is written back now (every workgroup has read its rows of
        // the panel: it published a candidate from them): what its thread's
        // registers of these columns hold afterwards no longer matters
        if (g == 0 && wave == kWaves - 1 && lane < kPw) {
          const int c = (lane + q * kSub) % kPw;
          if (c >= j && c < w) A[(r0 + j) * lda + c0 + c] = u;
        }
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          if (act[r] && pos[r] == p) {
            act[r] = false;
            pos[r] = j;
            const int lr = g * (kThreads * RPT) + r * kThreads + tid;
            mv->src[j] = lr;
            if (lr < w) mv->dst[lr] = j;
          }
          if (act[r] && pos[r] == j) pos[r] = p;
        }
        double x[RPT];
        if (!zero) {
          double l[RPT];
          const double pj = lane_value(u, jj);
#pragma unroll
          for (int r = 0; r < RPT; ++r) {
            l[r] = a[r][jj] / pj;
            a[r][jj] = l[r];
          }
          auto update = [&](int cb, int ce) {
#pragma unroll
            for (int c = cb; c < ce; ++c) {
              const double uc = lane_value(u, c);
#pragma unroll
              for (int r = 0; r < RPT; ++r) a[r][c] = fma(-l[r], uc, a[r][c]);
            }
          };
          update(jj + 1, kSub);
#pragma unroll
          for (int b = 1; b < kPw / kSub; ++b)
            if (q + b < kPw / kSub) update(b * kSub, (b + 1) * kSub);
        }
#pragma unroll
        for (int r = 0; r < RPT; ++r) x[r] = a[r][jj + 1];
        search(x);
      }
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      double t[kSub];
#pragma unroll
      for (int c = 0; c < kSub; ++c) t[c] = a[r][c];
#pragma unroll
      for (int c = 0; c + kSub < kPw; ++c) a[r][c] = a[r][c + kSub];
#pragma unroll
      for (int c = 0; c < kSub; ++c) a[r][kPw - kSub + c] = t[c];
    }
  }
  // the rows below the panel's triangle, and the L part of the pivot rows
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int lr = g * (kThreads * RPT) + r * kThreads + tid;
    double* dst = A + (r0 + pos[r]) * lda + c0;
    if (act[r] && vec) {
#pragma unroll
      for (int c = 0; c < kPw; c += 2) *reinterpret_cast<D2*>(dst + c) = D2{a[r][c], a[r][c + 1]};
    } else if (lr < h) {
      const int last = act[r] ? w : pos[r];
#pragma unroll
      for (int c = 0; c < kPw; ++c)
        if (c < last) dst[c] = a[r][c];
    }
    if (act[r] && lr < w) mv->dst[lr] = pos[r];
  }
  __syncthreads();
  if (g == 0 && tid < w) ipiv[c0 + tid] = r0 + piv[tid];
}

// A panel's row exchanges in the columns outside it, and the panel's U rows in
// the block's remaining columns [c0 + w, e0): one thread per column gathers
// the (at most 2 w) rows the panel moved -- all loads before the first store
// -- and for those columns solves with the panel's unit lower triangle (x_i =
// b_i - sum_{p<i} l_ip x_p, i and p ascending) before it writes them.  One
// pass over at most 2 w rows of the matrix: 16 us at n = 4096; exchanging the
// rows one pair at a time was a chain of w dependent memory round trips (1 to
// 1.5 us each), once for the block's columns and once for all others.
constexpr int kMoveCols = 64;
__global__ __launch_bounds__(kMoveCols) void panel_apply_kernel(double* __restrict__ A,
                                                                int64_t lda, int64_t n,
                                                                int64_t c0, int w, int64_t e0,
                                                                const Moves* __restrict__ mv) {
  typedef double D2 __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(16))) double Lt[kPw][kPw];   // Lt[p][i] = l_ip
  const int64_t t = (int64_t)blockIdx.x * kMoveCols + threadIdx.x;
  const int64_t col = t < c0 ? t : t + w;
  const bool live = col < n;
  const bool inside = live && col >= c0 + w && col < e0;
  const bool any = __any(inside);
  double* __restrict__ P = A + c0 * lda + (live ? col : 0);
  const int h = (int)(n - c0);
  double x[kPw], y[kPw];
#pragma unroll
  for (int i = 0; i < kPw; ++i)
    x[i] = i < w ? P[(int64_t)moved_row(mv->src[i], i, h) * lda] : 0.0;
#pragma unroll
  for (int i = 0; i < kPw; ++i) y[i] = i < w ? P[(int64_t)i * lda] : 0.0;
  if (any) {
    double l[kPw * kPw / kMoveCols];
#pragma unroll
    for (int e = 0; e < kPw * kPw / kMoveCols; ++e) {
      const int i = (e * kMoveCols + threadIdx.x) / kPw, p = threadIdx.x % kPw;
      l[e] = (i < w && p < i) ? A[(c0 + i) * lda + c0 + p] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < kPw * kPw / kMoveCols; ++e)
      Lt[threadIdx.x % kPw][(e * kMoveCols + threadIdx.x) / kPw] = l[e];
  }
  __syncthreads();
  if (inside) {
#pragma unroll
    for (int p = 0; p + 1 < kPw; ++p)
#pragma unroll
      for (int i = (p + 1) & ~1; i < kPw; i += 2) {
        const D2 l = *reinterpret_cast<const D2*>(&Lt[p][i]);
        if (i > p) x[i] = fma(-l.x, x[p], x[i]);
        x[i + 1] = fma(-l.y, x[p], x[i + 1]);
      }
  }
  if (!live) return;
#pragma unroll
  for (int i = 0; i < kPw; ++i)
    if (i < w) {
      if (inside || mv->src[i] != i) P[(int64_t)i * lda] = x[i];
      const int d = moved_row(mv->dst[i], i, h);
      if (d >= w) P[(int64_t)d * lda] = y[i];
    }
}

// "Swap rows k and ipiv[k]" for k = k0 .. k1-1, in order, on the first ncols
// columns of B (one thread per column).  The exchanges are taken kPw at a
// time: the rows a group names are lane slots of each wave (slot i: row k + i;
// slot kPw + i: row ipiv[k + i] if it is outside the group and no earlier
// exchange of the group names it), the group's exchanges are done on the slot
// contents, and then every named row is loaded once and stored where its
// contents belong, all loads before the first store.  With few columns it is bound by
// the instructions of one wave, so the rows' addresses are made by the lanes, one each,
// and passed by readlane, and the next group's ipiv is on its way meanwhile.
// Measured (one exchange at a time, a memory round trip each, in brackets): 4096
// exchanges of 1 column 663 us (668), 1000 of 10 162 (165), 100 of 100000 44 (41), 8192 of
// 8192 1990 (3610).
constexpr int kSwapCols = 256;
__global__ __launch_bounds__(kSwapCols) void swap_rows_kernel(double* __restrict__ B, int64_t ldb,
                                                              const int64_t* __restrict__ ipiv,
                                                              int64_t k0, int64_t k1,
                                                              int64_t ncols) {
  // All lanes of a wave stay active to the end: a value passed by readlane is lost
  // where its lane is not.  Lanes past the last column repeat it (the same values to
  // the same places), and a wave with none leaves.
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t first = (int64_t)blockIdx.x * kSwapCols + 64 * wave;   // the wave's first column
  if (first >= ncols) return;
  const int lane = threadIdx.x & 63;
  const unsigned c = (unsigned)min((int64_t)lane, ncols - 1 - first);
  double* __restrict__ P = B + first;
  // row `row` (relative to k) of these columns as a lane's address, and a lane's
  // address for every lane
  typedef __attribute__((address_space(1))) double* Row;
  auto address = [&](int64_t k, int row) {
    return __builtin_bit_cast(double, (Row)(P + (k + row) * ldb));
  };
  auto row_of = [&](double adr, int slot) {
    return __builtin_bit_cast(Row, lane_value(adr, slot));
  };
  int64_t next = k0 + lane < k1 ? ipiv[k0 + lane] : k0;
  for (int64_t k = k0; k < k1; k += kPw) {
    const int w = (int)(k1 - k < kPw ? k1 - k : kPw);
    // target of exchange `lane` (lanes 0 .. w-1) as a row relative to k
    const int64_t q = lane < w ? next : k;
    next = k + kPw + lane < k1 ? ipiv[k + kPw + lane] : k0;
    const int off = (int)(q - k);
    const int far = __shfl(off, lane - kPw, 64);
    const int place = lane < kPw ? lane : far;   // the row that this slot names
    int cur = place;                             // and the row now in it
    unsigned long long used = ~0ull >> (64 - w);
    for (int i = 0; i < w; ++i) {
      const int oi = __builtin_amdgcn_readlane(off, i);
      // the slot of the target: its own in the group, or that of the first exchange with it
      const unsigned long long same = __ballot(off == oi) & ~(~0ull << i);
      const int t = oi >= 0 && oi < w ? oi : kPw + (same ? __ffsll(same) - 1 : i);
      used |= 1ull << t;
      const int x = __builtin_amdgcn_readlane(cur, i), y = __builtin_amdgcn_readlane(cur, t);
      cur = lane == i ? y : (lane == t ? x : cur);
    }
    const bool named = used >> lane & 1;
    const double from = address(k, named ? cur : 0), to = address(k, named ? place : 0);
    double v[2 * kPw];
#pragma unroll
    for (int s = 0; s < 2 * kPw; ++s) {
      v[s] = row_of(from, s)[c];
      // (few addresses at a time: the scalar registers do not hold all of them)
      if (s % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
    const unsigned long long mm = __ballot(named && cur != place);
    asm volatile("" : "+v"(next));          // waited for here, not after the stores
#pragma unroll
    for (int s = 0; s < 2 * kPw; ++s)
      if ((mm >> s) & 1) row_of(to, s)[c] = v[s];
  }
}

#define PIV_HIP(...)                                              \
  do {                                                            \
    hipError_t e_ = (__VA_ARGS__);                                \
    if (e_ != hipSuccess) return (trsm_status)note_hip_error(e_); \
  } while (0)

struct Layout {
  int64_t nb, m;
  size_t words, slots, wu, split, total, inv_bytes;
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
  L->words = al(sizeof(Words));
  L->slots = al((size_t)2 * kMaxGroups * kSlotWords * 8) + al(sizeof(Moves));
  L->wu = al((size_t)nb * std::max<int64_t>(n - nb, 1) * 8);
  L->split = kSplitBytes;
  L->total = L->words + L->slots + L->wu + L->split;
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
  return small_tile<double>(p, 1)
             ? launch_gemm<double, double, double, float, 64, 64, 2, 2, false>(p, 1, s)
             : launch_gemm<double, double, double, float, 128, 128, 2, 2, false>(p, 1, s);
}

// One panel.  Rows per thread and workgroups: one workgroup while the rows fit
// (no meeting); then one row per thread while every wave has at most one
// candidate to wait for, because a step's update and LDS traffic grow with
// the rows per thread; two beyond that, to bound the candidates to read.
//
// Several workgroups wait for each other, so all of them have to run at once.  Few of
// one row per thread are launched like any other kernel where the device has room
// for many such panels (plain_groups): every kernel beside them ends by itself, and a
// wait that lasts all the same ends at kSpinLimit with the error word set.  A
// cooperative launch idles about 11 us before and after it (n = 4096, 96 panels of 78
// us: 15.7 ms with it, 13.7 without) and remains for more workgroups and for smaller
// devices.

// Panels' workgroups of one row per thread that the current device has room for;
// looked up once per device.
hipError_t panel_places(int* places) {
  constexpr int kMaxDevices = 64;
  static std::atomic<int> known[kMaxDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  int v = dev >= 0 && dev < kMaxDevices ? known[dev].load(std::memory_order_relaxed) : 0;
  if (v == 0) {
    int per = 0, units = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per, reinterpret_cast<const void*>(piv_panel_kernel<1, true>), kThreads, 0);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    v = per * units;
    if (dev >= 0 && dev < kMaxDevices) known[dev].store(v, std::memory_order_relaxed);
  }
  *places = v;
  return hipSuccess;
}

template <int RPT, bool MULTI>
hipError_t launch_panel(double* A, int64_t lda, int64_t c, int h, int w, int64_t* ipiv,
                        unsigned long long* slots, Words* words, Moves* mv, hipStream_t s) {
  if constexpr (!MULTI) {
    piv_panel_kernel<RPT, false><<<1, kThreads, 0, s>>>(A, lda, c, c, h, w, ipiv, slots, words, mv);
    return hipGetLastError();
  } else {
    const int64_t groups = ceil_div(h, kThreads * RPT);
    int places = 0;
    if (RPT == 1) {
      const hipError_t e = panel_places(&places);
      if (e != hipSuccess) return e;
    }
    if (RPT == 1 && groups <= plain_groups(places)) {
      piv_panel_kernel<RPT, true><<<(unsigned)groups, kThreads, 0, s>>>(A, lda, c, c, h, w, ipiv,
                                                                       slots, words, mv);
      return hipGetLastError();
    }
    int64_t r0 = c, cc = c;
    void* args[] = {&A, &lda, &r0, &cc, &h, &w, &ipiv, &slots, &words, &mv};
    return hipLaunchCooperativeKernel(
        reinterpret_cast<const void*>(piv_panel_kernel<RPT, true>),
        dim3((unsigned)groups), dim3(kThreads), args, 0, s);
  }
}

trsm_status factor(int64_t n, double* A, int64_t lda, const Layout& L, int64_t* ipiv,
                   double* Linv, char* ws, hipStream_t s) {
  const int64_t nb = L.nb;
  Words* words = (Words*)ws;
  char* q = ws + L.words;
  unsigned long long* slots = (unsigned long long*)q;
  Moves* mv = (Moves*)(q + al((size_t)2 * kMaxGroups * kSlotWords * 8));
  q += L.slots;
  double* WU = (double*)q;     q += L.wu;
  void* split = q;
  // words: bad = all ones, err = 0; no slot carries a step number of this call
  PIV_HIP(launch_fill_u32((unsigned*)words, 2, 0xFFFFFFFFu, s));
  PIV_HIP(launch_fill_u32((unsigned*)words + 2, 2, 0u, s));
  if (n > kThreads * kMaxRpt)
    PIV_HIP(launch_fill_u32((unsigned*)slots, (int64_t)4 * kMaxGroups * kSlotWords, 0u, s));
  trsm_status st = TRSM_OK;
  for (int64_t j = 0; j < L.m && st == TRSM_OK; ++j) {
    const int64_t c0 = j * nb, sb = std::min(nb, n - c0), e0 = c0 + sb;
    hipError_t e = hipSuccess;
    for (int64_t c = c0; c < e0 && e == hipSuccess; c += kPw) {
      const int w = (int)std::min<int64_t>(kPw, e0 - c);
      const int h = (int)(n - c);
      if (h <= kThreads)
        e = launch_panel<1, false>(A, lda, c, h, w, ipiv, slots, words, mv, s);
      else if (h <= 2 * kThreads)
        e = launch_panel<2, false>(A, lda, c, h, w, ipiv, slots, words, mv, s);
      else if (h <= kWaves * kThreads)
        e = launch_panel<1, true>(A, lda, c, h, w, ipiv, slots, words, mv, s);
      else
        e = launch_panel<2, true>(A, lda, c, h, w, ipiv, slots, words, mv, s);
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
    double* Lj = Linv + j * nb * nb;
    if (e == hipSuccess)
      e = launch_block_inverse<double>(A + c0 * lda + c0, lda, sb, nb, 1, Lj, nullptr, false, true,
                                       s);
    if (e == hipSuccess) e = rec_tri_inv_levels(Lj, nb, 1, s);
    if (e == hipSuccess && nb > kInvRows)
      e = launch_block_finish<double>(nullptr, 0, 0, nb, 1, Lj, nullptr, nullptr, s);
    const int64_t t = n - e0;
    if (e == hipSuccess && t > 0) {
      // U(S_j, T_j) = Linv_jj A(S_j, T_j), then the trailing update
      e = prod(Lj, nb, A + c0 * lda + e0, lda, WU, t, sb, t, sb, 1.0, false,
               G_A_LOWER | G_A_ZERO_UPPER, split, kSplitBytes, s);
      if (e == hipSuccess) e = launch_copy2d<double, double>(WU, t, A + c0 * lda + e0, lda, sb, t,
                                                             1.0, s);
      if (e == hipSuccess)
        e = prod(A + e0 * lda + c0, lda, A + c0 * lda + e0, lda, A + e0 * lda + e0, lda, t, t, sb,
                 -1.0, true, 0u, split, kSplitBytes, s);
    }
    if (e != hipSuccess) st = (trsm_status)note_hip_error(e);
  }
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
