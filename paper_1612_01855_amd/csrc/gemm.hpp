// Tiled matrix-core GEMM for gfx950, the workhorse of every dense product on
// the solve path: the diagonal-block apply X(S_i) = Linv_ii * B'(S_i) and the
// trailing update B'(T_{i+1}) -= L(T_{i+1}, S_i) X(S_i) of Alg. It-Inv-TRSM,
// the two products of each Alg. RecTriInv combine level, the recursive
// baseline's off-diagonal update, and the residual B - L X.
//
//   Cout = beta * Cin + alpha * rowscale .* (op(A) * op(B))        (per batch)
//
// * A is M x K row-major (k contiguous).  B is K x N row-major (n contiguous)
//   or, with BKMAJOR, stored N x K (k contiguous).  Both are staged through
//   LDS k-contiguous, so every lane reads 32 contiguous bytes of a row.
// * G_A_LOWER: A is lower triangular (A[i][k] = 0 for k > i).  Whole tiles
//   past the diagonal are skipped and the diagonal tile is masked, so
//   whatever is stored above A's diagonal is never used.
// * G_B_LOWER: B is lower triangular (B[k][j] = 0 for k < j), same treatment.
// * G_A_UPPER: A is upper triangular and stores zeros below its diagonal;
//   the chunks left of a tile's diagonal are skipped.
// * Optional second output C2 (another precision, optionally transposed,
//   optionally scaled) feeds a following low-precision product.
// * Batches: z -> offset (z / zdiv) * outer + (z % zdiv) * inner.
//
// Work decomposition: a workgroup of WGM x WGN waves owns a BM x BN tile;
// each wave owns (BM/WGM) x (BN/WGN) made of 16x16 MFMA tiles.  K advances in
// chunks of 128 bytes with two LDS stages and one barrier per chunk.
// Binary64/binary32 products copy their operands from HBM directly into LDS
// (buffer loads with the LDS modifier, no register staging), other types stage
// them through registers.  Square lower-triangular products are
// folded so that every workgroup gets equal work.  Tiles are visited in groups of GROUP_M row
// tiles (column-major inside a group) so that concurrently running
// workgroups share A and B panels in L2.  The hardware deals consecutive
// workgroup ids to the eight XCDs in turn; dense products regroup the ids so
// that each XCD works on a contiguous range of tiles (2.3x less L2-miss
// traffic), triangular products keep the round-robin order because a
// contiguous range per XCD unbalanced their uneven tile costs (the
// lower-triangular residual ran twice as slow).
#pragma once

#include "common.hpp"

#include <algorithm>
#include <type_traits>

namespace trsm {

// How a product's operands reach LDS (gemm_mode).
enum GemmMode { kStaged, kDma4, kDma16A, kDma16 };
// Which way a tile runs through K: as its flags say, or known when compiled.
enum GemmDir { kByFlags, kUp, kDown };

enum GemmFlags : uint32_t {
  G_A_LOWER = 1u,
  G_B_LOWER = 2u,
  G_C2_T = 4u,       // C2 stored transposed: C2[col * ldc2 + row]
  G_BETA = 8u,       // read Cin
  G_ROWSCALE = 16u,  // multiply the product by rscale[row * ld_rs]
  G_A_ZERO_UPPER = 32u,  // with G_A_LOWER: A's upper triangle is stored as zeros (no masking)
  G_A_UPPER = 64u,       // A upper triangular with zeros stored below the diagonal: the
                         // zero chunks are skipped (no masking)
  G_C_LOWER = 128u,      // only the lower triangle of a square C (M == N, BM == BN) is
                         // computed: tiles above the diagonal are not launched and elements
                         // above it are left untouched (the symmetric rank-K update)
};

template <typename TIn, typename TCin, typename TCout, typename TC2>
struct GemmParams {
  const TIn* A; int64_t lda; int64_t sa_o, sa_i;
  const TIn* B; int64_t ldb; int64_t sb_o, sb_i;
  const TCin* Cin; int64_t ldci; int64_t sci_o, sci_i;
  TCout* Cout; int64_t ldco; int64_t sco_o, sco_i;
  TC2* C2; int64_t ldc2;
  const float* rscale; int64_t ld_rs;
  const float* ascale;        // if set, alpha is multiplied by *ascale (device value)
  void* part;                 // split-K scratch (element type Mfma<TIn>::Acc), or null
  int64_t part_bytes;         // its size; the launcher picks ksplit to fit
  int ksplit;                 // set by the launcher: K slices (<= 1: no split)
  int M, N, K;
  int zdiv;
  double alpha, beta;
  float c2scale;
  uint32_t flags;
};

template <typename T> struct VecOf;
template <> struct VecOf<double> { typedef double T2 __attribute__((ext_vector_type(2))); };
template <> struct VecOf<float> { typedef float T2 __attribute__((ext_vector_type(4))); };
template <> struct VecOf<bf16_t> { typedef __bf16 T2 __attribute__((ext_vector_type(8))); };
template <> struct VecOf<f16_t> { typedef _Float16 T2 __attribute__((ext_vector_type(8))); };
template <> struct VecOf<fp8_t> { typedef uint8_t T2 __attribute__((ext_vector_type(16))); };

// Buffer descriptor word 3 for the gfx9 family (raw, untyped loads).
constexpr int kBufWord3 = 0x00020000;
// Offsets at or above this value read as zero (outside the descriptor).
constexpr int kBufOOB = 0x7FFFFFF0;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, kBufOOB, kBufWord3);
}

template <typename V>
__device__ __forceinline__ V buf_load16(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}


// A square lower-triangular A (M == K) makes the tile cost grow with the
// row index.  Such products are "folded": one workgroup computes row tile t
// and row tile ntm-1-t of the same column, so every workgroup gets the same
// amount of work (and half as many workgroups are launched).
__host__ __device__ inline bool tri_fold(int M, int K, uint32_t flags, int BM) {
  return (flags & (G_A_LOWER | G_A_UPPER)) && M == K && (M + BM - 1) / BM >= 2;
}

// Workgroups one product needs.
__host__ __device__ inline int gemm_wgs(int M, int N, int K, uint32_t flags, int BM, int BN) {
  const int ntm = (M + BM - 1) / BM, ntn = (N + BN - 1) / BN;
  if (flags & G_C_LOWER) return ntm * (ntm + 1) / 2;
  return (tri_fold(M, K, flags, BM) ? (ntm + 1) / 2 : ntm) * ntn;
}

// Tile (tm, tn), tn <= tm, of workgroup `bid` among the t (t + 1) / 2 that
// cover the lower triangle of a t x t tile grid.  Row tiles are paired, a
// with t - 1 - a, so that a run of t + 1 consecutive ids covers one pair
// (a + 1 tiles of row a, then t - a of row t - 1 - a); with a multiple of 8
// workgroups the ids are regrouped so that each XCD takes a contiguous range
// of pairs (they share their rows of A in its L2).
__device__ __forceinline__ void lower_tile(int t, int bid, int nwg, int& tm, int& tn) {
  if ((nwg & 7) == 0) bid = (bid & 7) * (nwg >> 3) + (bid >> 3);
  const int pr = bid / (t + 1), q = bid - pr * (t + 1);
  if (q <= pr) {
    tm = pr;
    tn = q;
  } else {
    tm = t - 1 - pr;
    tn = q - pr - 1;
  }
}

// Row slot and column of workgroup `bid` among the nwg workgroups of one
// product: groups of GROUP_M row slots, column-major inside a group.  The
// hardware deals consecutive workgroup ids to the eight XCDs in turn;
// products with uniform tile cost (dense, folded, or a single group of row
// slots) regroup the ids so that each XCD works on a contiguous range of
// tiles and its concurrent workgroups share panels in its own L2 (2.3x less
// L2-miss traffic).  Other triangular products keep the round-robin order,
// which spreads their uneven tile costs over the XCDs (a contiguous range of
// row groups per XCD made an unfolded lower-triangular product twice as slow).
template <int GROUP_M, bool XCD_REMAP>
__device__ __forceinline__ void tile_slot(int rows, int ntn, bool uniform, int bid, int nwg,
                                          int& slot, int& tn) {
  const bool remap = XCD_REMAP || uniform || rows <= GROUP_M;
  if (remap && (nwg & 7) == 0) bid = (bid & 7) * (nwg >> 3) + (bid >> 3);
  const int per_group = GROUP_M * ntn;
  const int grp = bid / per_group;
  const int first_m = grp * GROUP_M;
  const int gsize = min(rows - first_m, GROUP_M);
  const int in_grp = bid % per_group;
  slot = first_m + in_grp % gsize;
  tn = in_grp / gsize;
}

// Reduction range of a tile: whole chunks of BK from kbeg, skipping the zero
// part of a triangular operand.  Returns the number of chunks.
template <int BM, int BK>
__device__ __forceinline__ int chunk_range(int K, uint32_t flags, int r0, int c0, int& kbeg) {
  int kend = K;
  kbeg = 0;
  if (flags & G_A_LOWER) kend = min(K, r0 + BM);
  if (flags & G_A_UPPER) kbeg = (min(r0, K) / BK) * BK;
  if (flags & G_B_LOWER) kbeg = (min(c0, K) / BK) * BK;
  return kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
}

// Split-K: slice s of S covers the global chunks [s*cps, (s+1)*cps) of K,
// intersected with the tile's own range.
template <int BK>
__device__ __forceinline__ int split_range(int K, int s, int S, int nchunks, int& kbeg) {
  if (S <= 1) return nchunks;
  const int nck = (K + BK - 1) / BK, cps = (nck + S - 1) / S;
  const int lo = max(s * cps, kbeg / BK), hi = min((s + 1) * cps, kbeg / BK + nchunks);
  kbeg = lo * BK;
  return hi > lo ? hi - lo : 0;
}

template <typename TIn, typename TCin, typename TCout>
using EpiType = typename std::conditional<std::is_same<TCout, double>::value ||
                                              std::is_same<TCin, double>::value,
                                          double, typename Mfma<TIn>::Acc>::type;

// One output element: Cout = beta*Cin + alpha*rs*v (+ second output).
template <typename TIn, typename TCin, typename TCout, typename TC2, typename Epi>
__device__ __forceinline__ void epi_store(const GemmParams<TIn, TCin, TCout, TC2>& p,
                                          TCout* __restrict__ Co, const TCin* __restrict__ Ci,
                                          int row, int col, Epi v, Epi alpha, Epi beta,
                                          bool use_beta, Epi rs) {
  v = alpha * (v * rs);
  if (use_beta) v += beta * static_cast<Epi>(Ci[(int64_t)row * p.ldci + col]);
  Co[(int64_t)row * p.ldco + col] = static_cast<TCout>(v);
  if (p.C2) {
    const TC2 w = cvt<TC2>(v * static_cast<Epi>(p.c2scale));
    if (p.flags & G_C2_T) p.C2[(int64_t)col * p.ldc2 + row] = w;
    else p.C2[(int64_t)row * p.ldc2 + col] = w;
  }
}

// Epilogue: Cout = beta*Cin + alpha*rowscale*acc (+ optional second output).
// Lane (gi, g) holds column gi and rows out_row(g, r) of every 16x16 tile.
template <typename TIn, typename TCin, typename TCout, typename TC2, int TM, int TN, int WTM,
          int WTN>
__device__ __forceinline__ void gemm_epilogue(const GemmParams<TIn, TCin, TCout, TC2>& p,
                                              const typename Mfma<TIn>::Out (&acc)[TM][TN],
                                              int zo, int zi, int z, int s, int r0, int c0,
                                              int wm, int wn, int g, int gi) {
  using MF = Mfma<TIn>;
  using Acc = typename MF::Acc;
  const int M = p.M, N = p.N;
  if (p.ksplit > 1) {
    // split-K: raw partial sums, summed and finished by gemm_splitk_finish
    Acc* __restrict__ P = static_cast<Acc*>(p.part) + ((int64_t)z * p.ksplit + s) * M * N;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = r0 + wm * WTM + i * 16 + MF::out_row(g, r);
        if (row >= M) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int col = c0 + wn * WTN + j * 16 + gi;
          if (col < N) P[(int64_t)row * N + col] = acc[i][j][r];
        }
      }
    return;
  }
  TCout* __restrict__ Co = p.Cout + zo * p.sco_o + zi * p.sco_i;
  const TCin* __restrict__ Ci = p.Cin ? p.Cin + zo * p.sci_o + zi * p.sci_i : nullptr;
  const bool use_beta = (p.flags & G_BETA) && Ci;
  const bool use_rs = (p.flags & G_ROWSCALE) && p.rscale;
  // the epilogue runs in binary64 whenever C is binary64 on either side
  using Epi = EpiType<TIn, TCin, TCout>;
  Epi alpha = static_cast<Epi>(p.alpha);
  if (p.ascale) alpha *= static_cast<Epi>(*p.ascale);
  const Epi beta = static_cast<Epi>(p.beta);
  const bool c_lower = p.flags & G_C_LOWER;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = r0 + wm * WTM + i * 16 + MF::out_row(g, r);
      if (row >= M) continue;
      Epi rs = Epi(1);
      if (use_rs) rs = static_cast<Epi>(p.rscale[(int64_t)row * p.ld_rs]);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = c0 + wn * WTN + j * 16 + gi;
        if (col >= N || (c_lower && col > row)) continue;
        epi_store(p, Co, Ci, row, col, static_cast<Epi>(acc[i][j][r]), alpha, beta, use_beta, rs);
      }
    }
  }
}

// Epilogue for products computed with the MFMA operands swapped (the tile of
// C^T is accumulated): lane (gi, g) then holds row gi and the four adjacent
// columns 4g..4g+3 of every 16x16 tile, so binary32 C moves in 16-byte
// vectors.
template <typename TIn, typename TCin, typename TCout, typename TC2, int TM, int TN, int WTM,
          int WTN>
__device__ __forceinline__ void gemm_epilogue_t(const GemmParams<TIn, TCin, TCout, TC2>& p,
                                                const typename Mfma<TIn>::Out (&acc)[TM][TN],
                                                int zo, int zi, int z, int s, int r0, int c0,
                                                int wm, int wn, int g, int gi) {
  using MF = Mfma<TIn>;
  using Acc = typename MF::Acc;
  const int M = p.M, N = p.N;
  if (p.ksplit > 1) {
    Acc* __restrict__ P = static_cast<Acc*>(p.part) + ((int64_t)z * p.ksplit + s) * M * N;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = r0 + wm * WTM + i * 16 + gi;
      if (row >= M) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int col = c0 + wn * WTN + j * 16 + 4 * g + r;
          if (col < N) P[(int64_t)row * N + col] = acc[i][j][r];
        }
    }
    return;
  }
  TCout* __restrict__ Co = p.Cout + zo * p.sco_o + zi * p.sco_i;
  const TCin* __restrict__ Ci = p.Cin ? p.Cin + zo * p.sci_o + zi * p.sci_i : nullptr;
  const bool use_beta = (p.flags & G_BETA) && Ci;
  const bool use_rs = (p.flags & G_ROWSCALE) && p.rscale;
  using Epi = EpiType<TIn, TCin, TCout>;
  Epi alpha = static_cast<Epi>(p.alpha);
  if (p.ascale) alpha *= static_cast<Epi>(*p.ascale);
  const Epi beta = static_cast<Epi>(p.beta);
  constexpr bool F32C = std::is_same<TCout, float>::value && std::is_same<TCin, float>::value;
  const bool c_lower = p.flags & G_C_LOWER;
  const bool vec = F32C && !p.C2 && !c_lower &&
                   (((uintptr_t)Co | (uintptr_t)(Ci ? Ci : Co) | (uintptr_t)(p.ldco * 4) |
                     (uintptr_t)(p.ldci * 4)) & 15) == 0;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = r0 + wm * WTM + i * 16 + gi;
    if (row >= M) continue;
    const Epi rs = use_rs ? static_cast<Epi>(p.rscale[(int64_t)row * p.ld_rs]) : Epi(1);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col0 = c0 + wn * WTN + j * 16 + 4 * g;
      if constexpr (F32C) {
        if (vec && col0 + 3 < N) {
          typedef float F4 __attribute__((ext_vector_type(4)));
          F4 cin = {0.f, 0.f, 0.f, 0.f};
          if (use_beta) cin = *reinterpret_cast<const F4*>(Ci + (int64_t)row * p.ldci + col0);
          F4 o;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            Epi v = alpha * (static_cast<Epi>(acc[i][j][r]) * rs);
            if (use_beta) v += beta * static_cast<Epi>(cin[r]);
            o[r] = static_cast<float>(v);
          }
          *reinterpret_cast<F4*>(Co + (int64_t)row * p.ldco + col0) = o;
          continue;
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int col = col0 + r;
        if (col < N && !(c_lower && col > row))
          epi_store(p, Co, Ci, row, col, static_cast<Epi>(acc[i][j][r]), alpha, beta, use_beta, rs);
      }
    }
  }
}

// s_waitcnt immediate that waits for at most n outstanding vector-memory
// operations and nothing else (gfx9 encoding).
constexpr int vmcnt_imm(int n) {
  return (n & 0xF) | (((n >> 4) & 3) << 14) | (0x7 << 4) | (0xF << 8);
}

// s_waitcnt immediate that waits for every vector-memory and LDS operation.
constexpr int kWaitAll = 0x7 << 4;

// LDS of gemm_tile_dma: two stages of A's and B's 128 bytes of k (B row-major: 16
// bytes between the KB that one instruction copies).
template <typename TIn, int BM, int BN, bool BKMAJOR>
constexpr int dma_lds() {
  const int bk = 128 / (int)sizeof(TIn), row_b = BN * (int)sizeof(TIn);
  return 2 * (BM * 128 + (BKMAJOR ? BN * 128 : bk * row_b / 1024 * (1024 + 16)));
}

// Matrix-core tile with operands copied from HBM straight into LDS by
// buffer loads (no register staging), two LDS stages, one barrier per chunk.
// For one-k-per-lane instructions (binary64, binary32).  A16 / B16: the operand's
// rows are 16-byte aligned and are copied 16 bytes a lane; otherwise 4 bytes a
// lane into the same layout (element alignment is enough, and nothing past a row's
// end is read), four times as many copies but still without registers or a wait
// (6000 x 6000 x 1024 in 64 x 64 tiles: binary64 1372 us, staged through registers
// 1651 and in 128 x 128 tiles 1606; binary32 726, 1086 and 1042).  LDS layout
// per stage:
//  * A: BM rows of 128 bytes (BK elements), the eight 16-byte pieces of row r
//    stored XOR-swizzled (piece d at position d ^ (r & 7)), so that the 16
//    rows a fragment read touches fall in different banks;
//  * B, row-major (BKMAJOR false): BK rows of BN elements; each wave load
//    instruction writes 1 KB (one or more whole rows) and is followed by 16
//    bytes of padding;
//  * B given as B^T (BKMAJOR true: N rows of K, k contiguous): BN rows of
//    128 bytes swizzled like A, and read like A.
// A half-chunk's fragments are read one half ahead of their MFMAs, across the
// chunk boundary too: the second half while the first multiplies, and the
// next chunk's first half, after the one barrier per chunk, while the second
// multiplies.  At that barrier every wave holds both halves of chunk c, so its
// stage is free for chunk c + 2 and two stages keep a whole chunk time between
// a copy and its use.  (Reading each half right before its MFMAs left the
// matrix cores idle for two LDS latencies per chunk.)
// AHEAD false: each half is read right before its MFMAs, and the next chunk's copies go
// out at the start of a chunk.  For the persistent sweep, whose tiles are a few chunks
// between fences and wait for memory most of the time: 4 systems of 2000 x 500 in
// binary32 4605 us, with the reads ahead 6005.
// K runs towards the diagonal (for G_A_UPPER downwards, the lane groups in turn too):
// the diagonal's term, the largest of an inverted block's row, is added last, and the
// sum before it rounds at its own size.
// Triangular masks are applied to the fragments, only in chunks that cross
// the diagonal.
template <typename TIn, typename TCin, typename TCout, typename TC2, int BM, int BN, int WGM,
          int WGN, bool BKMAJOR = false, bool A16 = true, bool B16 = true, bool AHEAD = true,
          int DIR = kByFlags>
__device__ __forceinline__ void gemm_tile_dma(const GemmParams<TIn, TCin, TCout, TC2>& p, int z,
                                              int s, const int r0, const int c0,
                                              char* const smem) {
  using MF = Mfma<TIn>;
  using Acc = typename MF::Acc;
  using Out = typename MF::Out;
  using V16 = typename VecOf<TIn>::T2;
  constexpr int NW = WGM * WGN;
  constexpr int ES = sizeof(TIn);
  constexpr int VEC = 16 / ES;
  constexpr int BK = 128 / ES;
  constexpr int KL = BK / 4;                     // k per lane group per chunk (32 bytes)
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int A_BYTES = BM * 128;
  constexpr int ROW_B = BN * ES;                 // bytes of one B row
  constexpr int RPI = 1024 / ROW_B;              // B rows per wave instruction
  constexpr int B_INST_TOTAL = BK / RPI;
  constexpr int B_BYTES = BKMAJOR ? BN * 128 : B_INST_TOTAL * (1024 + 16);
  constexpr int STAGE = A_BYTES + B_BYTES;
  constexpr int A_INST = BM / 8 / NW;
  constexpr int B_INST = B_INST_TOTAL / NW;
  constexpr int BT_INST = BN / 8 / NW;
  static_assert(MF::kPerLane == 1, "one k per lane");
  static_assert(RPI * ROW_B == 1024, "a wave instruction must cover whole B rows");
  static_assert(A_INST * NW * 8 == BM && B_INST * NW == B_INST_TOTAL, "even split of loads");
  static_assert(!BKMAJOR || BT_INST * NW * 8 == BN, "even split of B^T loads");
  static_assert(2 * STAGE == dma_lds<TIn, BM, BN, BKMAJOR>(), "the caller's LDS");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN, gi = lane & 15, g = lane >> 4;
  const int zo = z / p.zdiv, zi = z % p.zdiv;
  const TIn* __restrict__ A = p.A + zo * p.sa_o + zi * p.sa_i;
  const TIn* __restrict__ B = p.B + zo * p.sb_o + zi * p.sb_i;
  const int M = p.M, N = p.N, K = p.K;
  const int lda = (int)p.lda, ldb = (int)p.ldb;
  int kbeg;
  int nchunks = chunk_range<BM, BK>(K, p.flags, r0, c0, kbeg);
  nchunks = split_range<BK>(K, s, p.ksplit, nchunks, kbeg);
  const bool a_lower = (p.flags & G_A_LOWER) && !(p.flags & G_A_ZERO_UPPER);
  const bool b_lower = p.flags & G_B_LOWER;
  const bool down = DIR == kByFlags ? p.flags & G_A_UPPER : DIR == kDown;
  const int kfirst = down ? kbeg + (nchunks - 1) * BK : kbeg, kstep = down ? -BK : BK;
  const int gk = down ? 3 - g : g;               // an instruction adds its lane groups in turn

  Out acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = Acc(0);

  // Copies of chunk c into stage st.  The large tile issues past the last chunk
  // too (RUNON: every lane's offset is then out of range, and zeros nobody reads
  // arrive): without a branch the copies' instructions are scheduled among
  // the MFMAs (n = k = 16384: 68.1 against 70.6 ms).  A small tile has few chunks
  // and skips them.
  constexpr bool RUNON = BM * BN >= 128 * 128;
  auto issue = [&](int c, int st) {
    const int k0 = kfirst + c * kstep;
    const int kend = !RUNON || c < nchunks ? K : DIR == kUp ? 0 : INT32_MIN;   // (k0 < 0 downwards)
    char* base = smem + st * STAGE;
    // rows [row0, row0 + 8 INST NW) of a k-contiguous operand, swizzled
    auto rows_of = [&](const TIn* P, int ld, int row0, int rows, char* dst, auto inst, auto wide) {
      const __amdgpu_buffer_rsrc_t rs = make_rsrc(P + (int64_t)row0 * ld + k0);
#pragma unroll
      for (int q = 0; q < inst(); ++q) {
        const int rb = 8 * (wave * inst() + q);
        if constexpr (wide()) {
          const int r = rb + (lane >> 3);
          const int d = (lane & 7) ^ (r & 7);
          const bool ok = (row0 + r < rows) && (k0 + d * VEC < kend);
          const int off = ok ? (r * ld + d * VEC) * ES : kBufOOB;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(
              rs, (__attribute__((address_space(3))) void*)(dst + rb * 128), 16, off, 0, 0, 0);
        } else {
#pragma unroll
          for (int w = 0; w < 4; ++w) {   // two rows a copy
            const int r = rb + 2 * w + (lane >> 5);
            const int byte = ((((lane & 31) >> 2) ^ (r & 7)) << 4) + ((lane & 3) << 2);
            const bool ok = (row0 + r < rows) && (k0 + byte / ES < kend);
            const int off = ok ? r * ld * ES + byte : kBufOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (__attribute__((address_space(3))) void*)(dst + rb * 128 + w * 256), 4, off, 0,
                0, 0);
          }
        }
      }
    };
    rows_of(A, lda, r0, M, base, std::integral_constant<int, A_INST>(),
            std::integral_constant<bool, A16>());
    if constexpr (BKMAJOR) {
      rows_of(B, ldb, c0, N, base + A_BYTES, std::integral_constant<int, BT_INST>(),
              std::integral_constant<bool, B16>());
    } else {
      const __amdgpu_buffer_rsrc_t rbs = make_rsrc(B + (int64_t)k0 * ldb + c0);
#pragma unroll
      for (int q = 0; q < B_INST; ++q) {
        const int qi = wave * B_INST + q;
        char* dst = base + A_BYTES + qi * (1024 + 16);
        if constexpr (B16) {
          const int kr = qi * RPI + lane / (64 / RPI);
          const int cv = (lane % (64 / RPI)) * VEC;
          const bool ok = (k0 + kr < kend) && (c0 + cv < N);
          const int off = ok ? (kr * ldb + cv) * ES : kBufOOB;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(
              rbs, (__attribute__((address_space(3))) void*)dst, 16, off, 0, 0, 0);
        } else {
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int x = w * 256 + lane * 4;   // byte of this copy's 1 KB of rows
            const int kr = qi * RPI + x / ROW_B, byte = x % ROW_B;
            const bool ok = (k0 + kr < kend) && (c0 + byte / ES < N);
            const int off = ok ? kr * ldb * ES + byte : kBufOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rbs, (__attribute__((address_space(3))) void*)(dst + w * 256), 4, off, 0, 0, 0);
          }
        }
      }
    }
  };
  // Fragments of half h (the lane group's h-th 16-byte piece of k) of chunk c.
  struct Half {
    V16 a[TM];
    TIn b[VEC][TN];
  };
  auto fetch = [&](Half& f, int c, int h) {
    const char* as = smem + (c & 1) * STAGE;
    const char* bs = as + A_BYTES;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int r = wm * WTM + i * 16 + gi;
      const int slot = (2 * gk + h) ^ (r & 7);
      f.a[i] = *reinterpret_cast<const V16*>(as + r * 128 + slot * 16);
    }
    if constexpr (BKMAJOR) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int r = wn * WTN + j * 16 + gi;
        const int slot = (2 * gk + h) ^ (r & 7);
        const V16 v = *reinterpret_cast<const V16*>(bs + r * 128 + slot * 16);
#pragma unroll
        for (int e = 0; e < VEC; ++e) f.b[e][j] = v[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const int kr = gk * KL + h * VEC + e;
#pragma unroll
        for (int j = 0; j < TN; ++j)
          f.b[e][j] = *reinterpret_cast<const TIn*>(bs + (kr / RPI) * (1024 + 16) +
                                                    (kr % RPI) * ROW_B +
                                                    (wn * WTN + j * 16 + gi) * ES);
      }
    }
  };
  // 16-byte pieces of A beside 4-byte copies of B: the last piece may reach past K
  const int k_tail = A16 && !B16 && K % VEC ? K : INT32_MAX;
  auto mask = [&](Half& f, int c, int h) {
    const int k0 = kfirst + c * kstep;
    if (k0 + BK > k_tail) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < VEC; ++e)
          if (k0 + gk * KL + h * VEC + e >= k_tail) f.a[i][e] = TIn(0);
    }
    if (a_lower && k0 + BK - 1 > r0 + wm * WTM) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < VEC; ++e)
          if (k0 + gk * KL + h * VEC + e > r0 + wm * WTM + i * 16 + gi) f.a[i][e] = TIn(0);
    }
    if (b_lower && k0 < c0 + wn * WTN + WTN - 1) {
#pragma unroll
      for (int e = 0; e < VEC; ++e)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          if (k0 + gk * KL + h * VEC + e < c0 + wn * WTN + j * 16 + gi) f.b[e][j] = TIn(0);
    }
  };
  auto multiply = [&](const Half& f) {
#pragma unroll
    for (int e = 0; e < VEC; ++e)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = MF::mma(f.a[i][e], f.b[e][j], acc[i][j]);
  };

  if constexpr (!AHEAD) {
    const bool masked = a_lower || b_lower || k_tail != INT32_MAX;
    if (nchunks > 0) issue(0, 0);
    for (int c = 0; c < nchunks; ++c) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // this wave's part of chunk c has landed
      __syncthreads();                            // ... everyone's; and chunk c - 1 is consumed
      if (c + 1 < nchunks) issue(c + 1, (c + 1) & 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        Half f;
        fetch(f, c, h);
        if (masked) mask(f, c, h);
        multiply(f);
      }
    }
  } else if (nchunks > 0) {
    // copies per wave and chunk
    constexpr int LPC = A_INST * (A16 ? 1 : 4) + (BKMAJOR ? BT_INST : B_INST) * (B16 ? 1 : 4);
    static_assert(LPC < 32, "two chunks' copies fit the counter of outstanding copies");
    Half f0, f1;
    issue(0, 0);
    if (RUNON || nchunks > 1) {
      issue(1, 1);
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(LPC));   // this wave's part of chunk 0 has landed
    } else {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    }
    __syncthreads();                                // ... everyone's
    fetch(f0, 0, 0);
    const bool masked = a_lower || b_lower || k_tail != INT32_MAX;
    for (int c = 0; c < nchunks; ++c) {
      // the reads go out before the MFMAs (the scheduler would sink them)
      fetch(f1, c, 1);
      __builtin_amdgcn_sched_barrier(0);
      if (masked) mask(f0, c, 0);
      multiply(f0);
      // both halves of chunk c are in registers and chunk c + 1 has landed,
      // for every wave: its stage takes chunk c + 2
      if (RUNON || c + 1 < nchunks) {
        __builtin_amdgcn_s_waitcnt(kWaitAll);
        __syncthreads();
      }
      if (RUNON || c + 1 < nchunks) fetch(f0, c + 1, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (RUNON || c + 2 < nchunks) issue(c + 2, c & 1);
      if (masked) mask(f1, c, 1);
      multiply(f1);
    }
    // RUNON's last copies: nothing may still be writing the stages
    if (RUNON) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  }
  gemm_epilogue<TIn, TCin, TCout, TC2, TM, TN, WTM, WTN>(p, acc, zo, zi, z, s, r0, c0, wm, wn, g,
                                                        gi);
}

// Register-staged tile: bfloat16/half products with k-contiguous B, and any product
// whose tiles span more than a buffer descriptor.
template <typename TIn, typename TCin, typename TCout, typename TC2,
          int BM, int BN, int WGM, int WGN, bool BKMAJOR, bool ALIGNED>
__device__ __forceinline__ void gemm_tile_staged(const GemmParams<TIn, TCin, TCout, TC2>& p,
                                                 int z, int s, const int r0, const int c0) {
  using MF = Mfma<TIn>;
  using Acc = typename MF::Acc;
  using Out = typename MF::Out;
  using V16 = typename VecOf<TIn>::T2;          // 16-byte vector of TIn
  constexpr int NT = WGM * WGN * 64;
  constexpr int VEC = 16 / sizeof(TIn);         // elements per 16-byte vector
  constexpr int BK = 128 / sizeof(TIn);         // one 128-byte row segment per chunk
  constexpr int KL = BK / 4;                    // contiguous k per lane group per chunk
  constexpr int STEPS = KL / MF::kPerLane;      // MFMAs per 16x16 tile per chunk
  constexpr int WTM = BM / WGM, WTN = BN / WGN; // wave tile
  constexpr int TM = WTM / 16, TN = WTN / 16;   // MFMA tiles per wave
  // LDS: A as [row][k]; B as [k][n] (row-major B) or [n][k] (BKMAJOR).
  constexpr int LDA_S = BK + VEC;
  constexpr int LDB_S = BKMAJOR ? (BK + VEC) : (BN + VEC);
  constexpr int B_ELEMS = BKMAJOR ? BN * LDB_S : BK * LDB_S;
  constexpr int VPR = BK / VEC;                 // vectors per k segment of one A row
  constexpr int A_ITERS = BM * VPR / NT;
  constexpr int B_VPL = BKMAJOR ? VPR : BN / VEC;   // vectors per stored B line
  constexpr int B_ITERS = (BKMAJOR ? BN * VPR : BK * (BN / VEC)) / NT;
  static_assert(A_ITERS * NT == BM * VPR, "A tile load must divide evenly");
  static_assert(B_ITERS * NT == (BKMAJOR ? BN * VPR : BK * (BN / VEC)), "B tile load must divide evenly");
  static_assert(BKMAJOR || MF::kPerLane == 1, "row-major B needs a one-k-per-lane instruction");
  // With both operands k-contiguous the MFMA can take them in either order;
  // taking B first accumulates the tile of C^T, whose lane layout lets the
  // epilogue move binary32 C in 16-byte vectors.
  constexpr bool SWAP = BKMAJOR && (MF::kPerLane > 1) && std::is_same<Acc, float>::value;

  __shared__ __attribute__((aligned(16))) TIn As[2][BM * LDA_S];
  __shared__ __attribute__((aligned(16))) TIn Bs[2][B_ELEMS];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int gi = lane & 15, g = lane >> 4;

  // ---- batch offsets --------------------------------------------------
  const int zo = z / p.zdiv, zi = z % p.zdiv;
  const TIn* __restrict__ A = p.A + zo * p.sa_o + zi * p.sa_i;
  const TIn* __restrict__ B = p.B + zo * p.sb_o + zi * p.sb_i;
  const int M = p.M, N = p.N, K = p.K;
  const int64_t lda = p.lda, ldb = p.ldb;

  const bool a_lower = p.flags & G_A_LOWER;
  const bool b_lower = p.flags & G_B_LOWER;
  int kbeg;
  int nchunks = chunk_range<BM, BK>(K, p.flags, r0, c0, kbeg);
  nchunks = split_range<BK>(K, s, p.ksplit, nchunks, kbeg);

  Out acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = Acc(0);

  // ---- global -> register staging (no per-lane branches) -------------------
  V16 ra[A_ITERS], rb[B_ITERS];

  auto load_a = [&](int k0) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(A + (int64_t)r0 * lda + k0);
#pragma unroll
    for (int it = 0; it < A_ITERS; ++it) {
      const int idx = tid + it * NT;
      const int row = idx / VPR, kv = (idx % VPR) * VEC;
      const int gr = r0 + row, gk = k0 + kv;
      V16 v;
      if constexpr (ALIGNED) {
        const bool ok = gr < M && gk < K;
        v = buf_load16<V16>(rs, ok ? (int)((row * lda + kv) * (int64_t)sizeof(TIn)) : kBufOOB);
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const bool ok = gr < M && gk + e < K;
          const TIn x = A[ok ? (int64_t)gr * lda + gk + e : 0];
          v[e] = ok ? x : TIn(0);
        }
      }
      ra[it] = v;
    }
  };
  auto load_b = [&](int k0) {
#pragma unroll
    for (int it = 0; it < B_ITERS; ++it) {
      const int idx = tid + it * NT;
      V16 v;
      if constexpr (BKMAJOR) {
        // B stored N x K: a stored row is a column of B.
        const int col = idx / VPR, kv = (idx % VPR) * VEC;
        const int gc = c0 + col, gk = k0 + kv;
        if constexpr (ALIGNED) {
          const __amdgpu_buffer_rsrc_t rs = make_rsrc(B + (int64_t)c0 * ldb + k0);
          const bool ok = gc < N && gk < K;
          v = buf_load16<V16>(rs, ok ? (int)((col * ldb + kv) * (int64_t)sizeof(TIn)) : kBufOOB);
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            const bool ok = gc < N && gk + e < K;
            const TIn x = B[ok ? (int64_t)gc * ldb + gk + e : 0];
            v[e] = ok ? x : TIn(0);
          }
        }
      } else {
        // B stored K x N: BK rows of BN/VEC vectors.
        const int krow = idx / B_VPL, cv = (idx % B_VPL) * VEC;
        const int gk = k0 + krow, gc = c0 + cv;
        if constexpr (ALIGNED) {
          const __amdgpu_buffer_rsrc_t rs = make_rsrc(B + (int64_t)k0 * ldb + c0);
          const bool ok = gk < K && gc < N;
          v = buf_load16<V16>(rs, ok ? (int)((krow * ldb + cv) * (int64_t)sizeof(TIn)) : kBufOOB);
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            const bool ok = gk < K && gc + e < N;
            const TIn x = B[ok ? (int64_t)gk * ldb + gc + e : 0];
            v[e] = ok ? x : TIn(0);
          }
        }
      }
      rb[it] = v;
    }
  };
  // Triangular masks are applied when the staged data is written to LDS, so
  // that the global loads of the next chunk stay in flight during the MFMAs.
  auto store_ab = [&](int buf, int k0) {
#pragma unroll
    for (int it = 0; it < A_ITERS; ++it) {
      const int idx = tid + it * NT;
      const int row = idx / VPR, kv = (idx % VPR) * VEC;
      V16 v = ra[it];
      if (a_lower) {
        const int gr = r0 + row, gk = k0 + kv;
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = (gk + e > gr) ? TIn(0) : v[e];
      }
      *reinterpret_cast<V16*>(&As[buf][row * LDA_S + kv]) = v;
    }
#pragma unroll
    for (int it = 0; it < B_ITERS; ++it) {
      const int idx = tid + it * NT;
      const int line = idx / B_VPL, vo = (idx % B_VPL) * VEC;
      V16 v = rb[it];
      if (b_lower) {
        // BKMAJOR: line = column, vo = k offset; else line = k row, vo = column offset
        const int gc = c0 + (BKMAJOR ? line : vo), gk = k0 + (BKMAJOR ? vo : line);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const bool zero = BKMAJOR ? (gk + e < gc) : (gk < gc + e);
          v[e] = zero ? TIn(0) : v[e];
        }
      }
      *reinterpret_cast<V16*>(&Bs[buf][line * LDB_S + vo]) = v;
    }
  };

  // ---- main loop --------------------------------------------------------
  if (nchunks > 0) {
    load_a(kbeg);
    load_b(kbeg);
    store_ab(0, kbeg);
    __syncthreads();
    for (int c = 0; c < nchunks; ++c) {
      const int buf = c & 1;
      const bool more = c + 1 < nchunks;
      if (more) {
        load_a(kbeg + (c + 1) * BK);
        load_b(kbeg + (c + 1) * BK);
      }
      const TIn* as = As[buf];
      const TIn* bs = Bs[buf];
#pragma unroll
      for (int s = 0; s < STEPS; ++s) {
        // lane group g feeds k = g*KL + s*kPerLane ... + kPerLane - 1
        const int kk = g * KL + s * MF::kPerLane;
        typename MF::Frag fa[TM], fb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
          fa[i] = *reinterpret_cast<const typename MF::Frag*>(&as[(wm * WTM + i * 16 + gi) * LDA_S + kk]);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if constexpr (BKMAJOR)
            fb[j] = *reinterpret_cast<const typename MF::Frag*>(&bs[(wn * WTN + j * 16 + gi) * LDB_S + kk]);
          else
            fb[j] = bs[kk * LDB_S + wn * WTN + j * 16 + gi];
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = SWAP ? MF::mma(fb[j], fa[i], acc[i][j]) : MF::mma(fa[i], fb[j], acc[i][j]);
      }
      if (more) store_ab(buf ^ 1, kbeg + (c + 1) * BK);
      __syncthreads();
    }
  }

  if constexpr (SWAP)
    gemm_epilogue_t<TIn, TCin, TCout, TC2, TM, TN, WTM, WTN>(p, acc, zo, zi, z, s, r0, c0, wm, wn,
                                                            g, gi);
  else
    gemm_epilogue<TIn, TCin, TCout, TC2, TM, TN, WTM, WTN>(p, acc, zo, zi, z, s, r0, c0, wm, wn, g,
                                                          gi);
}


// The output tiles of workgroup `bid` (of nwg) of one batch entry z: one
// tile, or two for a folded triangular product.  smem: tile_lds bytes.
template <typename TIn, int BM, int BN, bool BKMAJOR, int MODE>
constexpr int tile_lds() {
  return MODE != kStaged && Mfma<TIn>::kPerLane == 1 ? dma_lds<TIn, BM, BN, BKMAJOR>() : 16;
}

template <typename TIn, typename TCin, typename TCout, typename TC2,
          int BM, int BN, int WGM, int WGN, bool BKMAJOR, int MODE, bool CLOWER = false,
          int DIR = kByFlags, int GROUP_M = 8, bool XCD_REMAP = false>
__device__ __forceinline__ void gemm_tile(const GemmParams<TIn, TCin, TCout, TC2>& p, int z,
                                          int s, int bid, int nwg, char* smem) {
  const int ntm = (p.M + BM - 1) / BM, ntn = (p.N + BN - 1) / BN;
  auto one = [&](int tm, int tn) {
    if constexpr (MODE != kStaged && Mfma<TIn>::kPerLane == 1)
      gemm_tile_dma<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, MODE != kDma4, MODE == kDma16,
                    true, DIR>(p, z, s, tm * BM, tn * BN, smem);
    else
      gemm_tile_staged<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, MODE == kDma16>(
          p, z, s, tm * BM, tn * BN);
  };
  if constexpr (CLOWER) {
    int tm, tn;
    lower_tile(ntm, bid, nwg, tm, tn);
    one(tm, tn);
    return;
  }
  const bool fold = tri_fold(p.M, p.K, p.flags, BM);
  const bool uniform = fold || !(p.flags & (G_A_LOWER | G_B_LOWER | G_A_UPPER));
  const int rows = fold ? (ntm + 1) / 2 : ntm;
  int slot, tn;
  tile_slot<GROUP_M, XCD_REMAP>(rows, ntn, uniform, bid, nwg, slot, tn);
  one(slot, tn);
  if (fold && ntm - 1 - slot != slot) {
    __syncthreads();   // the second tile reuses the LDS stages
    one(ntm - 1 - slot, tn);
  }
}

// Small products straight from global memory to registers: one wave computes a
// 16 x 16 tile, four waves a workgroup.  KW = 1: the waves take a 2 x 2 group of
// tiles and share operand rows in the unit's cache; KW = 4: they take the
// quarters of K of one tile, summed in a fixed order through LDS.  Such a
// product is bound by its chain, not by its work: no staging, no barrier per
// chunk, the loads of 32 (binary64) or 64 (binary32) k in flight while the previous
// ones multiply, and four times as many workgroups as 64 x 64 tiles.  VEC16:
// operands with contiguous k are read 16 bytes at a time (aligned); otherwise
// one element at a time, any alignment.  K runs towards the diagonal as in
// gemm_tile_dma: U X = B, 3001 x 500 in binary32, relative error 7.0e-8 and 110.9 us,
// upwards 2.9e-7 and 108.3; with a step's elements in reverse too 6.3e-8, but
// choosing their order at run time costs up to half of the speed (4096 x 8 in binary64:
// 49.5 us for 31.4).  Triangles are skipped and masked per
// 16 x 16 tile.  C must not overlap A or B, but for the strips: kRowStrip
// (kColStrip), for products of at most 64 columns (rows), gives a workgroup 16 rows
// (columns) of C in full, and its waves have read all they need of A (B) before the
// first of them writes, so C may be A (B) itself.
constexpr int kRowStrip = -1, kColStrip = -2;

template <typename TIn, typename TCin, typename TCout, typename TC2, bool BKMAJOR, bool VEC16,
          int KW>
__device__ __forceinline__ void gemm_direct_tile(const GemmParams<TIn, TCin, TCout, TC2>& p,
                                                 int bid, int z) {
  using MF = Mfma<TIn>;
  using Out = typename MF::Out;
  using V16 = typename VecOf<TIn>::T2;
  constexpr int VEC = 16 / (int)sizeof(TIn);   // k per lane and step
  constexpr int SK = 4 * VEC;                  // k per step of the wave
  constexpr int U = 4;                         // steps in flight
  static_assert(MF::kPerLane == 1, "one k per lane and instruction");
  const int lane = threadIdx.x & 63, gi = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int zo = z / p.zdiv, zi = z % p.zdiv;
  const int M = p.M, N = p.N, K = p.K;
  const int ntn = (N + 15) / 16, ntm = (M + 15) / 16;
  int tm, tn;
  if (KW == 1) {
    const int gn = (ntn + 1) / 2;
    tm = 2 * (bid / gn) + (wave >> 1);
    tn = 2 * (bid % gn) + (wave & 1);
  } else if (KW < 0) {
    tm = KW == kRowStrip ? bid : wave;
    tn = KW == kRowStrip ? wave : bid;
  } else {
    tm = bid / ntn;
    tn = bid % ntn;
  }
  const bool idle = KW < 0 && (tm >= ntm || tn >= ntn);   // still has to meet the others
  const bool c_lower = p.flags & G_C_LOWER;
  if (KW == 1 && (tm >= ntm || tn >= ntn || (c_lower && tn > tm))) return;
  if (KW > 1 && c_lower && tn > tm) return;
  const int r0 = tm * 16, c0 = tn * 16;
  const bool a_mask = (p.flags & G_A_LOWER) && !(p.flags & G_A_ZERO_UPPER);
  const bool b_mask = p.flags & G_B_LOWER;
  int kend = K, kbeg = 0;
  if (p.flags & G_A_LOWER) kend = min(K, r0 + 16);
  if (p.flags & G_A_UPPER) kbeg = min(r0, K) / SK * SK;
  if (p.flags & G_B_LOWER) kbeg = min(c0, K) / SK * SK;
  int steps = kend > kbeg && !idle ? (kend - kbeg + SK - 1) / SK : 0;
  const bool down = p.flags & G_A_UPPER;
  const int gk = down ? 3 - g : g;             // an instruction adds its lane groups in turn
  if (KW > 1) {
    // the quarters in the order of the sum: the diagonal's is the last
    const int per = (steps + KW - 1) / KW, first = (down ? KW - 1 - wave : wave) * per;
    kbeg += min(first, steps) * SK;
    steps = max(0, min(per, steps - first));
  }
  const int row = min(r0 + gi, M - 1), col = min(c0 + gi, N - 1);
  const TIn* __restrict__ A = p.A + zo * p.sa_o + zi * p.sa_i + (int64_t)row * p.lda;
  const TIn* __restrict__ B = p.B + zo * p.sb_o + zi * p.sb_i +
                              (BKMAJOR ? (int64_t)col * p.ldb : (int64_t)col);
  struct Step {
    TIn a[VEC], b[VEC];
  };
  // the lane group's VEC consecutive k of one step
  auto load = [&](Step& f, int k0) {
    const int k = k0 + gk * VEC;
    if (k0 + SK <= K) {
      if (VEC16) {
        const V16 v = *reinterpret_cast<const V16*>(A + k);
#pragma unroll
        for (int e = 0; e < VEC; ++e) f.a[e] = v[e];
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) f.a[e] = A[k + e];
      }
      if (BKMAJOR && VEC16) {
        const V16 v = *reinterpret_cast<const V16*>(B + k);
#pragma unroll
        for (int e = 0; e < VEC; ++e) f.b[e] = v[e];
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) f.b[e] = BKMAJOR ? B[k + e] : B[(int64_t)(k + e) * p.ldb];
      }
    } else {   // the last, partial step: zeros past K
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const bool ok = k + e < K;
        const int64_t q = ok ? k + e : 0;
        const TIn va = A[q], vb = BKMAJOR ? B[q] : B[q * p.ldb];
        f.a[e] = ok ? va : TIn(0);
        f.b[e] = ok ? vb : TIn(0);
      }
    }
  };
  auto mask = [&](Step& f, int k0) {
    const int k = k0 + gk * VEC;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      if (a_mask && k + e > r0 + gi) f.a[e] = TIn(0);
      if (b_mask && k + e < c0 + gi) f.b[e] = TIn(0);
    }
  };
  Out acc[1][1] = {};
  Step f[U];
  const int kfirst = down ? kbeg + (steps - 1) * SK : kbeg, kstep = down ? -SK : SK;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < steps) load(f[u], kfirst + u * kstep);
  for (int t = 0; t < steps; t += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (t + u < steps) {
        const int k0 = kfirst + (t + u) * kstep;
        if (a_mask || b_mask) mask(f[u], k0);
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[0][0] = MF::mma(f[u].a[e], f[u].b[e], acc[0][0]);
        if (t + u + U < steps) load(f[u], k0 + U * kstep);
      }
    }
  }
  if (KW > 1) {
    __shared__ typename MF::Acc part[KW > 1 ? KW - 1 : 1][64][4];
    if (wave > 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave - 1][lane][r] = acc[0][0][r];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w + 1 < KW; ++w)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[0][0][r] += part[w][lane][r];
  }
  if (KW < 0) {
    __syncthreads();
    if (idle) return;
  }
  gemm_epilogue<TIn, TCin, TCout, TC2, 1, 1, 16, 16>(p, acc, zo, zi, z, 0, r0, c0, 0, 0, g, gi);
}

template <typename TIn, typename TCin, typename TCout, typename TC2, bool BKMAJOR, bool VEC16,
          int KW>
__global__ __launch_bounds__(256) void gemm_direct_kernel(GemmParams<TIn, TCin, TCout, TC2> p) {
  gemm_direct_tile<TIn, TCin, TCout, TC2, BKMAJOR, VEC16, KW>(p, blockIdx.x, blockIdx.z);
}

// Two independent products in one launch, the first in workgroups [0, first): chains
// of small products (a factorization's diagonal block) are bound by the number of
// launches, 4.6 us each on an idle card and 12 us beside large products.
template <typename T, bool VEC16, int KW0, int KW1>
__global__ __launch_bounds__(256) void gemm_direct_pair_kernel(GemmParams<T, T, T, float> p0,
                                                               GemmParams<T, T, T, float> p1,
                                                               int first) {
  const int bid = blockIdx.x;
  if constexpr (KW0 == KW1) {
    gemm_direct_tile<T, T, T, float, false, VEC16, KW0>(bid < first ? p0 : p1,
                                                       bid < first ? bid : bid - first, 0);
  } else {
    if (bid < first) gemm_direct_tile<T, T, T, float, false, VEC16, KW0>(p0, bid, 0);
    else gemm_direct_tile<T, T, T, float, false, VEC16, KW1>(p1, bid - first, 0);
  }
}

template <typename TIn, typename TCin, typename TCout, typename TC2,
          int BM, int BN, int WGM, int WGN, bool BKMAJOR, int MODE, bool CLOWER = false,
          int DIR = kByFlags>
__global__ __launch_bounds__(WGM * WGN * 64, 2)
void gemm_kernel(GemmParams<TIn, TCin, TCout, TC2> p) {
  __shared__ __attribute__((aligned(1024))) char smem[tile_lds<TIn, BM, BN, BKMAJOR, MODE>()];
  gemm_tile<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, MODE, CLOWER, DIR>(
      p, blockIdx.z, blockIdx.y, blockIdx.x, gridDim.x, smem);
}

// As gemm_direct_pair_kernel, in 64 x 64 tiles of aligned operands.
template <typename T>
__global__ __launch_bounds__(256, 2) void gemm_pair_kernel(GemmParams<T, T, T, float> p0,
                                                           GemmParams<T, T, T, float> p1,
                                                           int first) {
  const int bid = blockIdx.x;
  // (two copies of the code: a reference chosen at run time puts both structures into
  // private memory, 67 us instead of 38 for the panels of 7168 rows)
  __shared__ __attribute__((aligned(1024))) char smem[dma_lds<T, 64, 64, false>()];
  if (bid < first)
    gemm_tile<T, T, T, float, 64, 64, 2, 2, false, kDma16>(p0, 0, 0, bid, first, smem);
  else
    gemm_tile<T, T, T, float, 64, 64, 2, 2, false, kDma16>(p1, 0, 0, bid - first,
                                                          (int)gridDim.x - first, smem);
}

// Split-K finish: the fixed-order sum of the ksplit partial products of
// every element (towards the diagonal, as in the tiles), then the usual epilogue
// (deterministic: the order of the sum never depends on scheduling).
template <typename TIn, typename TCin, typename TCout, typename TC2>
__global__ __launch_bounds__(256) void gemm_splitk_finish(GemmParams<TIn, TCin, TCout, TC2> p,
                                                          int batch) {
  using Acc = typename Mfma<TIn>::Acc;
  using Epi = EpiType<TIn, TCin, TCout>;
  const int64_t MN = (int64_t)p.M * p.N, total = MN * batch;
  const bool use_rs = (p.flags & G_ROWSCALE) && p.rscale;
  Epi alpha = static_cast<Epi>(p.alpha);
  if (p.ascale) alpha *= static_cast<Epi>(*p.ascale);
  const Epi beta = static_cast<Epi>(p.beta);
  const Acc* __restrict__ P = static_cast<const Acc*>(p.part);
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int z = (int)(e / MN);
    const int64_t rc = e - z * MN;
    const int row = (int)(rc / p.N), col = (int)(rc - (int64_t)row * p.N);
    if ((p.flags & G_C_LOWER) && col > row) continue;
    const bool down = p.flags & G_A_UPPER;
    const Acc* q = P + ((int64_t)z * p.ksplit + (down ? p.ksplit - 1 : 0)) * MN + rc;
    const int64_t step = down ? -MN : MN;
    Acc v = q[0];
    for (int t = 1; t < p.ksplit; ++t) v += q[t * step];
    const int zo = z / p.zdiv, zi = z % p.zdiv;
    TCout* Co = p.Cout + zo * p.sco_o + zi * p.sco_i;
    const TCin* Ci = p.Cin ? p.Cin + zo * p.sci_o + zi * p.sci_i : nullptr;
    const Epi rs = use_rs ? static_cast<Epi>(p.rscale[(int64_t)row * p.ld_rs]) : Epi(1);
    epi_store(p, Co, Ci, row, col, static_cast<Epi>(v), alpha, beta, (p.flags & G_BETA) && Ci, rs);
  }
}

// Grouped launch: many independent products of one element type in one
// grid.  Entry e owns workgroups [tile_start[e], tile_start[e+1]); within an
// entry the workgroups cover ksplit x tiles (K slice, then tile).
template <typename TIn, typename TCin, typename TCout, typename TC2,
          int BM, int BN, int WGM, int WGN, bool BKMAJOR, int MODE, int DIR = kByFlags>
__global__ __launch_bounds__(WGM * WGN * 64, 2)
void gemm_grouped_kernel(const GemmParams<TIn, TCin, TCout, TC2>* __restrict__ entries,
                         const int* __restrict__ tile_start, int nentries) {
  const int b = blockIdx.x;
  int lo = 0, hi = nentries - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tile_start[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  const GemmParams<TIn, TCin, TCout, TC2>& p = entries[lo];
  const int tiles = gemm_wgs(p.M, p.N, p.K, p.flags, BM, BN);
  const int local = b - tile_start[lo];
  __shared__ __attribute__((aligned(1024))) char smem[tile_lds<TIn, BM, BN, BKMAJOR, MODE>()];
  gemm_tile<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, MODE, false, DIR>(
      p, 0, local / tiles, local % tiles, tiles, smem);
}

// How a product's operands reach LDS.  Binary64/binary32: kDma16 if the rows of both
// are 16-byte aligned, kDma16A if those of A are (batches: A is a packed inverted
// block, B has the caller's leading dimension), else kDma4; kStaged only where a
// tile's rows span more than a buffer descriptor.  Other types: kDma16 for the
// 16-byte staged path, else kStaged.
template <typename TIn, int BM, int BN, bool BKMAJOR, typename P>
inline int gemm_mode(const P& p) {
  constexpr int VEC = 16 / sizeof(TIn);
  constexpr int BK = 128 / sizeof(TIn);
  auto al = [](const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15) == 0; };
  const int64_t span_a = (int64_t)BM * p.lda * (int64_t)sizeof(TIn);
  const int64_t span_b = (int64_t)(BKMAJOR ? BN : BK) * p.ldb * (int64_t)sizeof(TIn);
  if (span_a >= kBufOOB || span_b >= kBufOOB) return kStaged;
  const bool a = al(p.A) && p.lda % VEC == 0 && p.sa_o % VEC == 0 && p.sa_i % VEC == 0;
  const bool b = al(p.B) && p.ldb % VEC == 0 && p.sb_o % VEC == 0 && p.sb_i % VEC == 0;
  if (a && b && p.K % VEC == 0 && (BKMAJOR || p.N % VEC == 0)) return kDma16;
  if constexpr (Mfma<TIn>::kPerLane == 1) {
    // K need not be a multiple of the piece: the last piece of a row then holds an
    // element of A (it stays inside that 16-byte granule) and its rest is masked
    if (a && !BKMAJOR) return kDma16A;
    return kDma4;
  }
  return kStaged;
}

// Split-K policy: products with at most half of `target` workgroups split K into
// S slices (each at least kSplitMinChunks chunks) so that at most `target`
// workgroups run, as far as the scratch in p.part holds the partial products.
// Without scratch (p.part null) nothing is split.  The target is kSplitTarget,
// two 128 x 128 workgroups per compute unit.
constexpr int kSplitTarget = 512;
constexpr int kSplitMinChunks = 4;
constexpr int kSplitMax = 16;
template <typename TIn, typename P>
inline int gemm_ksplit(const P& p, int64_t wgs, int batch, int target) {
  if (!p.part || 2 * wgs > target) return 1;
  constexpr int BK = 128 / sizeof(TIn);
  const int64_t nck = (p.K + BK - 1) / BK;
  int64_t S = std::min<int64_t>(target / wgs, nck / kSplitMinChunks);
  S = std::min<int64_t>(S, kSplitMax);
  const int64_t per = (int64_t)p.M * p.N * batch * (int64_t)sizeof(typename Mfma<TIn>::Acc);
  if (per > 0) S = std::min<int64_t>(S, p.part_bytes / per);
  return S > 1 ? (int)S : 1;
}

// Whether a small binary64/binary32 product takes gemm_direct_kernel.  Its rate
// is that of the caches, about 10.7 (binary64) or 20 (binary32) 16x16x4 matrix
// instructions per ns however they are spread, after about 3.5 us; a 64 x 64
// tile takes 4 us and about 0.7 us per 128 bytes of K (binary32: 0.4 us per 16
// k) however few tiles there are, or, split over K, 13 us with its finish pass
// and then 23 instructions per ns.  The line lies where the two meet.  Measured
// direct / 64 x 64 (best of split and not), binary64: 128^3 triangular 3.7 /
// 12.9 us, 512^3 triangular 10.7 / 19.8, 1024 x 128 x 1024 triangular 12.0 /
// 18.9, 3968 x 128 x 128 9.5 / 10.1, 2048 x 128 x 1024 26.5 / 24.8, 1024 x 1024 x
// 128 15.6 / 11.0.  With one wave a tile (more than 2048 tiles: launch_direct) the rate
// is half of that, so that near the line the 64 x 64 tiles would be ahead: three 512^3
// triangular products, right on it, take 38 us.  C may be neither A nor B: another
// workgroup would read what one has overwritten.
template <typename TIn, typename P>
inline bool direct_ok(const P& p, int batch) {
  if ((const void*)p.Cout == (const void*)p.A || (const void*)p.Cout == (const void*)p.B)
    return false;
  int64_t tiles = (int64_t)((p.M + 15) / 16) * ((p.N + 15) / 16) * batch;
  int64_t steps = (p.K + 3) / 4;
  if (p.flags & G_C_LOWER) tiles = (tiles + 1) / 2;
  if (((p.flags & (G_A_LOWER | G_A_UPPER)) && p.M == p.K) ||
      ((p.flags & G_B_LOWER) && p.N == p.K))
    steps = (steps + 1) / 2;
  const int64_t most = sizeof(TIn) == 8 ? 192 * 1024 : 256 * 1024;
  return tiles * steps <= std::min<int64_t>(most, (int64_t)512 * p.K);
}

// Whether a direct product's operands with contiguous k can be read 16 bytes at a time.
template <typename TIn, bool BKMAJOR, typename P>
inline bool direct_vec(const P& p) {
  constexpr int VEC = 16 / (int)sizeof(TIn);
  auto al = [](const void* x) { return (reinterpret_cast<uintptr_t>(x) & 15) == 0; };
  return al(p.A) && p.lda % VEC == 0 && p.sa_o % VEC == 0 && p.sa_i % VEC == 0 &&
         (!BKMAJOR || (al(p.B) && p.ldb % VEC == 0 && p.sb_o % VEC == 0 && p.sb_i % VEC == 0));
}

// Launch of gemm_direct_kernel (the caller has checked direct_ok).  K is split
// over a workgroup's waves unless there are many tiles or hardly any steps.
template <typename TIn, typename TCin, typename TCout, typename TC2, bool BKMAJOR>
inline hipError_t launch_direct(const GemmParams<TIn, TCin, TCout, TC2>& p, int batch,
                                hipStream_t stream) {
  GemmParams<TIn, TCin, TCout, TC2> q = p;
  q.ksplit = 1;
  const unsigned ntm = (unsigned)((p.M + 15) / 16), ntn = (unsigned)((p.N + 15) / 16);
  const int kw = (int64_t)ntm * ntn * batch > 2048 || p.K * (int)sizeof(TIn) < 512 ? 1 : 4;
  const dim3 grid(kw == 1 ? ((ntm + 1) / 2) * ((ntn + 1) / 2) : ntm * ntn, 1, (unsigned)batch);
  const bool vec = direct_vec<TIn, BKMAJOR>(p);
  auto go = [&](auto kernel) { kernel<<<grid, 256, 0, stream>>>(q); };
  if (kw == 1) {
    if (vec) go(gemm_direct_kernel<TIn, TCin, TCout, TC2, BKMAJOR, true, 1>);
    else go(gemm_direct_kernel<TIn, TCin, TCout, TC2, BKMAJOR, false, 1>);
  } else {
    if (vec) go(gemm_direct_kernel<TIn, TCin, TCout, TC2, BKMAJOR, true, 4>);
    else go(gemm_direct_kernel<TIn, TCin, TCout, TC2, BKMAJOR, false, 4>);
  }
  return hipGetLastError();
}

// K slices of a product of `wgs` 64 x 64 tiles on the direct-to-LDS path: the S
// with the least modelled time.  A chunk (128 bytes of K) takes about 0.70 us
// (binary64) or 0.9 us (binary32) a workgroup per compute unit, one or several on
// it, so the tiles take as long as the fullest of 256 units; the finish pass
// of a split takes 4 us and reads and writes S + 2 times C at 3 TB/s.  Measured at
// N = 128, K = 1024, binary64: 480 workgroups (M = 15360) 89 us unsplit and 95 in
// two, 256 (8192) 49 and 54, 64 (2048) 45 and, in eight, 25.  With one column tile no
// neighbour brings A's rows into the cache: a chunk then takes 1.0 us alone on its unit,
// 0.6 each beside others.
//
// Folded triangles: a workgroup's two tiles have nck + 4 chunks together, but a slice of
// K cuts both of them in the lower half and one in the upper, so the longest slice
// has twice the mean.  It sets the time of few slices (0.7 us a chunk); many
// slices run at 0.6 us a chunk and unit and leave a quarter of the longest over.
// n = 8192 by 8 columns, binary64 (S = 1, 4, 8, 16): 360, 185, 121, 99 us; 4096 by 300:
// 170, 155, 128, 130; 2048 by 400: 90, 66, 59, 65.
template <typename TIn, typename P>
inline int chain_ksplit(const P& p, int64_t wgs, int batch) {
  if (!p.part) return 1;
  constexpr int BK = 128 / sizeof(TIn);
  const int64_t nck = (p.K + BK - 1) / BK;
  const int64_t per = (int64_t)p.M * p.N * batch * (int64_t)sizeof(typename Mfma<TIn>::Acc);
  const bool fold = tri_fold(p.M, p.K, p.flags, 64);
  const double alone = p.N <= 64 ? 1.0 : sizeof(TIn) == 8 ? 0.70 : 0.9;
  const double each = p.N <= 64 ? 0.6 : alone;
  int best = 1;
  double least = 1e300;
  for (int64_t S = 1; S <= kSplitMax; ++S) {
    if (S > 1 && (nck / S < kSplitMinChunks || S * per > p.part_bytes)) break;
    const double cps = (double)((nck + S - 1) / S);
    double t;
    if (fold) {
      const double longest = 0.7 * (S > 1 ? std::min(2 * cps, (double)nck + 4) : (double)nck + 4);
      t = std::max(longest, 0.6 * (double)(wgs * (nck + 4)) / 256 + longest / 4);
    } else {
      const int64_t on_unit = (wgs * S + 255) / 256;
      t = cps * std::max(alone, (double)on_unit * each);
    }
    if (S > 1) t += 4.0 + (double)(S + 2) * (double)per / (fold ? 8e6 : 3e6);
    if (t < least) {
      least = t;
      best = (int)S;
    }
  }
  return best;
}

// Tile of a binary64/binary32 product: 64 x 64 (else 128 x 128) below two 128 x 128
// workgroups per compute unit, and for short K: a 128 x 128 workgroup's first
// copies and its stores of C run beside one other workgroup, those of the 64 x 64
// tiles beside three or four.  From K = 1024 (binary64) or 2048 (binary32) the
// large tiles' fewer LDS reads count for more.  8192 x 8192 x K, 64 / 128 tiles, us:
// binary64 K = 128 434 / 592, 512 1183 / 1204, 1024 2195 / 2112; binary32 128
// 278 / 435, 512 633 / 773, 1024 1113 / 1194, 2048 2125 / 2149, 4096 4144 / 4119.
template <typename TIn, typename P>
inline bool small_tile(const P& p, int batch) {
  return gemm_wgs(p.M, p.N, p.K, p.flags, 128, 128) * (int64_t)batch < kSplitTarget ||
         p.K <= (sizeof(TIn) == 8 ? 512 : 1024);
}

// Host-side launch helper.
template <typename TIn, typename TCin, typename TCout, typename TC2,
          int BM, int BN, int WGM, int WGN, bool BKMAJOR>
inline hipError_t launch_gemm(const GemmParams<TIn, TCin, TCout, TC2>& p, int batch,
                              hipStream_t stream) {
  if (p.M <= 0 || p.N <= 0 || batch <= 0) return hipSuccess;
  if ((p.flags & G_C_LOWER) && (p.M != p.N || BM != BN)) return hipErrorInvalidValue;
  if constexpr (BM == 64 && BN == 64 && Mfma<TIn>::kPerLane == 1) {
    if (direct_ok<TIn>(p, batch))
      return launch_direct<TIn, TCin, TCout, TC2, BKMAJOR>(p, batch, stream);
  }
  const int mode = gemm_mode<TIn, BM, BN, BKMAJOR>(p);
  constexpr bool kDirect = Mfma<TIn>::kPerLane == 1;
  // operands that are not 16-byte aligned take 64 x 64 tiles: a large tile's 4-byte
  // copies of two chunks would exceed the counter of outstanding copies, and
  // staged through registers it is slower at every size (gemm_tile_dma)
  if constexpr (kDirect && BM * BN > 64 * 64) {
    if (mode != kDma16 && mode != kStaged)
      return launch_gemm<TIn, TCin, TCout, TC2, 64, 64, 2, 2, BKMAJOR>(p, batch, stream);
  }
  const int64_t tiles = gemm_wgs(p.M, p.N, p.K, p.flags, BM, BN);
  GemmParams<TIn, TCin, TCout, TC2> q = p;
  // one round of workgroups: two per compute unit for the 128 x 128 tiles,
  // four for the smaller ones (their registers and LDS allow it)
  const int target = (BM * BN >= 128 * 128) ? kSplitTarget : 2 * kSplitTarget;
  const bool chain = BM * BN < 128 * 128 && kDirect && mode != kStaged;
  q.ksplit = chain ? chain_ksplit<TIn>(p, tiles * batch, batch)
                   : gemm_ksplit<TIn>(p, tiles * batch, batch, target);
  // lower-triangle products take their own instantiation (tile enumeration)
  const bool clower = p.flags & G_C_LOWER;
  dim3 grid((unsigned)tiles, (unsigned)q.ksplit, (unsigned)batch);
  dim3 block(WGM * WGN * 64);
  auto go = [&](auto kernel) { kernel<<<grid, block, 0, stream>>>(q); };
  // one for each direction of K: chosen at run time it costs binary32 1 % (16384 x
  // 16384 by 2048: 4850 and 4900 us)
  constexpr int kDirUp = kDirect ? kUp : kByFlags, kDirDown = kDirect ? kDown : kByFlags;
  if (mode == kDma16) {
    if (clower)
      go(gemm_kernel<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, kDma16, true, kDirUp>);
    else if (kDirect && (p.flags & G_A_UPPER))
      go(gemm_kernel<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, kDma16, false, kDirDown>);
    else
      go(gemm_kernel<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, kDma16, false, kDirUp>);
  } else if (mode == kStaged) {
    if (clower) go(gemm_kernel<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, kStaged, true>);
    else go(gemm_kernel<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, kStaged>);
  } else if constexpr (kDirect && BM == 64 && BN == 64) {
    if (clower) go(gemm_kernel<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, kDma4, true>);
    else go(gemm_kernel<TIn, TCin, TCout, TC2, BM, BN, WGM, WGN, BKMAJOR, kDma4>);
  }
  if (q.ksplit > 1) {
    const int64_t total = (int64_t)p.M * p.N * batch;
    const unsigned g = (unsigned)std::min<int64_t>((total + 255) / 256, 4096);
    gemm_splitk_finish<TIn, TCin, TCout, TC2><<<g, 256, 0, stream>>>(q, batch);
  }
  return hipGetLastError();
}

template <typename TIn, typename TCin, typename TCout, typename TC2>
inline GemmParams<TIn, TCin, TCout, TC2> gemm_params() {
  GemmParams<TIn, TCin, TCout, TC2> p{};
  p.zdiv = 1;
  p.alpha = 1.0;
  p.beta = 0.0;
  p.c2scale = 1.0f;
  return p;
}

// Two independent products without a split, in one launch where both have the same
// form (small: 16 x 16 tiles; else 64 x 64 tiles of aligned operands) and otherwise one
// after the other.
template <typename T>
inline hipError_t launch_pair(const GemmParams<T, T, T, float>& p0,
                              const GemmParams<T, T, T, float>& p1, hipStream_t stream) {
  const bool same = p0.M > 0 && p0.N > 0 && p1.M > 0 && p1.N > 0;
  if (same && direct_ok<T>(p0, 1) && direct_ok<T>(p1, 1)) {
    auto tiles = [](const auto& p) { return ((p.M + 15) / 16) * ((p.N + 15) / 16); };
    const int n0 = tiles(p0), n1 = tiles(p1);
    const dim3 grid((unsigned)(n0 + n1));
    if (direct_vec<T, false>(p0) && direct_vec<T, false>(p1))
      gemm_direct_pair_kernel<T, true, 4, 4><<<grid, 256, 0, stream>>>(p0, p1, n0);
    else
      gemm_direct_pair_kernel<T, false, 4, 4><<<grid, 256, 0, stream>>>(p0, p1, n0);
    return hipGetLastError();
  }
  if (same && gemm_mode<T, 64, 64, false>(p0) == kDma16 &&
      gemm_mode<T, 64, 64, false>(p1) == kDma16) {
    GemmParams<T, T, T, float> q0 = p0, q1 = p1;
    q0.ksplit = q1.ksplit = 1;
    const int n0 = gemm_wgs(p0.M, p0.N, p0.K, p0.flags, 64, 64);
    const int n1 = gemm_wgs(p1.M, p1.N, p1.K, p1.flags, 64, 64);
    gemm_pair_kernel<T><<<(unsigned)(n0 + n1), 256, 0, stream>>>(q0, q1, n0);
    return hipGetLastError();
  }
  hipError_t e = launch_gemm<T, T, T, float, 64, 64, 2, 2, false>(p0, 1, stream);
  return e != hipSuccess ? e : launch_gemm<T, T, T, float, 64, 64, 2, 2, false>(p1, 1, stream);
}

// X = X B (at most 64 columns, p0: C = A) and Y = A Y (at most 64 rows, p1: C = B) in
// one launch.
template <typename T>
inline hipError_t launch_strips(const GemmParams<T, T, T, float>& p0,
                                const GemmParams<T, T, T, float>& p1, hipStream_t stream) {
  if (p0.N > 64 || p1.M > 64) return hipErrorInvalidValue;
  const int n0 = (p0.M + 15) / 16, n1 = (p1.N + 15) / 16;
  if (n0 + n1 == 0) return hipSuccess;
  const dim3 grid((unsigned)(n0 + n1));
  if (direct_vec<T, false>(p0) && direct_vec<T, false>(p1))
    gemm_direct_pair_kernel<T, true, kRowStrip, kColStrip><<<grid, 256, 0, stream>>>(p0, p1, n0);
  else
    gemm_direct_pair_kernel<T, false, kRowStrip, kColStrip><<<grid, 256, 0, stream>>>(p0, p1, n0);
  return hipGetLastError();
}

}  // namespace trsm
