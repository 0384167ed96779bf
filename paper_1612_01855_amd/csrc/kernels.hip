// Non-GEMM kernels of the gfx950 triangular solver: the LDS base case of the
// recursive triangular inversion, the substitution leaf of the recursive baseline, precision conversions and
// deterministic norm reductions.
#include "kernels.hpp"

#include <math.h>

#include "diag.hpp"

namespace trsm {

namespace {

// threads for a workgroup that walks one row of n0 elements
inline unsigned row_threads(int64_t n0) { return (unsigned)std::min<int64_t>(256, (n0 + 63) / 64 * 64); }

inline unsigned grid_for(int64_t work, int threads, int64_t cap = 1 << 20) {
  int64_t g = (work + threads - 1) / threads;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

// ---------------------------------------------------------------------------
// Alg. Diagonal-Inverter: every diagonal block S_b of L becomes a packed n0 x n0
// binary64 block of Linv, worked on in squares of ts = min(n0, 128) rows, one
// workgroup each.  An off-diagonal square of the lower triangle is copied.  A
// diagonal one is inverted in LDS, the base case of Alg. RecTriInv (4 x 4 blocks
// by substitution, then its combine for 4 to 64 rows on the matrix cores); zeros
// above its diagonal.
// Positions past row/column n hold the identity.  With `upper`, L is an
// upper-triangular U read transposed; with `unit` its diagonal is one.
// The first workgroup starts the status word.
// Measured: 8 us for one square of 64 rows and 15 for one of 128; extraction, a
// 64-row leaf by substitution and (128 rows) two combine launches took 44 and 58.
// All of n = 16384 in squares of 128: 21 us.
// ---------------------------------------------------------------------------
constexpr int kInvNt = kInvRows / 16;

// TS: the square's rows, or 0 for `small` of them (below kInvRows).
template <typename TL, int TS>
__global__ __launch_bounds__(kInvThreads) void block_inverse_kernel(
    const TL* __restrict__ L, int64_t ldl, int64_t n, int64_t n0, int small, int64_t m,
    double* __restrict__ Linv, unsigned long long* __restrict__ bad, bool upper, bool unit) {
  using namespace diag;
  using Map = LowerTiles;
  __shared__ __attribute__((aligned(16))) double S[Map::count(kInvNt) * kTile];
  const int ts = TS ? TS : small;
  // workgroups: the diagonal squares first (they take longest), then the others
  const int nt = (int)(n0 / ts), diagonals = (int)(m * nt), id = blockIdx.x, tid = threadIdx.x;
  int b, ti, tj;
  if (id < diagonals) {
    b = id / nt;
    ti = tj = id - b * nt;
  } else {
    const int per = nt * (nt - 1) / 2, e = id - diagonals;
    b = e / per;
    int q = e - b * per;
    ti = 1;
    while (q >= ti) q -= ti++;
    tj = q;
  }
  if (bad && id == 0 && tid == 0) *bad = ~0ull;
  const int64_t gr0 = b * n0 + (int64_t)ti * ts, gc0 = b * n0 + (int64_t)tj * ts;
  double* __restrict__ out = Linv + b * n0 * n0 + (int64_t)ti * ts * n0 + (int64_t)tj * ts;
  // A thread's elements: `fast` along L's rows in memory, `slow` = s0 + q ds.
  const SquareShare own = square_share(tid, ts);
  const int fast = own.fast, s0 = own.s0, ds = own.ds;
  constexpr int kEach = kInvRows * kInvRows / kInvThreads;
  const int64_t slow0 = upper ? gc0 : gr0, fast0 = upper ? gr0 : gc0;
  const int slows = (int)min((int64_t)ts, n - slow0), fasts = (int)min((int64_t)ts, n - fast0);
  const bool diagonal = ti == tj;
  // The slow indexes a thread reads, [lo, hi).  All its loads go out before the
  // first is used; a load outside is clamped to the square's first element (a
  // predicated load would be waited for before the next), and pointers advance by
  // a uniform step (a 64-bit product an element cost 36 instructions a load, more
  // than the memory's latency).
  const int lo = diagonal && !upper ? fast : 0;
  const int hi = fast >= fasts ? 0 : diagonal && upper ? min(slows, fast + 1) : slows;
  TL v[kEach];
  {
    const TL* __restrict__ first = L + (slows > 0 && fasts > 0 ? slow0 * ldl + fast0 : 0);
    const TL* __restrict__ p = first + ((int64_t)s0 * ldl + fast);
    const int64_t step = (int64_t)ds * ldl;
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
      const int slow = s0 + q * ds;
      v[q] = *(slow >= lo && slow < hi ? p + q * step : first);
    }
  }
  auto value = [&](int q) {
    const int slow = s0 + q * ds;
    const double x = slow < slows && fast < fasts ? static_cast<double>(v[q]) : 0.0;
    return diagonal && slow == fast && (unit || slow >= slows) ? 1.0 : x;
  };
  // tile row / column of slow index q, and the index inside it
  auto tile_of = [&](int q) { return TS ? q * (kInvThreads / kInvRows) / 16 : (s0 + q * ds) >> 4; };
  auto in_tile = [&](int q) {
    return TS ? s0 + q * (kInvThreads / kInvRows) % 16 : (s0 + q * ds) & 15;
  };
  if (!diagonal && !upper) {
#pragma unroll
    for (int q = 0; q < kEach; ++q) out[((int64_t)s0 * n0 + fast) + q * (ds * n0)] = value(q);
    return;
  }
  if (!diagonal) {
    // a transposed square goes through LDS, 64 of its columns at a time: it
    // came in along its columns and leaves along its rows (ts = kInvRows)
    constexpr int kHalf = kInvRows / 2, kLd = kHalf + 1;
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int q = 0; q < kEach; ++q)
        if (q / (kEach / 2) == h) S[fast * kLd + s0 + q * ds - h * kHalf] = value(q);
      __syncthreads();
#pragma unroll
      for (int e = 0; e < kEach / 2; ++e) {
        const int x = e * kInvThreads + tid;
        out[(int64_t)(x / kHalf) * n0 + h * kHalf + x % kHalf] = S[x / kHalf * kLd + x % kHalf];
      }
      __syncthreads();
    }
    return;
  }
  const int ntile = (ts + 15) / 16;
  if (ts < 16) {                        // a part of one tile: identity around it
    if (tid < 256) S[(tid >> 4) * kTld + (tid & 15)] = (tid >> 4) == (tid & 15) ? 1.0 : 0.0;
    __syncthreads();
  }
  const int ft = fast >> 4, fr = fast & 15;
  if (upper) {                          // column `slow` of row `fast`
    double* row = Map::at(S, ft, 0) + fr * kTld;
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
      const int slow = s0 + q * ds;
      if (slow <= fast) row[tile_of(q) * kTile + in_tile(q)] = value(q);
    }
  } else {
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
      const int slow = s0 + q * ds;
      if (slow < ts && fast <= slow) Map::at(S, tile_of(q), ft)[in_tile(q) * kTld + fr] = value(q);
    }
  }
  __syncthreads();
  const int wave = tid >> 6;
  if (wave < ntile) invert_tile(Map::at(S, wave, wave), false, false);
  __syncthreads();
  combine<Map, kInvNt>(S, ntile, false, false);
  double* __restrict__ o = out + ((int64_t)s0 * n0 + fast);
#pragma unroll
  for (int q = 0; q < kEach; ++q) {
    if (!TS && q >= own.most) break;
    const int i = s0 + q * ds, r = TS ? i : square_line(own, q, ts);
    const int rt = TS ? tile_of(q) : r >> 4;
    const double x = Map::at(S, rt, min(ft, rt))[(TS ? in_tile(q) : r & 15) * kTld + fr];
    if (i < ts) o[q * (ds * n0)] = fast <= i ? x : 0.0;
  }
}

// The last pass over the packed blocks: zeros above the diagonal (Alg.
// RecTriInv's products used that space), the binary32 copy if one is wanted,
// and the check of L's diagonal.  One row of one block per workgroup.
template <typename TL>
__global__ __launch_bounds__(256) void block_finish_kernel(const TL* __restrict__ L, int64_t ldl,
                                                           int64_t n, int64_t n0,
                                                           double* __restrict__ Linv,
                                                           float* __restrict__ Linv32,
                                                           unsigned long long* bad) {
  const int64_t row = blockIdx.x, i = row % n0;
  double* __restrict__ out = Linv + row * n0;
  if (threadIdx.x == 0 && bad && row < n) {
    const double d = static_cast<double>(L[row * ldl + row]);
    if (!(d != 0.0) || !isfinite(d)) atomicMin(bad, (unsigned long long)row);
  }
  if (Linv32) {
    float* __restrict__ o32 = Linv32 + row * n0;
    for (int64_t j = threadIdx.x; j < n0; j += blockDim.x) {
      o32[j] = j <= i ? static_cast<float>(out[j]) : 0.0f;
      if (j > i) out[j] = 0.0;
    }
  } else {
    for (int64_t j = i + 1 + threadIdx.x; j < n0; j += blockDim.x) out[j] = 0.0;
  }
}

template <typename TI, typename TO>
__global__ void convert_kernel(const TI* __restrict__ in, TO* __restrict__ out, int64_t count) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = cvt<TO>(in[i]);
}

template <typename TI, typename TO>
__global__ void copy2d_kernel(const TI* __restrict__ in, int64_t ldi, TO* __restrict__ out,
                              int64_t ldo, int64_t rows, int64_t cols, double scale) {
  const int64_t total = rows * cols;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / cols, c = i % cols;
    out[r * ldo + c] = cvt<TO>(static_cast<double>(in[r * ldi + c]) * scale);
  }
}

__global__ void axpy_kernel(const float* __restrict__ D, int64_t ldd, double* __restrict__ X,
                            int64_t ldx, int64_t rows, int64_t cols, double scale, int assign) {
  const int64_t total = rows * cols;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / cols, c = i % cols;
    const double d = scale * static_cast<double>(D[r * ldd + c]);
    if (assign) X[r * ldx + c] = d;
    else X[r * ldx + c] += d;
  }
}

// One wave per (row r, column block c).  Waves for c >= floor(r / n0) (the
// diagonal block and beyond) only write a unit scale.
template <typename TO>
__global__ __launch_bounds__(256) void lowcopy_kernel(const double* __restrict__ L, int64_t ldl,
                                                      int64_t n, int64_t n0, int64_t m,
                                                      TO* __restrict__ Llow,
                                                      float* __restrict__ rscale, float target) {
  const int lane = threadIdx.x & 63;
  const int64_t wid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (wid >= n * m) return;
  const int64_t r = wid / m, c = wid % m;
  if (c >= r / n0) {
    if (lane == 0) rscale[r * m + c] = 1.0f;
    return;
  }
  const double* src = L + r * ldl + c * n0;
  double mx = 0.0;
  for (int64_t j = lane; j < n0; j += 64) mx = fmax(mx, fabs(src[j]));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
  int e = 0;
  if (mx > 0.0) e = ilogb((double)target) - ilogb(mx) - 1;
  TO* dst = Llow + r * n + c * n0;
  for (int64_t j = lane; j < n0; j += 64) dst[j] = cvt<TO>(ldexp(src[j], e));
  if (lane == 0) rscale[r * m + c] = ldexpf(1.0f, -e);
}

// out[r * cols + c] = low(a[r * cols + c] 2^e_r) with one power-of-two scale
// per row (its largest magnitude placed just below `target`) and
// rs[r] = 2^-e_r; one wave per row.
template <typename TO>
__global__ __launch_bounds__(256) void rowscale_copy_kernel(const double* __restrict__ a,
                                                            int64_t rows, int64_t cols,
                                                            TO* __restrict__ out,
                                                            float* __restrict__ rs, float target) {
  const int lane = threadIdx.x & 63;
  const int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (r >= rows) return;
  const double* src = a + r * cols;
  double mx = 0.0;
  for (int64_t j = lane; j < cols; j += 64) mx = fmax(mx, fabs(src[j]));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
  int e = 0;
  if (mx > 0.0) e = ilogb((double)target) - ilogb(mx) - 1;
  for (int64_t j = lane; j < cols; j += 64) out[r * cols + j] = cvt<TO>(ldexp(src[j], e));
  if (lane == 0) rs[r] = ldexpf(1.0f, -e);
}

// Largest |D| over a rows x cols block as float bits: the bit patterns of
// non-negative floats order like their values (and a NaN orders above
// infinity, so it is not lost).  out[0] must start at zero.  VEC elements a load (4:
// rows 16-byte aligned) and four loads in flight a thread, the last ones of a row
// clamped into it (a maximum may see an element twice): 1024 x 8192 21 us, now 11.
template <int VEC>
__global__ __launch_bounds__(256) void absmax_bits_kernel(const float* __restrict__ D, int64_t ldd,
                                                          int64_t rows, int64_t cols,
                                                          unsigned* __restrict__ out) {
  typedef unsigned V __attribute__((ext_vector_type(VEC)));
  __shared__ unsigned wmax[4];
  unsigned mx = 0;
  const int64_t nv = cols / VEC;
  for (int64_t r = blockIdx.x; r < rows; r += gridDim.x) {
    const V* __restrict__ row = reinterpret_cast<const V*>(D + r * ldd);
    for (int64_t c = threadIdx.x; c < nv; c += 4 * 256) {
      V v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = row[min(c + u * 256, nv - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < VEC; ++e) mx = max(mx, v[u][e] & 0x7FFFFFFFu);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = max(mx, (unsigned)__shfl_xor((int)mx, off));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    mx = max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3]));
    if (mx) atomicMax(out, mx);
  }
}

__global__ void fill_u32_kernel(unsigned* __restrict__ p, int64_t count, unsigned v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = v;
}

// XT[c * ldx + r] = low(2^e * D[r * ldd + c]) with 2^e putting the block's
// largest magnitude in [2^etarget, 2^(etarget+1)); *xinv = 2^-e.  64 x 64
// tiles transposed through LDS.
template <typename TO>
__global__ __launch_bounds__(256) void lowx_kernel(const float* __restrict__ D, int64_t ldd,
                                                   int64_t rows, int64_t cols, TO* __restrict__ XT,
                                                   int64_t ldx, const unsigned* __restrict__ amax,
                                                   float* __restrict__ xinv, int etarget) {
  __shared__ float tile[64][65];
  const float mx = __uint_as_float(*amax);
  int e = 0;
  if (mx > 0.0f && isfinite(mx)) e = etarget - ilogbf(mx);
  if (blockIdx.x == 0 && threadIdx.x == 0) *xinv = ldexpf(1.0f, -e);
  const int64_t ntc = (cols + 63) / 64;
  const int64_t tr = (blockIdx.x / ntc) * 64, tc = (blockIdx.x % ntc) * 64;
  const int lo = threadIdx.x & 63, hi = threadIdx.x >> 6;
#pragma unroll 4
  for (int j = 0; j < 16; ++j) {
    const int64_t r = tr + hi + 4 * j, c = tc + lo;
    tile[hi + 4 * j][lo] = (r < rows && c < cols) ? D[r * ldd + c] : 0.0f;
  }
  __syncthreads();
#pragma unroll 4
  for (int j = 0; j < 16; ++j) {
    const int64_t c = tc + hi + 4 * j, r = tr + lo;
    if (r < rows && c < cols) XT[c * ldx + r] = cvt<TO>(ldexpf(tile[lo][hi + 4 * j], e));
  }
}

// Uniform in [0, 1) from a 64-bit counter (splitmix64 finaliser).
__device__ inline double hash_unit(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  x ^= x >> 31;
  return (double)(x >> 11) * (1.0 / 9007199254740992.0);
}

template <typename T>
__global__ void fill_system_kernel(T* __restrict__ L, int64_t n, T* __restrict__ B, int64_t k,
                                   uint64_t seed) {
  const int64_t tl = n * n, total = tl + n * k;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const double u = hash_unit(seed * 0x100000001B3ull + (uint64_t)e);
    if (e < tl) {
      const int64_t i = e / n, j = e - i * n;
      L[e] = (T)(j == i ? 1.0 + u : (j < i ? (2.0 * u - 1.0) / (double)n : 0.0));
    } else {
      B[e - tl] = (T)(u - 0.5);
    }
  }
}

// 64 x 64 tiles transposed through LDS; one workgroup per (matrix, tile).
template <typename TI, typename TO>
__global__ __launch_bounds__(256) void transpose_kernel(const TI* __restrict__ in, int64_t ldi,
                                                        TO* __restrict__ out, int64_t ldo,
                                                        int64_t rows, int64_t cols, int64_t si,
                                                        int64_t so, int64_t tiles_per,
                                                        bool lower_only) {
  __shared__ TO tile[64][65];
  const int64_t b = blockIdx.x / tiles_per, t = blockIdx.x % tiles_per;
  const int64_t ntc = (cols + 63) / 64;
  const int64_t tr = (t / ntc) * 64, tc = (t % ntc) * 64;
  const TI* src = in + b * si;
  TO* dst = out + b * so;
  const int lo = threadIdx.x & 63, hi = threadIdx.x >> 6;
#pragma unroll 4
  for (int j = 0; j < 16; ++j) {
    const int64_t r = tr + hi + 4 * j, c = tc + lo;
    TO v = TO(0);
    if (r < rows && c < cols && !(lower_only && r < c)) v = (TO)src[r * ldi + c];
    tile[hi + 4 * j][lo] = v;
  }
  __syncthreads();
#pragma unroll 4
  for (int j = 0; j < 16; ++j) {
    const int64_t c = tc + hi + 4 * j, r = tr + lo;
    if (r < rows && c < cols) dst[c * ldo + r] = tile[lo][hi + 4 * j];
  }
}

// Recursive baseline leaf: forward substitution, one thread per column.
template <typename T>
__global__ __launch_bounds__(64) void subst_leaf_kernel(const T* __restrict__ L, int64_t ldl,
                                                        T* __restrict__ X, int64_t ldx,
                                                        int64_t nb, int64_t k) {
  __shared__ T Ls[64][65];
  __shared__ T Xs[64][65];
  const int t = threadIdx.x;
  const int64_t c = (int64_t)blockIdx.x * 64 + t;
  for (int i = 0; i < nb; ++i) Ls[i][t] = (t < nb && t <= i) ? L[(int64_t)i * ldl + t] : T(0);
  __syncthreads();
  if (c < k) {
    for (int i = 0; i < nb; ++i) {
      T s = X[(int64_t)i * ldx + c];
      for (int p = 0; p < i; ++p) s -= Ls[i][p] * Xs[p][t];
      const T x = s / Ls[i][i];
      Xs[i][t] = x;
      X[(int64_t)i * ldx + c] = x;
    }
  }
}

// Deterministic reductions: a fixed grid of kNormBlocks blocks; block b takes
// rows b, b + kNormBlocks, ... in order and thread t of it the columns t,
// t + 256, ... of each row (whole rows per block: coalesced, no index
// division), then a fixed-shape reduction: butterflies inside each wavefront
// and a fixed sum of the four wavefronts' results.
__device__ inline void block_reduce2(double& s, double& mx) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s += __shfl_xor(s, o, 64);
    mx = fmax(mx, __shfl_xor(mx, o, 64));
  }
  __shared__ double ws[4], wm[4];
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    ws[w] = s;
    wm[w] = mx;
  }
  __syncthreads();
  s = (ws[0] + ws[1]) + (ws[2] + ws[3]);
  mx = fmax(fmax(wm[0], wm[1]), fmax(wm[2], wm[3]));
}

__global__ __launch_bounds__(256) void sumsq_max_part(const double* __restrict__ A, int64_t lda,
                                                      int64_t rows, int64_t cols,
                                                      double* __restrict__ part) {
  double s = 0.0, mx = 0.0;
  for (int64_t r = blockIdx.x; r < rows; r += kNormBlocks) {
    const double* __restrict__ a = A + r * lda;
    for (int64_t c = threadIdx.x; c < cols; c += 256) {
      const double v = a[c];
      s += v * v;
      mx = fmax(mx, fabs(v));
    }
  }
  block_reduce2(s, mx);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = s;
    part[kNormBlocks + blockIdx.x] = mx;
  }
}

template <typename TL>
__global__ __launch_bounds__(256) void sumsq_lower_part(const TL* __restrict__ L, int64_t ldl,
                                                        int64_t n, double* __restrict__ part) {
  double s = 0.0, mx = 0.0;
  for (int64_t r = blockIdx.x; r < n; r += kNormBlocks) {
    const TL* __restrict__ l = L + r * ldl;
    for (int64_t c = threadIdx.x; c <= r; c += 256) {
      const double v = static_cast<double>(l[c]);
      s += v * v;
      mx = fmax(mx, fabs(v));
    }
  }
  block_reduce2(s, mx);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = s;
    part[kNormBlocks + blockIdx.x] = mx;
  }
}

__global__ __launch_bounds__(256) void reduce_final(const double* __restrict__ part,
                                                    double* __restrict__ out) {
  double s = 0.0, mx = 0.0;
  for (int i = threadIdx.x; i < kNormBlocks; i += 256) {
    s += part[i];
    mx = fmax(mx, part[kNormBlocks + i]);
  }
  block_reduce2(s, mx);
  if (threadIdx.x == 0) {
    out[0] = s;
    out[1] = mx;
  }
}

}  // namespace

template <typename TL>
hipError_t launch_block_inverse(const TL* L, int64_t ldl, int64_t n, int64_t n0, int64_t m,
                                double* Linv, unsigned long long* bad, bool upper, bool unit,
                                hipStream_t s) {
  if (m <= 0) return hipSuccess;
  const int ts = (int)std::min<int64_t>(n0, kInvRows);
  const int64_t nt = n0 / ts;
  const unsigned grid = (unsigned)(m * nt * (nt + 1) / 2);
  if (ts == kInvRows)
    block_inverse_kernel<TL, kInvRows><<<grid, kInvThreads, 0, s>>>(L, ldl, n, n0, ts, m, Linv, bad,
                                                                    upper, unit);
  else
    block_inverse_kernel<TL, 0><<<grid, kInvThreads, 0, s>>>(L, ldl, n, n0, ts, m, Linv, bad, upper,
                                                             unit);
  return hipGetLastError();
}
template hipError_t launch_block_inverse<double>(const double*, int64_t, int64_t, int64_t, int64_t,
                                                 double*, unsigned long long*, bool, bool,
                                                 hipStream_t);
template hipError_t launch_block_inverse<float>(const float*, int64_t, int64_t, int64_t, int64_t,
                                                double*, unsigned long long*, bool, bool,
                                                hipStream_t);

template <typename TL>
hipError_t launch_block_finish(const TL* L, int64_t ldl, int64_t n, int64_t n0, int64_t m,
                               double* Linv, float* Linv32, unsigned long long* bad,
                               hipStream_t s) {
  if (m <= 0) return hipSuccess;
  block_finish_kernel<TL><<<(unsigned)(m * n0), row_threads(n0), 0, s>>>(L, ldl, n, n0, Linv,
                                                                         Linv32, bad);
  return hipGetLastError();
}
template hipError_t launch_block_finish<double>(const double*, int64_t, int64_t, int64_t, int64_t,
                                                double*, float*, unsigned long long*, hipStream_t);
template hipError_t launch_block_finish<float>(const float*, int64_t, int64_t, int64_t, int64_t,
                                               double*, float*, unsigned long long*, hipStream_t);

template <typename TI, typename TO>
hipError_t launch_convert(const TI* in, TO* out, int64_t count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  convert_kernel<TI, TO><<<grid_for(count, 256), 256, 0, s>>>(in, out, count);
  return hipGetLastError();
}
template hipError_t launch_convert<double, float>(const double*, float*, int64_t, hipStream_t);

template <typename TI, typename TO>
hipError_t launch_copy2d(const TI* in, int64_t ldi, TO* out, int64_t ldo, int64_t rows,
                         int64_t cols, double scale, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  copy2d_kernel<TI, TO><<<grid_for(rows * cols, 256), 256, 0, s>>>(in, ldi, out, ldo, rows, cols,
                                                                   scale);
  return hipGetLastError();
}
template hipError_t launch_copy2d<double, double>(const double*, int64_t, double*, int64_t,
                                                  int64_t, int64_t, double, hipStream_t);
template hipError_t launch_copy2d<float, float>(const float*, int64_t, float*, int64_t, int64_t,
                                                int64_t, double, hipStream_t);
template hipError_t launch_copy2d<double, float>(const double*, int64_t, float*, int64_t, int64_t,
                                                 int64_t, double, hipStream_t);
template hipError_t launch_copy2d<float, double>(const float*, int64_t, double*, int64_t, int64_t,
                                                 int64_t, double, hipStream_t);

hipError_t launch_axpy_f32_to_f64(const float* D, int64_t ldd, double* X, int64_t ldx,
                                  int64_t rows, int64_t cols, double scale, bool assign,
                                  hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  axpy_kernel<<<grid_for(rows * cols, 256), 256, 0, s>>>(D, ldd, X, ldx, rows, cols, scale,
                                                         assign ? 1 : 0);
  return hipGetLastError();
}

template <typename TO>
hipError_t launch_lowcopy(const double* L, int64_t ldl, int64_t n, int64_t n0, int64_t m,
                          TO* Llow, float* rscale, float target, hipStream_t s) {
  if (n <= 0 || m <= 0) return hipSuccess;
  const int64_t waves = n * m;
  lowcopy_kernel<TO><<<grid_for(waves * 64, 256, INT64_MAX), 256, 0, s>>>(L, ldl, n, n0, m, Llow,
                                                                          rscale, target);
  return hipGetLastError();
}
template <typename TO>
hipError_t launch_rowscale_copy(const double* a, int64_t rows, int64_t cols, TO* out, float* rs,
                               float target, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  rowscale_copy_kernel<TO><<<grid_for(rows * 64, 256, INT64_MAX), 256, 0, s>>>(a, rows, cols, out,
                                                                              rs, target);
  return hipGetLastError();
}
template hipError_t launch_rowscale_copy<bf16_t>(const double*, int64_t, int64_t, bf16_t*, float*,
                                                 float, hipStream_t);
template hipError_t launch_rowscale_copy<f16_t>(const double*, int64_t, int64_t, f16_t*, float*,
                                                float, hipStream_t);

template hipError_t launch_lowcopy<bf16_t>(const double*, int64_t, int64_t, int64_t, int64_t,
                                           bf16_t*, float*, float, hipStream_t);
template hipError_t launch_lowcopy<f16_t>(const double*, int64_t, int64_t, int64_t, int64_t,
                                          f16_t*, float*, float, hipStream_t);
template hipError_t launch_lowcopy<fp8_t>(const double*, int64_t, int64_t, int64_t, int64_t,
                                          fp8_t*, float*, float, hipStream_t);

hipError_t launch_fill_u32(unsigned* p, int64_t count, unsigned v, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  fill_u32_kernel<<<(unsigned)ceil_div(count, 256), 256, 0, s>>>(p, count, v);
  return hipGetLastError();
}

template <typename TO>
hipError_t launch_lowx(const float* D, int64_t ldd, int64_t rows, int64_t cols, TO* XT,
                       int64_t ldx, unsigned* amax, float* xinv, int etarget, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  // few workgroups: each ends in one atomic on the same word, about 10 ns apiece
  const unsigned wgs = (unsigned)std::min<int64_t>(rows, 512);
  if (((uintptr_t)D & 15) == 0 && ldd % 4 == 0 && cols % 4 == 0)
    absmax_bits_kernel<4><<<wgs, 256, 0, s>>>(D, ldd, rows, cols, amax);
  else
    absmax_bits_kernel<1><<<wgs, 256, 0, s>>>(D, ldd, rows, cols, amax);
  const int64_t tiles = ceil_div(rows, 64) * ceil_div(cols, 64);
  lowx_kernel<TO><<<(unsigned)tiles, 256, 0, s>>>(D, ldd, rows, cols, XT, ldx, amax, xinv, etarget);
  return hipGetLastError();
}
template hipError_t launch_lowx<bf16_t>(const float*, int64_t, int64_t, int64_t, bf16_t*, int64_t,
                                        unsigned*, float*, int, hipStream_t);
template hipError_t launch_lowx<f16_t>(const float*, int64_t, int64_t, int64_t, f16_t*, int64_t,
                                       unsigned*, float*, int, hipStream_t);
template hipError_t launch_lowx<fp8_t>(const float*, int64_t, int64_t, int64_t, fp8_t*, int64_t,
                                       unsigned*, float*, int, hipStream_t);

template <typename T>
hipError_t launch_fill_system(T* L, int64_t n, T* B, int64_t k, uint64_t seed, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  fill_system_kernel<T><<<grid_for(n * n + n * k, 256, 16384), 256, 0, s>>>(L, n, B, k, seed);
  return hipGetLastError();
}
template hipError_t launch_fill_system<double>(double*, int64_t, double*, int64_t, uint64_t,
                                               hipStream_t);
template hipError_t launch_fill_system<float>(float*, int64_t, float*, int64_t, uint64_t,
                                              hipStream_t);

template <typename TI, typename TO>
hipError_t launch_transpose(const TI* in, int64_t ldi, TO* out, int64_t ldo, int64_t rows,
                            int64_t cols, int64_t batch, int64_t si, int64_t so, bool lower_only,
                            hipStream_t s) {
  if (rows <= 0 || cols <= 0 || batch <= 0) return hipSuccess;
  const int64_t per = ceil_div(rows, 64) * ceil_div(cols, 64);
  transpose_kernel<TI, TO><<<(unsigned)(per * batch), 256, 0, s>>>(in, ldi, out, ldo, rows, cols,
                                                                   si, so, per, lower_only);
  return hipGetLastError();
}
template hipError_t launch_transpose<double, double>(const double*, int64_t, double*, int64_t,
                                                     int64_t, int64_t, int64_t, int64_t, int64_t,
                                                     bool, hipStream_t);
template hipError_t launch_transpose<float, float>(const float*, int64_t, float*, int64_t, int64_t,
                                                   int64_t, int64_t, int64_t, int64_t, bool,
                                                   hipStream_t);

template <typename T>
hipError_t launch_subst_leaf(const T* L, int64_t ldl, T* X, int64_t ldx, int64_t nb, int64_t k,
                             hipStream_t s) {
  if (nb <= 0 || k <= 0) return hipSuccess;
  subst_leaf_kernel<T><<<(unsigned)ceil_div(k, 64), 64, 0, s>>>(L, ldl, X, ldx, nb, k);
  return hipGetLastError();
}
template hipError_t launch_subst_leaf<double>(const double*, int64_t, double*, int64_t, int64_t,
                                              int64_t, hipStream_t);
template hipError_t launch_subst_leaf<float>(const float*, int64_t, float*, int64_t, int64_t,
                                             int64_t, hipStream_t);

hipError_t launch_sumsq_max(const double* A, int64_t lda, int64_t rows, int64_t cols,
                            double* part, double* out, hipStream_t s) {
  sumsq_max_part<<<kNormBlocks, 256, 0, s>>>(A, lda, rows, cols, part);
  reduce_final<<<1, 256, 0, s>>>(part, out);
  return hipGetLastError();
}

template <typename TL>
hipError_t launch_sumsq_lower(const TL* L, int64_t ldl, int64_t n, double* part, double* out,
                              hipStream_t s) {
  sumsq_lower_part<TL><<<kNormBlocks, 256, 0, s>>>(L, ldl, n, part);
  reduce_final<<<1, 256, 0, s>>>(part, out);
  return hipGetLastError();
}
template hipError_t launch_sumsq_lower<double>(const double*, int64_t, int64_t, double*, double*,
                                               hipStream_t);
template hipError_t launch_sumsq_lower<float>(const float*, int64_t, int64_t, double*, double*,
                                              hipStream_t);

}  // namespace trsm
