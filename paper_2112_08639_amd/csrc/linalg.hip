// Dense linear algebra of the hot path: Gram / projection products, blocked
// FP64 Cholesky with the inverse of the factor (for CholQR), the triangular
// update X R^{-1}, and the FP64 extreme eigenvalues of H_s by shifted
// repeated squaring.
#include <cmath>

#include "ctx.h"
#include "gemm.h"
#include "gemm_f64.h"

namespace dk {

namespace {

constexpr int NB = 32;  // Cholesky block size

// out = scale * sum_s P[s]; mirror_upper: out(i,j) = out(j,i) = the sum at
// (min(i,j), max(i,j)) (the upper tiles are the only ones computed);
// otherwise symmetrise, (P + P^T)/2.  One workgroup per pair of 16 x 16 tiles
// (bi, bj) and (bj, bi) with bi <= bj: both are read along columns and the
// transposes go through LDS, so every global access is coalesced.
constexpr int RT = 16;
template <typename PT>
__global__ __launch_bounds__(256) void reduce_square_kernel(const PT* __restrict__ part,
                                                            int splits, int n, double scale,
                                                            int mirror_upper,
                                                            double* __restrict__ out) {
  const int bi = blockIdx.x, bj = blockIdx.y;
  if (bi > bj) return;
  __shared__ double ta[RT][RT + 1];  // ta[c][r] = P(bi RT + r, bj RT + c)
  __shared__ double tb[RT][RT + 1];  // tb[c][r] = P(bj RT + r, bi RT + c)
  const long nn = (long)n * n;
  const int r = threadIdx.x % RT, c = threadIdx.x / RT;
  auto sum_at = [&](int i, int j) {
    double v = 0.0;
    if (i < n && j < n)
      for (int k = 0; k < splits; ++k) v += (double)part[(long)k * nn + i + (long)j * n];
    return v;
  };
  ta[c][r] = sum_at(bi * RT + r, bj * RT + c);
  if (!mirror_upper && bi != bj) tb[c][r] = sum_at(bj * RT + r, bi * RT + c);
  __syncthreads();
  // tile (bi, bj): element (i, j) = (bi RT + r, bj RT + c)
  {
    const int i = bi * RT + r, j = bj * RT + c;
    double v;
    if (mirror_upper) v = (bi < bj || r <= c) ? ta[c][r] : ta[r][c];
    else v = 0.5 * (ta[c][r] + (bi == bj ? ta[r][c] : tb[r][c]));
    if (i < n && j < n) out[i + (long)j * n] = scale * v;
  }
  // tile (bj, bi): element (bj RT + r, bi RT + c)
  if (bi < bj) {
    const int i = bj * RT + r, j = bi * RT + c;
    const double v = mirror_upper ? ta[r][c] : 0.5 * (tb[c][r] + ta[r][c]);
    if (i < n && j < n) out[i + (long)j * n] = scale * v;
  }
}

// Inverse Cholesky factor Z = L^{-1} of a symmetric positive definite G, NB columns a
// step, by elimination on [G; I] (right-looking): with Z_k the inverse of the factor of
// the current diagonal block,
//   P_a   = G_ak Z_k^T                 for every block row a (L_ak below the diagonal)
//   G_ab -= P_a P_b^T                  for a >= b > k   (trailing update)
//   W_ab -= P_a P_b^T                  for a <= k < b   (forward substitution of I, W = Z^T)
// where the row a = k of the second form starts from I (P_k = Z_k^T, W_kb = 0).  The
// strictly upper blocks of G hold W: the lower triangle of G and the upper one of W never
// meet, operands of all rows stand in block column k, and row k of Z is P_a^T, a < k.
// The chain of steps is what takes the time (n = 512: 16 of them), so a step is one
// launch: each workgroup forms the two P it needs itself (two 32^3 products, 0.5 us)
// rather than wait for a panel launch, and the one with the next diagonal block
// factors it at once.  Measured, factor and inverse: n = 512 740 -> 240 us, n = 2048
// 4.8 -> 1.2 ms (before: a launch each for diagonal block, panel and trailing update, then
// two per block row of the inverse); a step is 14 us at n = 512, most of it the
// diagonal block's chain, and 18 us on average at n = 2048.
typedef double f64x2_c __attribute__((ext_vector_type(2)));
constexpr int CP = NB + 2;  // pitch of a block in LDS: rows four banks apart

// 1 / sqrt(d) for d > 0: the hardware estimate and two Newton steps in residual form
__device__ __forceinline__ double rsqrt_f64(double d) {
  double y = __builtin_amdgcn_rsq(d);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double e = __builtin_fma(-d * y, y, 1.0);
    y = __builtin_fma(0.5 * y, e, y);
  }
  return y;
}

// D = X Y^T of two 32 x 32 blocks in LDS ([row][k]); wave w computes the quadrant rows
// 16 (w & 1), columns 16 (w >> 1): register q of lane l is D[l / 16 + 4 q][l % 16].
__device__ __forceinline__ f64x4 block_nt(const double* X, const double* Y, int wave, int lane) {
  const double* x = X + (16 * (wave & 1) + (lane & 15)) * CP + 4 * (lane >> 4);
  const double* y = Y + (16 * (wave >> 1) + (lane & 15)) * CP + 4 * (lane >> 4);
  f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < NB; k += 16)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f64x2_c a = *reinterpret_cast<const f64x2_c*>(x + k + 2 * h);
      const f64x2_c b = *reinterpret_cast<const f64x2_c*>(y + k + 2 * h);
      d = mfma_f64(a[0], b[0], d);
      d = mfma_f64(a[1], b[1], d);
    }
  return d;
}

// Factor the NB x NB block A (LDS, [row][col], lower triangle) = L L^T and leave L^{-1}
// in Zi ([row][col]); one wave.  Lane r < 32 holds row r of A, lane 32 + r row r of I, and
// the columns are eliminated in registers: the same operations that turn A into L turn
// I into L^{-T}.  (The 32 steps are a serial chain of a reciprocal root and one column;
// with the block in LDS, a barrier per step and a separate inverse: 22.5 us.)  A pivot
// below 1e-14 of the original diagonal entry dref (lane r: of row r) is taken as
// singular: X is then rank-deficient to working precision.
__device__ void factor_block(const double* A, double* Zi, double dref, int lane, unsigned* err) {
  double a[NB];
  const int r = lane & (NB - 1);
#pragma unroll
  for (int c = 0; c < NB; ++c) a[c] = lane < NB ? A[r * CP + c] : (r == c ? 1.0 : 0.0);
  auto lane_value = [](double v, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
  };
  bool bad = false;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    double d = lane_value(a[k], k);
    if (!(d > 1e-14 * lane_value(dref, k)) || !isfinite(d)) {
      bad = true;
      d = 1.0;
    }
    const double l = a[k] * rsqrt_f64(d);
    a[k] = l;
#pragma unroll
    for (int c = k + 1; c < NB; ++c) a[c] = __builtin_fma(-l, lane_value(l, c), a[c]);
  }
  if (bad && lane == 0) atomicOr(err, kErrNotSpd);
  if (lane >= NB) {
#pragma unroll
    for (int c = 0; c < NB; ++c) Zi[c * CP + r] = c >= r ? a[c] : 0.0;
  }
}

// block (row0.., col0..) of the column-major n x n matrix m into LDS as [row][col]; rows
// and columns past n: of the identity (pad) or zero
__device__ __forceinline__ void load_block(const double* m, int n, int row0, int col0, bool pad,
                                           double* s, int t) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = t & 31, c = (t >> 5) + 8 * q;
    const bool in = row0 + r < n && col0 + c < n;
    const double v = m[min(row0 + r, n - 1) + (long)min(col0 + c, n - 1) * n];
    s[r * CP + c] = in ? v : (pad && r == c ? 1.0 : 0.0);
  }
}

// linv block k (on the diagonal) from LDS
__device__ __forceinline__ void store_diag(double* linv, int n, int k, const double* Zi, int t) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = t & 31, c = (t >> 5) + 8 * q;
    if (k * NB + r < n && k * NB + c < n)
      linv[(k * NB + r) + (long)(k * NB + c) * n] = Zi[r * CP + c];
  }
}

// diag = diagonal of g; linv = 0 outside its first diagonal block, which the first
// workgroup factors
__global__ __launch_bounds__(256) void chol_start_kernel(const double* __restrict__ g, int n,
                                                         double* __restrict__ linv,
                                                         double* __restrict__ diag, unsigned* err) {
  __shared__ __attribute__((aligned(16))) double A[NB * CP];
  __shared__ __attribute__((aligned(16))) double Zi[NB * CP];
  const int t = threadIdx.x;
  if (blockIdx.x > 0) {
    const long nn = (long)n * n, step = (long)(gridDim.x - 1) * 256;
    for (long e = (blockIdx.x - 1) * 256L + t; e < nn; e += step) {
      const int i = (int)(e % n), j = (int)(e / n);
      if (i >= NB || j >= NB) linv[e] = 0.0;
      if (i == j) diag[i] = g[e];
    }
    return;
  }
  load_block(g, n, 0, 0, true, A, t);
  __syncthreads();
  if (t < 64) {
    const int r = t & 31;
    factor_block(A, Zi, r < n ? g[r + (long)r * n] : 1.0, t, err);
  }
  __syncthreads();
  store_diag(linv, n, 0, Zi, t);
}

// Step k.  Workgroup (a, b), b > k: tile (a, b) of W (a <= k) or, as (b, a) with a > k,
// of G; the last step has no such tiles and writes row k of Z only.
__global__ __launch_bounds__(256) void chol_step_kernel(double* __restrict__ g, int n, int k,
                                                        double* __restrict__ linv,
                                                        const double* __restrict__ diag,
                                                        unsigned* err) {
  __shared__ __attribute__((aligned(16))) double Zk[NB * CP];
  __shared__ __attribute__((aligned(16))) double Pa[NB * CP];
  __shared__ __attribute__((aligned(16))) double Pb[NB * CP];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int nb = (n + NB - 1) / NB;
  const bool final_row = k == nb - 1;
  // tiles in order of b, then a = 0 .. b, but first the one to be factored, (k + 1, k + 1)
  int a, b = k;
  if (final_row) {
    a = blockIdx.x;
  } else {
    const int x = blockIdx.x;
    const long id = (long)(k + 1) * (k + 2) / 2 + (x == 0 ? k + 1 : x <= k + 1 ? x - 1 : x);
    b = (int)((sqrt(8.0 * (double)id + 1.0) - 1.0) * 0.5);
    while ((long)(b + 1) * (b + 2) / 2 <= id) ++b;
    while ((long)b * (b + 1) / 2 > id) --b;
    a = (int)(id - (long)b * (b + 1) / 2);
  }
  const bool upper = a <= k;  // a tile of W
  load_block(linv, n, k * NB, k * NB, false, Zk, t);
  if (a == k) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = t & 31, c = (t >> 5) + 8 * q;
      Pa[r * CP + c] = r == c ? 1.0 : 0.0;
    }
  } else {
    load_block(g, n, a * NB, k * NB, false, Pa, t);
  }
  if (!final_row) load_block(g, n, b * NB, k * NB, false, Pb, t);
  // the tile itself: rows a, columns b (W) or rows b, columns a (G).  The product below
  // has the tile's columns as its rows, so a lane's values are along 16 rows.
  const int row0 = (upper ? a : b) * NB + 16 * (wave >> 1) + (lane & 15);
  const int col0 = (upper ? b : a) * NB + 16 * (wave & 1) + (lane >> 4);
  double c[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    c[q] = (final_row || a == k || row0 >= n || col0 + 4 * q >= n)
               ? 0.0
               : g[row0 + (long)(col0 + 4 * q) * n];
  __syncthreads();
  const f64x4 pa = block_nt(Pa, Zk, wave, lane);
  f64x4 pb = pa;
  if (!final_row && a != b) pb = block_nt(Pb, Zk, wave, lane);
  const int pr = 16 * (wave & 1) + (lane >> 4), pc = 16 * (wave >> 1) + (lane & 15);
  // row k of Z, off the diagonal: the transposes of P_a, a < k, from the tiles of b = k + 1
  if (a < k && (final_row || b == k + 1)) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (k * NB + pc < n) linv[(k * NB + pc) + (long)(a * NB + pr + 4 * q) * n] = pa[q];
  }
  if (final_row) return;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    Pa[(pr + 4 * q) * CP + pc] = pa[q];
    Pb[(pr + 4 * q) * CP + pc] = pb[q];
  }
  __syncthreads();
  const f64x4 d = upper ? block_nt(Pb, Pa, wave, lane) : block_nt(Pa, Pb, wave, lane);
  const bool next = a == k + 1 && b == k + 1;
  if (next) __syncthreads();  // Pa becomes the block to be factored
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double v = c[q] - d[q];
    if (next) {
      const int r = row0 - b * NB, cc = col0 + 4 * q - b * NB;
      Pa[r * CP + cc] = (row0 < n && col0 + 4 * q < n) ? v : (r == cc ? 1.0 : 0.0);
    } else if (row0 < n && col0 + 4 * q < n) {
      g[row0 + (long)(col0 + 4 * q) * n] = v;
    }
  }
  if (!next) return;
  __syncthreads();
  if (t < 64) {
    const int r = b * NB + (t & 31);
    factor_block(Pa, Zk, r < n ? diag[r] : 1.0, t, err);
  }
  __syncthreads();
  store_diag(linv, n, b, Zk, t);
}

template <typename TS, typename TD>
__global__ void copy_block_kernel(const TS* __restrict__ src, TD* __restrict__ dst, long rows,
                                  long ld, int cols) {
  const long tot = rows * cols;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < tot;
       e += (long)gridDim.x * blockDim.x) {
    const long c = e / rows, r = e - c * rows;
    dst[r + c * ld] = (TD)src[r + c * ld];
  }
}

__global__ void finite_kernel(const double* __restrict__ p, long n, unsigned* err) {
  bool bad = false;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x)
    if (!isfinite(p[e])) bad = true;
  if (bad) atomicOr(err, kErrNonFinite);
}

inline int grid_for(long n) {
  long b = (n + 255) / 256;
  if (b > 8192) b = 8192;
  if (b < 1) b = 1;
  return (int)b;
}

}  // namespace

hipError_t copy_block(dk_ctx* c, const void* src, void* dst, long ld, int n_s) {
  if (c->precision == DK_PREC_FP64)
    hipLaunchKernelGGL((copy_block_kernel<double, double>), dim3(grid_for(c->ngrid * n_s)),
                       dim3(256), 0, c->stream, (const double*)src, (double*)dst, c->ngrid, ld, n_s);
  else
    hipLaunchKernelGGL((copy_block_kernel<float, float>), dim3(grid_for(c->ngrid * n_s)),
                       dim3(256), 0, c->stream, (const float*)src, (float*)dst, c->ngrid, ld, n_s);
  return hipGetLastError();
}

hipError_t check_finite(dk_ctx* c, const double* p, long n) {
  hipLaunchKernelGGL(finite_kernel, dim3(grid_for(n)), dim3(256), 0, c->stream, p, n, c->err_dev);
  return hipGetLastError();
}

// ----------------------------------------------------------------- Gram --

// Split-K of the N_grid-long FP64 products X^T Y: 64 x 64 tiles, four workgroups
// per CU (LDS).  Taken: the number of splits with the least of (rounds of 1024
// workgroups, and 0.15 of one for their unequal ends) x (K range of one) plus the
// traffic of the partials.  Gram of 110592 x 512: 28 splits (one round) 600 us, 56 570 us,
// 108 595 us; projection 16 splits 917, 32 895.
constexpr int kGramTile = 64, kGramSlab = 16;
static void plan_gram(NtArgs& g) {
  const long tm = ceil_div(g.M, kGramTile), tn = ceil_div(g.N, kGramTile);
  const long tiles = g.upper ? tm * (tm + 1) / 2 : tm * tn;
  const long kblocks = (g.K + 63) / 64;
  constexpr long kSlots = 1024;
  // per 64 of K, one round of the chip: 1024 x 64^3 x 2 FLOP at 70 TFLOP/s, in us
  constexpr double kBlockUs = 1024.0 * 64 * 64 * 64 * 2 / 70e6;
  // a partial of one tile, written and read, at 4 TB/s
  constexpr double kPartUs = 64.0 * 64 * 8 * 2 / 4e6;
  double best = 0.0;
  for (long s = 1; s <= 128 && s <= kblocks; ++s) {
    const long per = (kblocks + s - 1) / s, splits = (kblocks + per - 1) / per;
    const double us = ((double)((tiles * splits + kSlots - 1) / kSlots) + 0.15) * per * kBlockUs +
                      (double)(tiles * splits) * kPartUs;
    if (s == 1 || us < best) {
      best = us;
      g.k_per_split = per * 64;
      g.splits = (int)splits;
    }
  }
}

// The split-BF16 projection runs 128 x 128 tiles (four 64 x 64 sub-tiles per
// wave: enough MFMA work per slab to cover the split of the fragments) over
// about 1024 workgroups, with FP32 partials (its accumulators are FP32).
constexpr int kProjTile = 128;
static void plan_projection(GemmArgs& g) {
  const long tiles = (long)ceil_div(g.M, kProjTile) * ceil_div(g.N, kProjTile);
  long want = 1024 / (tiles > 0 ? tiles : 1);
  const long kblocks = (g.K + 63) / 64;
  if (want > 128) want = 128;
  // FP32 accumulation: at most kF32SplitBlocks blocks per split
  const long least = (kblocks + kF32SplitBlocks - 1) / kF32SplitBlocks;
  if (want < least) want = least;
  if (want > kblocks) want = kblocks;
  if (want < 1) want = 1;
  const long per = (kblocks + want - 1) / want;
  g.k_per_split = (int)(per * 64);
  g.splits = (int)((kblocks + per - 1) / per);
}

size_t gram_ws_bytes(const dk_ctx* c, int n_s) {
  size_t bytes = 0;
  for (int upper = 0; upper < 2; ++upper) {
    NtArgs g;
    g.M = g.N = n_s;
    g.K = c->ngrid;
    g.upper = upper;
    plan_gram(g);
    const size_t b = (size_t)g.splits * n_s * n_s * sizeof(double);
    if (b > bytes) bytes = b;
  }
  if (c->precision == DK_PREC_MIXED) {
    GemmArgs p;
    p.M = n_s;
    p.N = n_s;
    p.K = (int)c->ngrid;
    plan_projection(p);
    const size_t pb = (size_t)p.splits * n_s * n_s * sizeof(float);
    if (pb > bytes) bytes = pb;
    // the same slice holds the pieces of L^{-T} for X L^{-T}
    if (split_planes_bytes(n_s, n_s, 3) > bytes) bytes = split_planes_bytes(n_s, n_s, 3);
  }
  return ws_slice(bytes);
}

// out = scale * X^T Y (n_s x n_s FP64).  symmetric_x: Y == X, only the upper
// tiles are computed and mirrored; otherwise the result is symmetrised.
// FP64 context: FP64 MFMA.  Mixed context: FP64 MFMA on the widened FP32
// block (Gram), or split-BF16 MFMA (bf16x3, projection: never symmetric_x).
hipError_t gram(dk_ctx* c, const void* x, const void* y, long ld, int n_s, bool symmetric_x,
                double scale, double* out, void* ws, bool bf16x3, int kind) {
  KTimer kt(c, kind);
  const dim3 rgrid(ceil_div(n_s, RT), ceil_div(n_s, RT));
  hipError_t e;
  if (c->precision == DK_PREC_MIXED && bf16x3) {
    GemmArgs p;
    p.M = n_s;
    p.N = n_s;
    p.K = (int)c->ngrid;
    p.A = x;
    p.lda = ld;
    p.B = y;
    p.ldb = ld;
    p.C = ws;
    plan_projection(p);
    e = launch_gemm<kBF16X3S, float, float, true, true, kPartial, float, kProjTile, kProjTile, 32>(
        p, c->stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_square_kernel<float>, rgrid, dim3(256), 0, c->stream,
                       (const float*)ws, p.splits, n_s, scale, 0, out);
    return hipGetLastError();
  }
  NtArgs g;
  g.M = g.N = n_s;
  g.K = c->ngrid;
  g.A = x;
  g.lda = ld;
  g.B = y;
  g.ldb = ld;
  g.C = (double*)ws;
  g.upper = symmetric_x ? 1 : 0;
  plan_gram(g);
  e = c->precision == DK_PREC_FP64
          ? launch_nt<double, double, true, kGramTile, kGramSlab, 4>(g, c->stream)
          : launch_nt<float, float, true, kGramTile, kGramSlab, 4>(g, c->stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(reduce_square_kernel<double>, rgrid, dim3(256), 0, c->stream,
                     (const double*)ws, g.splits, n_s, scale, symmetric_x ? 1 : 0, out);
  return hipGetLastError();
}

// ------------------------------------------------------------ Cholesky --

// linv receives L^{-1} (zero above the diagonal) of the symmetric positive definite
// g = L L^T (n x n, column-major); g is overwritten.  diag (n doubles) receives the
// diagonal of G; a pivot below 1e-14 of it sets kErrNotSpd.
hipError_t cholesky_inverse(dk_ctx* c, double* g, int n, double* linv, double* diag) {
  const int nb = ceil_div(n, NB);
  hipLaunchKernelGGL(chol_start_kernel, dim3(1 + grid_for((long)n * n)), dim3(256), 0, c->stream, g,
                     n, linv, diag, c->err_dev);
  for (int k = 0; k < nb; ++k) {
    const long tiles = (long)nb * (nb + 1) / 2 - (long)(k + 1) * (k + 2) / 2;
    const long wgs = k == nb - 1 ? k : tiles;
    if (wgs > 0)
      hipLaunchKernelGGL(chol_step_kernel, dim3((unsigned)wgs), dim3(256), 0, c->stream, g, n, k,
                         linv, diag, c->err_dev);
  }
  return hipGetLastError();
}

// ----------------------------------------------------- bf16 piece planes --

// The NP bf16 pieces of an FP64 matrix, as the split-at-store products would
// split it on its way into LDS (rounded to FP32, then x = hi + lo or
// hi + mid + lo): element (k, n) = src[k*s_k + n*s_n], piece p to
// dst[p*plane + n*ldp + k] (k-contiguous), zeros for K <= k < ldp.  32 x 32
// tiles pass through LDS so that both the read (along the source's contiguous
// index) and the write (along k) are coalesced.
template <int NP>
__global__ __launch_bounds__(256) void split_planes_kernel(const double* __restrict__ src,
                                                           long s_k, long s_n, int K, int N,
                                                           __bf16* __restrict__ dst, long ldp,
                                                           long plane) {
  __shared__ float t[32][33];  // t[k][n]
  const int k0 = blockIdx.x * 32, n0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const bool n_contig = (s_n == 1);
  for (int r = ty; r < 32; r += 8) {
    const int kl = n_contig ? r : tx, nl = n_contig ? tx : r;
    const int k = k0 + kl, n = n0 + nl;
    t[kl][nl] = (k < K && n < N) ? (float)src[(long)k * s_k + (long)n * s_n] : 0.f;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int n = n0 + r, k = k0 + tx;
    if (n >= N || k >= ldp) continue;
    const float v = t[tx][r];
    __bf16* o = dst + (long)n * ldp + k;
    if constexpr (NP == 3) {
      __bf16 h, m, l;
      split3_bf16(v, h, m, l);
      o[0] = h; o[plane] = m; o[2 * plane] = l;
    } else {
      __bf16 h, l;
      split_bf16(v, h, l);
      o[0] = h; o[plane] = l;
    }
  }
}

long split_planes_ld(int K) { return ((long)K + 7) / 8 * 8; }

size_t split_planes_bytes(int K, int N, int np) {
  return ws_slice((size_t)np * N * split_planes_ld(K) * sizeof(__bf16));
}

hipError_t split_planes(dk_ctx* c, const double* src, long s_k, long s_n, int K, int N, int np,
                        void* dst) {
  const long ldp = split_planes_ld(K);
  const dim3 grid(ceil_div(ldp, 32), ceil_div(N, 32));
  if (np == 3)
    hipLaunchKernelGGL(split_planes_kernel<3>, grid, dim3(256), 0, c->stream, src, s_k, s_n, K, N,
                       (__bf16*)dst, ldp, (long)N * ldp);
  else
    hipLaunchKernelGGL(split_planes_kernel<2>, grid, dim3(256), 0, c->stream, src, s_k, s_n, K, N,
                       (__bf16*)dst, ldp, (long)N * ldp);
  return hipGetLastError();
}

// out = X L^{-T}: B(k,j) = linv(j,k) is upper triangular (zero for k > j).
// Mixed: ws receives the bf16 pieces of B (split_planes_bytes(n_s, n_s, 3)).
hipError_t apply_right_upper(dk_ctx* c, const void* x, long ld, int n_s, const double* linv,
                             void* out, void* ws) {
  GemmArgs g;
  g.M = (int)c->ngrid;
  g.N = n_s;
  g.K = n_s;
  g.A = x;
  g.lda = ld;
  g.B = linv;
  g.ldb = n_s;
  g.C = out;
  g.ldc = ld;
  g.b_upper_tri = 1;
  g.xcd_groups = 0;  // measured faster in plain round-robin order
  if (c->precision == DK_PREC_FP64)
    return launch_gemm<kF64, double, double, false, false, kStore, double>(g, c->stream);
  // mixed: three-piece split-BF16 (FP32-level products for an FP32 result),
  // 128 x 128 tiles; X split once on its way into LDS, L^{-T} split beforehand
  hipError_t e = split_planes(c, linv, n_s, 1, n_s, n_s, 3, ws);
  if (e != hipSuccess) return e;
  g.B = ws;
  g.ldb = split_planes_ld(n_s);
  g.b_plane = (long)n_s * g.ldb;
  return launch_gemm<kBF16X6S, float, __bf16, false, true, kStore, float, 128, 128, 32>(g, c->stream);
}

// ------------------------------------------------------- spectral bounds --
//
// Extreme eigenvalues of the symmetric n x n H_s by shifted repeated squaring.
// For the largest: M = H - s I with s a Gershgorin lower bound (M positive
// semidefinite), X_0 = M / tr M, Y_k = X_k X_k (FP64 MFMA), X_{k+1} = Y_k / tr Y_k.
// X_k is proportional to M^(2^k), so the Rayleigh-type quotient
//   q_k = <M, Y_k>_F / tr Y_k = sum_i mu_i^(2^(k+1)+1) / sum_i mu_i^(2^(k+1))
// (mu_i the eigenvalues of M) converges to max mu with the error shrinking
// like (mu_2/mu_max)^(2^(k+1)): doubly exponentially once the top separates.
// lambda_max = q + s.  The smallest eigenvalue uses M = s' I - H with s'
// the Gershgorin upper bound, so the two sequences are independent and run
// side by side: a step is one batched GEMM of both, one reduction and one
// scaling; the host stops when both q change by less than 1e-15 relative.

namespace {

constexpr int SB_THREADS = 256;

__device__ double block_sum256(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) sh[w] = v;
  __syncthreads();
  const double s = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return s;
}

// per row i of sym(H): lower[i] = H_ii - sum_{j!=i} |H_ij|, upper[i] = H_ii + ...,
// diag[i] = H_ii (one wave per row)
__global__ __launch_bounds__(256) void gersh_rows_kernel(const double* __restrict__ h, int n,
                                                         double* __restrict__ lower,
                                                         double* __restrict__ upper,
                                                         double* __restrict__ diag) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= n) return;
  double off = 0.0;
  for (int k = lane; k < n; k += 64)
    if (k != r) off += fabs(0.5 * (h[k + (long)r * n] + h[r + (long)k * n]));
  for (int o = 32; o > 0; o >>= 1) off += __shfl_xor(off, o);
  if (lane == 0) {
    const double d = h[r + (long)r * n];
    lower[r] = d - off;
    upper[r] = d + off;
    diag[r] = d;
  }
}

// scal[0] = min lower, scal[1] = max upper, scal[2] = trace
__global__ __launch_bounds__(256) void gersh_reduce_kernel(const double* lower, const double* upper,
                                                           const double* diag, int n, double* scal) {
  __shared__ double sh[4];
  __shared__ double mn[256], mx[256];
  const int t = threadIdx.x;
  double a = 1e300, b = -1e300, tr = 0.0;
  for (int i = t; i < n; i += 256) { a = fmin(a, lower[i]); b = fmax(b, upper[i]); tr += diag[i]; }
  mn[t] = a;
  mx[t] = b;
  tr = block_sum256(tr, sh);
  __syncthreads();
  if (t == 0) {
    for (int i = 1; i < 256; ++i) { a = fmin(a, mn[i]); b = fmax(b, mx[i]); }
    scal[0] = fmin(a, mn[0]);
    scal[1] = fmax(b, mx[0]);
    scal[2] = tr;
  }
}

// blockIdx.y = mode; mode 0: M = sym(H) - s I, s = scal[0];  mode 1:
// M = s I - sym(H), s = scal[3].  X = M / tr M.  Mode m writes M + m n^2, X + m n^2,
// and sets its sequence's product scale alpha[m] = 1.
__global__ __launch_bounds__(256) void squaring_init_kernel(const double* __restrict__ h, int n,
                                                            const double* __restrict__ scal,
                                                            double* __restrict__ M,
                                                            double* __restrict__ X,
                                                            double* __restrict__ alpha) {
  const long nn = (long)n * n;
  const int mode = blockIdx.y;
  M += mode * nn;
  X += mode * nn;
  if (blockIdx.x == 0 && threadIdx.x == 0) alpha[mode] = 1.0;
  const double sft = mode == 0 ? scal[0] : scal[3];
  const double trm = mode == 0 ? scal[2] - n * sft : n * sft - scal[2];
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < nn;
       e += (long)gridDim.x * blockDim.x) {
    const int i = (int)(e % n), j = (int)(e / n);
    double v = 0.5 * (h[e] + h[(long)j + (long)i * n]);
    if (mode == 0) v = v - (i == j ? sft : 0.0);
    else v = (i == j ? sft : 0.0) - v;
    M[e] = v;
    X[e] = v / trm;
  }
}

// The end of a squaring, one workgroup per sequence: tr Y and <M, Y>_F from the `tiles`
// partials that its product left, the estimate <M, Y> / tr Y to pinned host memory, and
// 1 / (tr Y)^2, the scale of the next product Y' = alpha Y Y (= (Y / tr Y)^2).  (A kernel
// reading M and Y for the two sums took 10 us at n = 512 and 72 us at n = 2048, and the
// copy of the estimates with the gaps around it 13 us; this one and its gap 5.)
__global__ __launch_bounds__(256) void squaring_finish_kernel(const double* __restrict__ part,
                                                              long tiles, double* host_est,
                                                              int est_stride,
                                                              double* __restrict__ alpha) {
  __shared__ double sh[4];
  part += 2 * tiles * blockIdx.x;
  double t = 0.0, m = 0.0;
  for (long i = threadIdx.x; i < tiles; i += 256) {
    t += part[2 * i];
    m += part[2 * i + 1];
  }
  t = block_sum256(t, sh);
  m = block_sum256(m, sh);
  if (threadIdx.x == 0) {
    host_est[blockIdx.x * est_stride] = m / t;
    alpha[blockIdx.x] = 1.0 / (t * t);
  }
}

__global__ void set_scalar_kernel(double* p, double v) { p[0] = v; }

constexpr int SB_MAX_STEPS = 48;
// partial sums of a squaring: two per tile of two sequences
size_t sb_parts(int n) {
  const size_t t = ceil_div(n, kSymmetricTile);
  return 4 * (t * (t + 1) / 2);
}

}  // namespace

size_t spectral_ws_bytes(int n) {
  const size_t nn = (size_t)n * n;
  return 3 * ws_slice(2 * nn * sizeof(double)) + 3 * ws_slice((size_t)n * sizeof(double)) +
         ws_slice(8 * sizeof(double)) + ws_slice(sb_parts(n) * sizeof(double)) +
         ws_slice(2 * sizeof(double));
}

// Both squaring sequences side by side (M, X, Y hold the two n x n
// matrices back to back); q[0], q[1] are the converged quotients, *steps the
// squarings taken (both sequences counted).  A sequence that has converged is left where it is and the
// other runs on alone.  X and Y alternate as the input and output of the
// squarings; each product carries the normalisation 1 / (tr)^2 of its input
// (alpha, set by the statistics of the step before), so no pass rescales the
// matrices.
static hipError_t squaring_pair(dk_ctx* c, const double* hs, int n, double* M, double* X,
                                double* Y, double* scal, double* part, double* alpha, double* q,
                                int* steps) {
  const long nn = (long)n * n;
  const int eblocks = (int)((nn + 255) / 256 < 4096 ? (nn + 255) / 256 : 4096);
  hipLaunchKernelGGL(squaring_init_kernel, dim3(eblocks, 2), dim3(256), 0, c->stream, hs, n, scal,
                     M, X, alpha);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  double cur[2] = {0, 0};
  bool done_m[2] = {false, false};
  bool conv = false;
  int k = 0, squarings = 0;
  // For N_s <= 1024 the host checks step k - 1 while step k runs: each step's
  // estimates go to their places in pinned memory and an event marks the step
  // done, so the GPU does not idle during the check (a converged sequence
  // may run one squaring more, which is discarded): al32 0.86 -> 0.72 ms.
  // Larger matrices check each step as it ends (a squaring outweighs the wait).
  // (Two steps behind was slower: 0.72 -> 0.77 ms.)
  const int lag = n <= 1024 ? 1 : 0;
  constexpr int kBufs = 2;
  if (!c->sb_host) {
    if ((e = hipHostMalloc((void**)&c->sb_host, 2 * SB_MAX_STEPS * sizeof(double))) !=
        hipSuccess)
      return e;
    for (hipEvent_t& ev : c->sb_ev)
      if ((e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) != hipSuccess) return e;
  }
  for (; k < SB_MAX_STEPS; ++k) {
    // the sequences still running: [first, first + active)
    const int first = done_m[0] ? 1 : 0;
    const int active = (done_m[0] ? 0 : 1) + (done_m[1] ? 0 : 1);
    double* P = (k & 1) ? Y : X;  // this step's input
    double* Q = (k & 1) ? X : Y;  // and output
    NtArgs g;
    g.M = n; g.N = n; g.K = n;
    g.A = P + first * nn; g.lda = n;
    g.B = P + first * nn; g.ldb = n;
    g.C = Q + first * nn; g.ldc = n;
    g.alpha_dev = alpha + first;
    g.batch = active;
    squarings += active;
    g.bs_a = g.bs_b = g.bs_c = nn;
    // X_k is symmetric (a power of M): upper tiles only, mirrored; the product also leaves
    // the estimate and the scale of the next one
    g.S = M + first * nn;
    g.part = part;
    e = symmetric_product(g, c->stream);
    if (e != hipSuccess) return e;
    const long t = ceil_div(n, symmetric_tile(n, active));
    hipLaunchKernelGGL(squaring_finish_kernel, dim3(active), dim3(256), 0, c->stream, part,
                       t * (t + 1) / 2, c->sb_host + first * SB_MAX_STEPS + k, SB_MAX_STEPS,
                       alpha + first);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipEventRecord(c->sb_ev[k % kBufs], c->stream)) != hipSuccess) return e;
    const int j = k - lag;  // the step checked now
    if (j >= 5) {
      if ((e = hipEventSynchronize(c->sb_ev[j % kBufs])) != hipSuccess) return e;
      const double* two = c->sb_host;
      bool finite = true;
      for (int m = 0; m < 2; ++m) {
        if (done_m[m]) continue;
        const double prev = two[m * SB_MAX_STEPS + j - 1];
        cur[m] = two[m * SB_MAX_STEPS + j];
        if (fabs(cur[m] - prev) <= 1e-15 * fabs(cur[m])) done_m[m] = true;
        finite = finite && std::isfinite(cur[m]);
      }
      if ((done_m[0] && done_m[1]) || !finite) { conv = done_m[0] && done_m[1]; ++k; break; }
    }
  }
  if (!conv && k >= SB_MAX_STEPS) {
    unsigned flag = 0;
    hipMemcpy(&flag, c->err_dev, sizeof flag, hipMemcpyDeviceToHost);
    flag |= kErrConvergence;
    hipMemcpy(c->err_dev, &flag, sizeof flag, hipMemcpyHostToDevice);
  }
  if (!std::isfinite(cur[0]) || !std::isfinite(cur[1])) {
    unsigned flag = 0;
    hipMemcpy(&flag, c->err_dev, sizeof flag, hipMemcpyDeviceToHost);
    flag |= kErrNonFinite;
    hipMemcpy(c->err_dev, &flag, sizeof flag, hipMemcpyHostToDevice);
  }
  q[0] = cur[0];
  q[1] = cur[1];
  *steps = squarings;
  return hipSuccess;
}

hipError_t spectral_bounds(dk_ctx* c, const double* hs, int n, void* ws, double* lo, double* hi,
                           int* iters) {
  const size_t nn = (size_t)n * n;
  WsCursor cur((char*)ws, spectral_ws_bytes(n));
  double* M = cur.take<double>(2 * nn);
  double* X = cur.take<double>(2 * nn);
  double* Y = cur.take<double>(2 * nn);
  double* lower = cur.take<double>(n);
  double* upper = cur.take<double>(n);
  double* diag = cur.take<double>(n);
  double* scal = cur.take<double>(8);
  double* part = cur.take<double>(sb_parts(n));
  double* alpha = cur.take<double>(2);
  if (!cur.ok) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gersh_rows_kernel, dim3((n + 3) / 4), dim3(256), 0, c->stream, hs, n, lower,
                     upper, diag);
  hipLaunchKernelGGL(gersh_reduce_kernel, dim3(1), dim3(256), 0, c->stream, lower, upper, diag, n,
                     scal);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  double gl[3];
  e = hipMemcpyAsync(gl, scal, 3 * sizeof(double), hipMemcpyDeviceToHost, c->stream);
  if (e != hipSuccess) return e;
  if ((e = hipStreamSynchronize(c->stream)) != hipSuccess) return e;
  // a Gershgorin interval of (numerically) zero width pins both eigenvalues
  // (n = 1, or H_s a multiple of the identity): M would vanish
  const double gscale = fmax(1.0, fmax(fabs(gl[0]), fabs(gl[1])));
  if (n == 1 || gl[1] - gl[0] <= 1e-13 * gscale) {
    *lo = gl[0];
    *hi = gl[1];
    if (n == 1) *lo = *hi = gl[2];
    if (iters) *iters = 0;
    return hipSuccess;
  }
  // shift for the smallest: the Gershgorin upper bound, nudged up so that
  // s'I - H stays semidefinite through rounding
  const double sh = gl[1] + 1e-12 * (1.0 + fabs(gl[1])) + 1e-12 * (gl[1] - gl[0]);
  hipLaunchKernelGGL(set_scalar_kernel, dim3(1), dim3(1), 0, c->stream, scal + 3, sh);
  double q[2] = {0, 0};
  int k = 0;
  if ((e = squaring_pair(c, hs, n, M, X, Y, scal, part, alpha, q, &k)) != hipSuccess)
    return e;
  *hi = q[0] + gl[0];
  *lo = sh - q[1];
  if (iters) *iters = k;
  return hipSuccess;
}

}  // namespace dk
