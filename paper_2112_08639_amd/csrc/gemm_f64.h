// FP64 MFMA products of two k-contiguous operands,
//   C(M x N) = sum_k A(m,k) B(k,n),   A(m,k) = A[m*lda + k], B(k,n) = B[n*ldb + k],
// for the Gram and projection products X^T Y over the grid (X, Y column-major, FP32 or
// FP64) and for products of symmetric N_s x N_s matrices.
//
// One workgroup (4 waves, 2 x 2) computes a BT x BT tile over a K range.  Slabs of BK
// are loaded along k (whole runs of each row), widened to FP64 and staged in LDS: two
// buffers, one barrier per slab, the next slab in registers while MFMA runs the current
// one.  The bound is the FP64 matrix rate, and a 16x16x4 MFMA holds its pipe for 64
// cycles; what keeps it busy is that little else is issued between: the row pointers
// are set up once (rows past the end repeat the last one and are not stored), only the
// last slab of a range is guarded, and a lane reads four consecutive k of its row at
// once (MFMA step r takes k = 4 g + r of every 16, the same for both operands).  Rows
// of BK + 2 doubles start four banks apart, so these 16-byte reads have no conflicts.
//
// Measured (the general LDS-tiled template before): Gram of 110592 x 512 in FP32 0.86 ->
// 0.56 ms (33 GFLOP: 59 of the 73 TFLOP/s a large FP64 product reaches), in FP64 0.81 ->
// 0.53 ms; of 373248 x 2048 in FP32 35 -> 26 ms; projection of 110592 x 512 1.09 ->
// 0.90 ms.  Tiles of 128 (0.58 ms) and slabs of 32 (0.58 ms) gain nothing at the Gram.
#pragma once

#include <algorithm>

#include "common.h"
#include "gemm.h"

namespace dk {

typedef double f64x2_m __attribute__((ext_vector_type(2)));
typedef double f64x2_ld __attribute__((ext_vector_type(2), aligned(8)));
typedef float f32x4_ld __attribute__((ext_vector_type(4), aligned(4)));

struct NtArgs {
  int M = 0, N = 0;
  long K = 0;
  const void* A = nullptr;
  long lda = 0;
  const void* B = nullptr;
  long ldb = 0;
  double* C = nullptr;       // store: output; partial: [split][M x N]
  long ldc = 0;
  const double* Cin = nullptr;
  long ldcin = 0;
  double alpha = 1.0, beta = 0.0;
  const double* alpha_dev = nullptr;  // store: alpha is multiplied by alpha_dev[b]
  int splits = 1;
  long k_per_split = 0;
  int batch = 1;             // (no split-K) operand b is offset by b times these
  long bs_a = 0, bs_b = 0, bs_c = 0, bs_cin = 0;
  int upper = 0;             // square: the tiles of the upper triangle only
  int mirror = 0;            // with upper, store: each off-diagonal tile's transpose too
  // with mirror: per tile of every operand of the batch, the tile's share (and its
  // mirror image's) of tr C and <S, C>_F of the symmetric result, S bs_c apart
  const double* S = nullptr;
  double* part = nullptr;
};

// Slab loader of one operand: BT rows by BK, along k.
template <typename T, int BT, int BK>
struct NtSlab {
  static constexpr int E = sizeof(T) == 4 ? 4 : 2;        // elements per 16-byte load
  static constexpr int LPR = BK / E;                      // lanes per row
  static constexpr int RPP = 256 / LPR;                   // rows per pass of the workgroup
  static constexpr int N = (BT + RPP - 1) / RPP;          // passes
  static constexpr int P = BK + 2;
  static_assert(BT % RPP == 0, "whole passes");
  const T* p[N];
  int at;  // LDS position of the first pass
  T v[N][E];

  __device__ __forceinline__ void init(const T* base, long ld, int row0, int rows, long k0, int tid) {
    const int r = tid / LPR, k = (tid % LPR) * E;
    at = r * P + k;
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = base + (long)min(row0 + r + RPP * i, rows - 1) * ld + k0 + k;
  }
  __device__ __forceinline__ void load() {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if constexpr (sizeof(T) == 4) {
        const f32x4_ld u = *reinterpret_cast<const f32x4_ld*>(p[i]);
#pragma unroll
        for (int j = 0; j < E; ++j) v[i][j] = u[j];
      } else {
        const f64x2_ld u = *reinterpret_cast<const f64x2_ld*>(p[i]);
#pragma unroll
        for (int j = 0; j < E; ++j) v[i][j] = u[j];
      }
      p[i] += BK;
    }
  }
  // the last, partial slab: `left` elements of k, zeros beyond
  __device__ __forceinline__ void load_tail(int left, int tid) {
    const int k = (tid % LPR) * E;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < E; ++j) v[i][j] = k + j < left ? p[i][j] : (T)0;
  }
  __device__ __forceinline__ void store(double* s) const {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < E; j += 2)
        *reinterpret_cast<f64x2_m*>(s + at + RPP * i * P + j) =
            f64x2_m{(double)v[i][j], (double)v[i][j + 1]};
  }
};

template <typename TA, typename TB, bool PARTIAL, int BT, int BK, int OCC>
__global__ __launch_bounds__(256, OCC) void nt_f64_kernel(NtArgs a) {
  constexpr int P = BK + 2;
  constexpr int W = BT / 2;    // a wave's rows and columns
  constexpr int MI = W / 16;   // 16 x 16 blocks per side
  extern __shared__ __attribute__((aligned(16))) double nt_lds[];  // [2][A, B][BT][P]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, c16 = lane & 15;
  const int tm = (a.M + BT - 1) / BT, tn = (a.N + BT - 1) / BT;
  const long tiles = a.upper ? (long)tm * (tm + 1) / 2 : (long)tm * tn;
  const long w = xcd_work_item(blockIdx.x, (long)gridDim.x);
  const long zi = w / tiles;
  const int tile = (int)(w - zi * tiles);
  int mt, nt;
  if (a.upper) {
    nt = (int)((sqrtf(8.0f * tile + 1.0f) - 1.0f) * 0.5f);
    while ((long)(nt + 1) * (nt + 2) / 2 <= tile) ++nt;
    while ((long)nt * (nt + 1) / 2 > tile) --nt;
    mt = tile - (int)((long)nt * (nt + 1) / 2);
  } else {
    mt = tile % tm;
    nt = tile / tm;
  }
  const int m0 = mt * BT, n0 = nt * BT;
  const long bi = PARTIAL ? 0 : zi;
  const long k0 = PARTIAL ? zi * a.k_per_split : 0;
  const long klen = PARTIAL ? min(a.k_per_split, a.K - k0) : a.K;
  NtSlab<TA, BT, BK> sa;
  NtSlab<TB, BT, BK> sb;
  sa.init((const TA*)a.A + bi * a.bs_a, a.lda, m0, a.M, k0, tid);
  sb.init((const TB*)a.B + bi * a.bs_b, a.ldb, n0, a.N, k0, tid);
  const int slabs = (int)((klen + BK - 1) / BK), whole = (int)(klen / BK);
  auto fetch = [&](int i) {
    if (i < whole) {
      sa.load();
      sb.load();
    } else if (i < slabs) {
      sa.load_tail((int)(klen - (long)whole * BK), tid);
      sb.load_tail((int)(klen - (long)whole * BK), tid);
    }
  };
  const int wm = (wave & 1) * W, wn = (wave >> 1) * W;
  f64x4 acc[MI][MI];  // [n block][m block]
#pragma unroll
  for (int j = 0; j < MI; ++j)
#pragma unroll
    for (int i = 0; i < MI; ++i) acc[j][i] = f64x4{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  for (int t = 0; t < slabs; ++t) {
    double* const s = nt_lds + (t & 1) * (2 * BT * P);
    sa.store(s);
    sb.store(s + BT * P);
    __syncthreads();
    fetch(t + 1);
    const double* const pa = s + (wm + c16) * P + 4 * g;
    const double* const pb = s + BT * P + (wn + c16) * P + 4 * g;
#pragma unroll
    for (int kk = 0; kk < BK; kk += 16) {
      f64x2_m fa[MI][2], fb[MI][2];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          fa[i][h] = *reinterpret_cast<const f64x2_m*>(pa + 16 * i * P + kk + 2 * h);
          fb[i][h] = *reinterpret_cast<const f64x2_m*>(pb + 16 * i * P + kk + 2 * h);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
          for (int i = 0; i < MI; ++i)
            acc[j][i] = mfma_f64(fb[j][r >> 1][r & 1], fa[i][r >> 1][r & 1], acc[j][i]);
    }
  }
  double trace = 0.0, dot = 0.0;  // of this lane's elements, the mirrored ones included
  // lane: m = c16 of block i, n = g + 4 q of block j
#pragma unroll
  for (int j = 0; j < MI; ++j)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + wm + 16 * i + c16, n = n0 + wn + 16 * j + g + 4 * q;
        if (m >= a.M || n >= a.N) continue;
        const double v = acc[j][i][q];
        if constexpr (PARTIAL) {
          a.C[(zi * a.N + n) * a.M + m] = v;
        } else {
          double out = (a.alpha_dev ? a.alpha * a.alpha_dev[bi] : a.alpha) * v;
          if (a.beta != 0.0) out += a.beta * (a.Cin + bi * a.bs_cin)[m + (long)n * a.ldcin];
          double* const C = a.C + bi * a.bs_c;
          C[m + (long)n * a.ldc] = out;
          if (a.mirror && mt != nt) C[n + (long)m * a.ldc] = out;
          if (a.S) {
            const double v2 = (a.S + bi * a.bs_c)[m + (long)n * a.ldc] * out;
            dot += mt != nt ? 2.0 * v2 : v2;
            if (m == n) trace += out;
          }
        }
      }
  if constexpr (!PARTIAL) {
    if (!a.S) return;
    for (int o = 32; o > 0; o >>= 1) {
      trace += __shfl_xor(trace, o);
      dot += __shfl_xor(dot, o);
    }
    __syncthreads();  // the slabs are done with
    if (lane == 0) {
      nt_lds[2 * wave] = trace;
      nt_lds[2 * wave + 1] = dot;
    }
    __syncthreads();
    if (tid < 2)
      a.part[2 * (bi * tiles + tile) + tid] =
          (nt_lds[tid] + nt_lds[2 + tid]) + (nt_lds[4 + tid] + nt_lds[6 + tid]);
  }
}

constexpr size_t nt_lds_bytes(int BT, int BK) { return (size_t)4 * BT * (BK + 2) * sizeof(double); }

template <typename TA, typename TB, bool PARTIAL, int BT, int BK, int OCC>
inline hipError_t launch_nt(const NtArgs& a, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  const long tm = ceil_div(a.M, BT), tn = ceil_div(a.N, BT);
  const long tiles = a.upper ? tm * (tm + 1) / 2 : tm * tn;
  const long z = PARTIAL ? a.splits : a.batch;
  constexpr size_t lds = nt_lds_bytes(BT, BK);
  const auto kernel = nt_f64_kernel<TA, TB, PARTIAL, BT, BK, OCC>;
  static_assert(lds <= 64 * 1024, "no limit to raise");
  hipLaunchKernelGGL(kernel, dim3((unsigned)(tiles * z)), dim3(256), lds, st, a);
  return hipGetLastError();
}

// A product of symmetric n x n matrices that is symmetric itself (powers and
// Chebyshev polynomials of one matrix): the upper tiles, each mirrored into the lower.
// Below 512 tiles of 64 x 64 (half of the workgroups the chip holds) 32 x 32 tiles spread
// the work wider.  At n = 512: 1 product 10 against 25 us, 2 15.8 against 25.5, 8 (288
// tiles) 32 against 44; from 32 on (1152 tiles) 64 x 64 run at the matrix rate (94 us,
// 46 TFLOP/s counted over the upper triangle).  Against the general template: two squarings at
// n = 512 20.6 -> 15.8 us, at n = 2048 0.60 -> 0.36 ms.
constexpr int kSymmetricTile = 32;  // the smaller of the two
inline int symmetric_tile(int n, int batch) {
  const long t = ceil_div(n, 64);
  return t * (t + 1) / 2 * batch < 512 ? kSymmetricTile : 64;
}
inline hipError_t symmetric_product(NtArgs g, hipStream_t st) {
  g.upper = 1;
  g.mirror = 1;
  if (symmetric_tile(g.M, g.batch) == kSymmetricTile)
    return launch_nt<double, double, false, 32, 32, 4>(g, st);
  return launch_nt<double, double, false, 64, 16, 4>(g, st);
}

}  // namespace dk
