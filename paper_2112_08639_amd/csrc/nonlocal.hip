// Projector integrals over the dense tables, for the forces and the stress:
//
//   out = scale * table^T X      (m rows x N_s; split over the grid, partials)
//
// with the table an FP64 N_grid x m array of projector values and / or their
// finite-difference gradients.  (The nonlocal term of H X runs over the compact
// supports, sweep.hip.)  Mixed path: three-piece split-BF16, FP32 partials.
#include <type_traits>

#include "ctx.h"
#include "gemm.h"

namespace dk {

namespace {

// out[e] = scale * sum_s part[s * mn + e].  A block owns 64 consecutive entries; its four
// waves sum interleaved quarters of the splits (two independent chains each), then combine
// in LDS.
template <typename PT>
__global__ __launch_bounds__(256) void reduce_rows_kernel(const PT* __restrict__ part, int splits,
                                                          long mn, double scale,
                                                          double* __restrict__ out) {
  __shared__ double sh[4][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (long e0 = blockIdx.x * 64L; e0 < mn; e0 += (long)gridDim.x * 64) {
    const long e = e0 + lane;
    double s0 = 0.0, s1 = 0.0;
    if (e < mn) {
      int k = wv;
      for (; k + 4 < splits; k += 8) {
        s0 += (double)part[(long)k * mn + e];
        s1 += (double)part[(long)(k + 4) * mn + e];
      }
      for (; k < splits; k += 4) s0 += (double)part[(long)k * mn + e];
    }
    sh[wv][lane] = s0 + s1;
    __syncthreads();
    if (wv == 0 && e < mn) {
      const double s = (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
      out[e] = s * scale;
    }
    __syncthreads();
  }
}

// The mixed path takes 128 x 128 tiles of three-piece split-BF16 MFMA (FP32-level
// products) once there are more than 64 rows; smaller tables 64-row FP32 tiles.
bool wide_tiles(const dk_ctx* c, int m) { return c->precision == DK_PREC_MIXED && m > 64; }

// Split count: about 2048 workgroups of 128x64 tiles (latency hiding needs many
// workgroups per CU), 1024 of the wide ones.
int integral_splits(const dk_ctx* c, int m, int n_s) {
  const bool wide = wide_tiles(c, m);
  const long tiles = (long)ceil_div(m, 128) * ceil_div(n_s, wide ? 128 : 64);
  const long kblocks = (c->ngrid + 63) / 64;
  long want = (wide ? 1024 : 2048) / (tiles > 0 ? tiles : 1);
  if (c->precision == DK_PREC_MIXED) {
    // FP32 accumulation: at most kF32SplitBlocks blocks per split
    const long least = (kblocks + kF32SplitBlocks - 1) / kF32SplitBlocks;
    if (want < least) want = least;
  }
  if (want > kblocks) want = kblocks;
  if (want < 1) want = 1;
  const long per = (kblocks + want - 1) / want;
  return (int)((kblocks + per - 1) / per);
}

// partials of an FP32-accumulating product are stored in FP32 (lossless)
template <int MODE> using PartialT = typename std::conditional<MODE == kF64, double, float>::type;

// out (m x n_s FP64) = scale * table^T X, X of type TX
template <int MODE, typename TX>
hipError_t table_transpose_product(dk_ctx* c, const double* table, const void* x, long ld, int n_s,
                                   double scale, double* out, void* part_raw, int m) {
  using PT = PartialT<MODE>;
  PT* part = (PT*)part_raw;
  GemmArgs g;
  g.M = m;
  g.N = n_s;
  g.K = (int)c->ngrid;
  g.A = table;
  g.lda = c->ngrid;
  g.B = x;
  g.ldb = ld;
  g.C = part;
  {
    const int want = integral_splits(c, m, n_s);
    const long kblocks = (g.K + 63) / 64;
    const long per = (kblocks + want - 1) / want;
    g.k_per_split = (int)(per * 64);
    g.splits = (int)((kblocks + per - 1) / per);
  }
  hipError_t e;
  if constexpr (MODE == kF32)
    // FP32 slabs of 32 give 128-byte row segments
    e = wide_tiles(c, m)
            ? launch_gemm<kBF16X6S, double, TX, true, true, kPartial, PT, 128, 128, 32>(g, c->stream)
            : launch_gemm<MODE, double, TX, true, true, kPartial, PT, 64, 64, 32>(g, c->stream);
  else
    e = (m > 64) ? launch_gemm<MODE, double, TX, true, true, kPartial, PT, 128, 64>(g, c->stream)
                 : launch_gemm<MODE, double, TX, true, true, kPartial, PT, 64, 64>(g, c->stream);
  if (e != hipSuccess) return e;
  const long mn = (long)g.M * g.N;
  int blocks = (int)((mn + 63) / 64);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(reduce_rows_kernel<PT>, dim3(blocks), dim3(256), 0, c->stream, part, g.splits,
                     mn, scale, out);
  return hipGetLastError();
}

}  // namespace

size_t projector_integrals_ws_bytes(const dk_ctx* c, int n_s, int m_rows) {
  const size_t elem = c->precision == DK_PREC_FP64 ? sizeof(double) : sizeof(float);
  return ws_slice((size_t)integral_splits(c, m_rows, n_s) * m_rows * n_s * elem);
}

// out (m_rows x n_s FP64) = scale * table^T X for an FP64 N_grid x m_rows table
// (projector values and/or their finite-difference gradients); X in the
// context precision.
hipError_t projector_integrals(dk_ctx* c, const void* x, long ld, int n_s, const void* table,
                               int m_rows, double scale, double* out, void* ws) {
  if (m_rows == 0 || n_s <= 0) return hipSuccess;
  WsCursor cur((char*)ws, projector_integrals_ws_bytes(c, n_s, m_rows));
  void* part = cur.take<char>(projector_integrals_ws_bytes(c, n_s, m_rows));
  if (!cur.ok) return hipErrorInvalidValue;
  if (c->precision == DK_PREC_FP64)
    return table_transpose_product<kF64, double>(c, (const double*)table, x, ld, n_s, scale, out,
                                                 part, m_rows);
  return table_transpose_product<kF32, float>(c, (const double*)table, x, ld, n_s, scale, out, part,
                                              m_rows);
}

}  // namespace dk
