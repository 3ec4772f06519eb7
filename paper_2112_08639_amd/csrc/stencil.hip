// Local part of the Hamiltonian on a block of grid vectors, fused with the
// Chebyshev-filter update:
//
//   Y_out = alpha * ((-1/2 Lap_h + V_eff - shift) Y_in) + beta * Y_prev
//
// -1/2 Lap_h is the twelfth-order central-difference kinetic operator of the
// paper's real-space discretisation (Sec. 5): a 37-point star of radius 6,
// periodic in x, y, z.  Y_prev may alias Y_out (the recurrence overwrites
// Y_{k-1} with Y_{k+1} point by point).  The nonlocal projector term is added
// by nonlocal_scatter.
//
// Kernel layout.  All kernels stream planes; the first and general one, for rows of any
// length: a workgroup owns one column of the block, TY full x-rows of
// an xy-plane, and streams through a chunk of z-planes.  Each thread keeps the
// 13 values of its points' z-columns in registers (a queue shifted once per
// plane), so every value of Y_in is loaded from memory once per chunk plus a
// 12-plane prologue.  The centre plane of the tile, with 6 periodic halo rows
// above and below, is staged in LDS for the x and y neighbours; x wraps within
// the row.
#include <algorithm>
#include <cmath>
#include <utility>

#include "ctx.h"

namespace dk {

struct StencilArgs {
  const void* yin;
  const void* yprev;
  void* yout;
  const void* veff;
  long ld;
  int nx, ny, nz;
  int ty_tile;  // rows per tile
  int zc;       // planes per z-chunk
  double cx[7], cy[7], cz[7];  // -1/2 w_k / h_a^2, k = 1..6 (index 0 unused)
  double alpha, beta, shift;
  // the same in FP32, converted once on the host (uniform SGPR operands)
  float fcx[7], fcy[7], fcz[7];
  float falpha, fbeta, fshift;
};

// (a + b) - 2 c with one rounding of the difference.  The kinetic term is
// accumulated as sum_k c_k ((x_{+k} + x_{-k}) - 2 x_0) per axis rather than
// as diag x_0 + sum_k c_k (x_{+k} + x_{-k}): the running sum then stays at the
// size of the kinetic term instead of cancelling diag x_0 (~45 Ha x_0 at
// h = 0.32 bohr), and a constant is annihilated exactly whatever the rounding
// of the coefficients.  In FP32 the other form shifts smooth states by
// ~3e-6 Ha (the rounded coefficients do not sum to zero) plus a correlated
// rounding bias of the cancelling sums.
template <typename T>
__device__ __forceinline__ T pair_d2(T a, T b, T c) {
  if constexpr (sizeof(T) == 4) return __builtin_fmaf(-2.0f, c, a + b);
  else return __builtin_fma(-2.0, c, a + b);
}

template <typename T, int PPT>
__global__ __launch_bounds__(256) void stencil_kernel(StencilArgs a) {
  extern __shared__ unsigned char smem_raw[];
  T* plane = reinterpret_cast<T*>(smem_raw);
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const long pstride = (long)nx * ny;
  const int col = blockIdx.z;
  const int y0 = blockIdx.x * a.ty_tile;
  const int ty = min(a.ty_tile, ny - y0);
  const int z0 = blockIdx.y * a.zc;
  const int z1 = min(nz, z0 + a.zc);
  const int npts = nx * ty;
  const int tid = threadIdx.x;

  const T* __restrict__ yin = reinterpret_cast<const T*>(a.yin) + (long)col * a.ld;
  const T* __restrict__ yprev =
      a.yprev ? reinterpret_cast<const T*>(a.yprev) + (long)col * a.ld : nullptr;
  T* yout = reinterpret_cast<T*>(a.yout) + (long)col * a.ld;
  const T* __restrict__ veff = reinterpret_cast<const T*>(a.veff);

  T cx[7], cy[7], cz[7];
#pragma unroll
  for (int k = 0; k < 7; ++k) { cx[k] = (T)a.cx[k]; cy[k] = (T)a.cy[k]; cz[k] = (T)a.cz[k]; }
  const T alpha = (T)a.alpha, beta = (T)a.beta, vshift = (T)a.shift;

  int px[PPT], prow[PPT];
  long poff[PPT];
  bool pval[PPT];
  T q[PPT][13];
#pragma unroll
  for (int r = 0; r < PPT; ++r) {
    const int p = tid + 256 * r;
    pval[r] = p < npts;
    px[r] = pval[r] ? p % nx : 0;
    prow[r] = pval[r] ? p / nx : 0;
    poff[r] = px[r] + (long)nx * (y0 + prow[r]);
  }
  // prologue: planes z0-6 .. z0+5
#pragma unroll
  for (int d = 0; d < 12; ++d) {
    int zz = z0 - 6 + d;
    zz = ((zz % nz) + nz) % nz;
#pragma unroll
    for (int r = 0; r < PPT; ++r) q[r][d] = pval[r] ? yin[zz * pstride + poff[r]] : (T)0;
  }
  const int halo_n = 12 * nx;

  for (int z = z0; z < z1; ++z) {
    int zn = z + 6;
    if (zn >= nz) zn -= nz;
#pragma unroll
    for (int r = 0; r < PPT; ++r) q[r][12] = pval[r] ? yin[zn * pstride + poff[r]] : (T)0;
    // centre plane of the tile into LDS (row offset 6)
#pragma unroll
    for (int r = 0; r < PPT; ++r)
      if (pval[r]) plane[(prow[r] + 6) * nx + px[r]] = q[r][6];
    for (int e = tid; e < halo_n; e += 256) {
      const int hr = e / nx, hx = e - hr * nx;
      const int row = hr < 6 ? hr - 6 : ty + hr - 6;
      int gy = y0 + row;
      gy = ((gy % ny) + ny) % ny;
      plane[(row + 6) * nx + hx] = yin[(long)z * pstride + hx + (long)nx * gy];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PPT; ++r) {
      if (!pval[r]) continue;
      const int x = px[r];
      const T* rowp = plane + (prow[r] + 6) * nx;
      const long g = (long)z * pstride + poff[r];
      const T x0 = q[r][6];
      T acc = 0;
#pragma unroll
      for (int k = 1; k <= kFdRadius; ++k) {
        int xp = x + k; if (xp >= nx) xp -= nx;
        int xm = x - k; if (xm < 0) xm += nx;
        acc += cx[k] * pair_d2(rowp[xp], rowp[xm], x0);
        acc += cy[k] * pair_d2(rowp[x + k * nx], rowp[x - k * nx], x0);
        acc += cz[k] * pair_d2(q[r][6 + k], q[r][6 - k], x0);
      }
      acc += (veff[g] - vshift) * x0;
      T out = alpha * acc;
      if (yprev) out += beta * yprev[g];
      yout[g] = out;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PPT; ++r)
#pragma unroll
      for (int d = 0; d < 12; ++d) q[r][d] = q[r][d + 1];
  }
}

// Whole-plane variant for planes of at most 4096 points with nx % 4 == 0.
// A workgroup owns one column and a chunk of z-planes; thread t owns the four
// consecutive points x0..x0+3 of row y (x0 = 4 (t % (nx/4)), y = t / (nx/4)),
// moved as one 16-byte (float) or 32-byte (double) vector.  Its 13-plane
// z-queue lives in registers and the load of the plane entering the queue is
// issued one step ahead.  The centre plane goes to one of two LDS buffers whose
// rows carry 8 periodic copies on each side, so the x and y neighbours are
// aligned vector reads with no wrap test; y wraps by row index.  One barrier
// per plane (double buffering).
template <typename T>
struct Vec4 { T v[4]; };

template <typename T>
__device__ __forceinline__ Vec4<T> ld4(const T* p) {
  Vec4<T> r;
  if constexpr (sizeof(T) == 4) {
    const float4 f = *reinterpret_cast<const float4*>(p);
    r.v[0] = f.x; r.v[1] = f.y; r.v[2] = f.z; r.v[3] = f.w;
  } else {
    const double2 a = *reinterpret_cast<const double2*>(p);
    const double2 b = *reinterpret_cast<const double2*>(p + 2);
    r.v[0] = a.x; r.v[1] = a.y; r.v[2] = b.x; r.v[3] = b.y;
  }
  return r;
}

template <typename T>
__device__ __forceinline__ void st4(T* p, const Vec4<T>& r) {
  if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<float4*>(p) = make_float4(r.v[0], r.v[1], r.v[2], r.v[3]);
  } else {
    *reinterpret_cast<double2*>(p) = make_double2(r.v[0], r.v[1]);
    *reinterpret_cast<double2*>(p + 2) = make_double2(r.v[2], r.v[3]);
  }
}

constexpr int kPad = 8;  // periodic copies on each side of an LDS row

// MAXT bounds the workgroup size: a plane of up to 640 threads (10 waves)
// runs one workgroup per CU at 3 waves per SIMD, which leaves up to 168
// VGPRs for the z-queue and the prefetched V_eff and Y_{k-1} vectors.
template <typename T, int MAXT>
__global__ __launch_bounds__(MAXT) void stencil_plane_kernel(StencilArgs a) {
  extern __shared__ unsigned char smem_raw[];
  T* lds = reinterpret_cast<T*>(smem_raw);
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int pitch = nx + 2 * kPad;
  const int plane_lds = ny * pitch;
  const long pstride = (long)nx * ny;
  const int col = blockIdx.z;
  const int z0 = blockIdx.y * a.zc;
  const int z1 = min(nz, z0 + a.zc);
  const int segs = nx / 4;
  const int t = threadIdx.x;
  const bool active = t < segs * ny;
  const int y = active ? t / segs : 0;
  const int x0 = active ? 4 * (t - y * segs) : 0;
  const long off = x0 + (long)nx * y;

  const T* __restrict__ yin = reinterpret_cast<const T*>(a.yin) + (long)col * a.ld;
  const T* __restrict__ yprev =
      a.yprev ? reinterpret_cast<const T*>(a.yprev) + (long)col * a.ld : nullptr;
  T* yout = reinterpret_cast<T*>(a.yout) + (long)col * a.ld;
  const T* __restrict__ veff = reinterpret_cast<const T*>(a.veff);

  T cx[7], cy[7], cz[7];
#pragma unroll
  for (int k = 0; k < 7; ++k) { cx[k] = (T)a.cx[k]; cy[k] = (T)a.cy[k]; cz[k] = (T)a.cz[k]; }
  const T alpha = (T)a.alpha, beta = (T)a.beta, vshift = (T)a.shift;

  // row offsets of the y neighbours (periodic), k = 1..6
  int yp[7], ym[7];
#pragma unroll
  for (int k = 1; k <= 6; ++k) {
    int u = y + k; if (u >= ny) u -= ny;
    int d = y - k; if (d < 0) d += ny;
    yp[k] = u * pitch + kPad + x0;
    ym[k] = d * pitch + kPad + x0;
  }
  const int own = y * pitch + kPad + x0;
  // periodic copies: the first kPad points of a row also go right of the row,
  // the last kPad points also go left of it
  const int copy_r = (x0 < kPad) ? y * pitch + kPad + nx + x0 : -1;
  const int copy_l = (x0 >= nx - kPad) ? y * pitch + x0 - (nx - kPad) : -1;

  Vec4<T> q[13];
  const Vec4<T> zero4 = {{(T)0, (T)0, (T)0, (T)0}};
#pragma unroll
  for (int d = 0; d < 12; ++d) {
    int zz = z0 - 6 + d;
    zz = ((zz % nz) + nz) % nz;
    q[d] = active ? ld4(yin + zz * pstride + off) : zero4;
  }
  int zn = z0 + 6; if (zn >= nz) zn -= nz;
  Vec4<T> nxt = active ? ld4(yin + zn * pstride + off) : zero4;
  // with registers to spare (MAXT <= 640), V_eff and Y_{k-1} of the next
  // plane are loaded one plane ahead
  constexpr bool PRE = MAXT <= 640;
  Vec4<T> vv_n = zero4, pv_n = zero4;
  if constexpr (PRE) {
    if (active && z0 < z1) {
      vv_n = ld4(veff + (long)z0 * pstride + off);
      if (yprev) pv_n = ld4(yprev + (long)z0 * pstride + off);
    }
  }
  int buf = 0;
  for (int z = z0; z < z1; ++z) {
    q[12] = nxt;
    Vec4<T> vv = vv_n, pv = pv_n;
    int zl = z + 7; if (zl >= nz) zl -= nz;
    if (z + 1 < z1 && active) {
      nxt = ld4(yin + zl * pstride + off);
      if constexpr (PRE) {
        const long gn = (long)(z + 1) * pstride + off;
        vv_n = ld4(veff + gn);
        if (yprev) pv_n = ld4(yprev + gn);
      }
    }
    const long g = (long)z * pstride + off;
    if constexpr (!PRE) {
      if (active) {
        vv = ld4(veff + g);
        if (yprev) pv = ld4(yprev + g);
      }
    }
    T* P = lds + buf * plane_lds;
    if (active) {
      st4(P + own, q[6]);
      if (copy_r >= 0) st4(P + copy_r, q[6]);
      if (copy_l >= 0) st4(P + copy_l, q[6]);
    }
    __syncthreads();
    if (active) {
      // x window: x0-8 .. x0+11
      T w[20];
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const Vec4<T> r = ld4(P + own - kPad + 4 * s);
        w[4 * s] = r.v[0]; w[4 * s + 1] = r.v[1]; w[4 * s + 2] = r.v[2]; w[4 * s + 3] = r.v[3];
      }
      T acc[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[i] = 0;
#pragma unroll
        for (int k = 1; k <= 6; ++k) acc[i] += cx[k] * pair_d2(w[8 + i + k], w[8 + i - k], q[6].v[i]);
      }
#pragma unroll
      for (int k = 1; k <= 6; ++k) {
        const Vec4<T> up = ld4(P + yp[k]);
        const Vec4<T> dn = ld4(P + ym[k]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i] += cy[k] * pair_d2(up.v[i], dn.v[i], q[6].v[i]) +
                    cz[k] * pair_d2(q[6 + k].v[i], q[6 - k].v[i], q[6].v[i]);
      }
      Vec4<T> out;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        out.v[i] = alpha * (acc[i] + (vv.v[i] - vshift) * q[6].v[i]) +
                   (yprev ? beta * pv.v[i] : (T)0);
      st4(yout + g, out);
    }
    buf ^= 1;
#pragma unroll
    for (int d = 0; d < 12; ++d) q[d] = q[d + 1];
  }
}

// FP32 whole-plane variant with the x halo taken by DPP row rotations, for
// nx = 16 P with P = 3, 6 <= ny <= 48 and nz >= 7.  Thread t owns the P
// consecutive points x0 = P (t % 16) .. x0 + P - 1 of row y = t / 16, so the
// 16 lanes of a DPP row hold one whole x-row of the plane: the x neighbours
// x0 - 6 .. x0 + P + 5 are the values of the lanes ceil(6/P) to either side,
// fetched by row_ror (periodic in x by construction: the rotation wraps within
// the row), and only the y neighbours go through LDS (rows of nx floats with 6
// periodic copies of rows above and below the plane).  The 13-plane z-queue of
// P values per thread lives in registers; the load of the plane entering it is
// issued one step ahead; V_eff and Y_{k-1} are loaded after the barrier.  At
// 12 waves per plane and at most 80 VGPRs two plane workgroups share a CU.
template <int D>
__device__ __forceinline__ float row_lane(float v) {
  // value of lane (r + D) mod 16 of this lane's row: row_ror:n moves lane
  // (r - n) mod 16 to lane r
  constexpr int n = ((-D) % 16 + 16) % 16;
  static_assert(n != 0, "a neighbour lane");
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 | n, 0xF, 0xF,
                                                    false));
}

// w[m] = value at x0 - 6 + m for the points of lane offset D (m in range)
template <int P, int D>
__device__ __forceinline__ void window_from_lane(const float (&own)[P], float (&w)[P + 12]) {
#pragma unroll
  for (int j = 0; j < P; ++j) {
    constexpr int base = 6 + D * P;
    const int m = base + j;
    if (m >= 0 && m < P + 12) w[m] = row_lane<D>(own[j]);
  }
}

template <int P, int D>
__device__ __forceinline__ void window_lane_dispatch(const float (&own)[P], float (&w)[P + 12]) {
  if constexpr (D != 0) window_from_lane<P, D>(own, w);
}

template <int P, int... I>
__device__ __forceinline__ void x_window_all(const float (&own)[P], float (&w)[P + 12],
                                             std::integer_sequence<int, I...>) {
  constexpr int L = (6 + P - 1) / P;
  (window_lane_dispatch<P, I - L>(own, w), ...);
}

__global__ __launch_bounds__(768) __attribute__((amdgpu_waves_per_eu(6)))
void stencil_dpp_kernel(StencilArgs a) {
  constexpr int P = 3;
  extern __shared__ unsigned char smem_raw[];
  float* lds = reinterpret_cast<float*>(smem_raw);
  const int nx = a.nx, ny = a.ny, nz = a.nz;  // nx = 16 P, blockDim = 16 ny
  const int plane_lds = (ny + 12) * nx;
  const int pstride = nx * ny;
  const int col = blockIdx.z;
  const int z0 = blockIdx.y * a.zc;
  const int z1 = min(nz, z0 + a.zc);
  const int t = threadIdx.x;
  const int y = t >> 4;
  const int x0 = P * (t & 15);
  const int off = x0 + nx * y;

  const float* __restrict__ yin = reinterpret_cast<const float*>(a.yin) + (long)col * a.ld;
  const float* __restrict__ yprev =
      a.yprev ? reinterpret_cast<const float*>(a.yprev) + (long)col * a.ld : nullptr;
  float* yout = reinterpret_cast<float*>(a.yout) + (long)col * a.ld;
  const float* __restrict__ veff = reinterpret_cast<const float*>(a.veff);
  const float* cx = a.fcx;
  const float* cy = a.fcy;
  const float* cz = a.fcz;
  const float alpha = a.falpha, beta = a.fbeta, vshift = a.fshift;

  // LDS row y + 6 holds plane row y; rows 0..5 and ny+6..ny+11 are periodic copies
  const int own = (y + 6) * nx + x0;
  const int copy_dn = (y < 6) ? own + ny * nx : -1;
  const int copy_up = (y >= ny - 6) ? own - ny * nx : -1;

  float q[13][P];
#pragma unroll
  for (int d = 0; d < 12; ++d) {
    int zz = z0 - 6 + d;
    zz = ((zz % nz) + nz) % nz;
#pragma unroll
    for (int j = 0; j < P; ++j) q[d][j] = yin[zz * pstride + off + j];
  }
  float nxt[P];
  {
    int zn = z0 + 6; if (zn >= nz) zn -= nz;
#pragma unroll
    for (int j = 0; j < P; ++j) nxt[j] = yin[zn * pstride + off + j];
  }
  int buf = 0;
  for (int z = z0; z < z1; ++z) {
#pragma unroll
    for (int j = 0; j < P; ++j) q[12][j] = nxt[j];
    int zl = z + 7; if (zl >= nz) zl -= nz;  // nz >= 7: one wrap
    if (z + 1 < z1) {
#pragma unroll
      for (int j = 0; j < P; ++j) nxt[j] = yin[zl * pstride + off + j];
    }
    const int g = z * pstride + off;
    float* B = lds + buf * plane_lds;
#pragma unroll
    for (int j = 0; j < P; ++j) {
      B[own + j] = q[6][j];
      if (copy_dn >= 0) B[copy_dn + j] = q[6][j];
      if (copy_up >= 0) B[copy_up + j] = q[6][j];
    }
    // x window from the row's lanes (every lane of the workgroup is active)
    float w[P + 12];
#pragma unroll
    for (int j = 0; j < P; ++j) w[6 + j] = q[6][j];
    x_window_all<P>(q[6], w, std::make_integer_sequence<int, 2 * ((6 + P - 1) / P) + 1>{});
    __syncthreads();
    float vv[P], pv[P];
#pragma unroll
    for (int j = 0; j < P; ++j) {
      vv[j] = veff[g + j];
      pv[j] = yprev ? yprev[g + j] : 0.f;
    }
    float acc[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
      acc[i] = 0.f;
#pragma unroll
      for (int k = 1; k <= 6; ++k) acc[i] += cx[k] * pair_d2(w[6 + i + k], w[6 + i - k], q[6][i]);
    }
#pragma unroll
    for (int k = 1; k <= 6; ++k) {
      const float* up = B + own + k * nx;
      const float* dn = B + own - k * nx;
#pragma unroll
      for (int i = 0; i < P; ++i)
        acc[i] += cy[k] * pair_d2(up[i], dn[i], q[6][i]) +
                  cz[k] * pair_d2(q[6 + k][i], q[6 - k][i], q[6][i]);
    }
#pragma unroll
    for (int i = 0; i < P; ++i)
      yout[g + i] = alpha * (acc[i] + (vv[i] - vshift) * q[6][i]) + (yprev ? beta * pv[i] : 0.f);
    buf ^= 1;
#pragma unroll
    for (int d = 0; d < 12; ++d)
#pragma unroll
      for (int j = 0; j < P; ++j) q[d][j] = q[d + 1][j];
  }
}

// W consecutive points moved as one 16-byte vector (float x 4, double x 2).
template <typename T, int W>
struct VecW { T v[W]; };

template <typename T, int W>
__device__ __forceinline__ VecW<T, W> ldw(const T* p) {
  static_assert(sizeof(T) * W == 16 || sizeof(T) * W == 8, "one 8- or 16-byte vector");
  VecW<T, W> r;
  if constexpr (sizeof(T) == 4 && W == 2) {
    const float2 f = *reinterpret_cast<const float2*>(p);
    r.v[0] = f.x; r.v[1] = f.y;
  } else if constexpr (sizeof(T) == 4) {
    const float4 f = *reinterpret_cast<const float4*>(p);
    r.v[0] = f.x; r.v[1] = f.y; r.v[2] = f.z; r.v[3] = f.w;
  } else {
    const double2 d = *reinterpret_cast<const double2*>(p);
    r.v[0] = d.x; r.v[1] = d.y;
  }
  return r;
}

template <typename T, int W>
__device__ __forceinline__ void stw(T* p, const VecW<T, W>& r) {
  if constexpr (sizeof(T) == 4 && W == 2)
    *reinterpret_cast<float2*>(p) = make_float2(r.v[0], r.v[1]);
  else if constexpr (sizeof(T) == 4)
    *reinterpret_cast<float4*>(p) = make_float4(r.v[0], r.v[1], r.v[2], r.v[3]);
  else
    *reinterpret_cast<double2*>(p) = make_double2(r.v[0], r.v[1]);
}

// Slab variant for planes too large for one workgroup (nx % W == 0): a
// workgroup owns one column, a slab of TY rows and a chunk of z-planes.  As
// in the whole-plane kernel each thread keeps the z-queue of its W points
// in registers; the centre plane of the slab goes to LDS together with 6
// periodic halo rows above and below, which are read from memory for every
// plane (12 / TY extra reads of the input block, mostly served by L2 since
// the neighbouring slabs read them as their own rows).
// With MAXT <= 768 (3 waves per SIMD, up to 168 VGPRs) V_eff, Y_{k-1} and the
// thread's halo vector (when the 12 halo rows need at most one vector per
// thread) are loaded one plane ahead.
template <typename T, int W, int MAXT>
__global__ __launch_bounds__(MAXT) void stencil_slab_kernel(StencilArgs a) {
  extern __shared__ unsigned char smem_raw[];
  T* lds = reinterpret_cast<T*>(smem_raw);
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int TY = a.ty_tile;
  const int pitch = nx + 2 * kPad;
  const int rows = TY + 12;
  const int plane_lds = rows * pitch;
  const long pstride = (long)nx * ny;
  const int col = blockIdx.z;
  const int y0 = blockIdx.x * TY;
  const int ty = min(TY, ny - y0);
  const int z0 = blockIdx.y * a.zc;
  const int z1 = min(nz, z0 + a.zc);
  const int segs = nx / W;
  const int t = threadIdx.x;
  const bool active = t < segs * ty;
  const int ly = active ? t / segs : 0;       // local row
  const int x0 = active ? W * (t - ly * segs) : 0;
  const long off = x0 + (long)nx * (y0 + ly);

  const T* __restrict__ yin = reinterpret_cast<const T*>(a.yin) + (long)col * a.ld;
  const T* __restrict__ yprev =
      a.yprev ? reinterpret_cast<const T*>(a.yprev) + (long)col * a.ld : nullptr;
  T* yout = reinterpret_cast<T*>(a.yout) + (long)col * a.ld;
  const T* __restrict__ veff = reinterpret_cast<const T*>(a.veff);

  T cx[7], cy[7], cz[7];
#pragma unroll
  for (int k = 0; k < 7; ++k) { cx[k] = (T)a.cx[k]; cy[k] = (T)a.cy[k]; cz[k] = (T)a.cz[k]; }
  const T alpha = (T)a.alpha, beta = (T)a.beta, vshift = (T)a.shift;

  const int own = (ly + 6) * pitch + kPad + x0;
  const int copy_r = (x0 < kPad) ? (ly + 6) * pitch + kPad + nx + x0 : -1;
  const int copy_l = (x0 >= nx - kPad) ? (ly + 6) * pitch + x0 - (nx - kPad) : -1;
  // halo work items: 12 rows x segs segments, spread over the workgroup
  const int halo_items = 12 * segs;

  VecW<T, W> q[13];
  VecW<T, W> zero4;
#pragma unroll
  for (int i = 0; i < W; ++i) zero4.v[i] = (T)0;
#pragma unroll
  for (int d = 0; d < 12; ++d) {
    int zz = z0 - 6 + d;
    zz = ((zz % nz) + nz) % nz;
    q[d] = active ? ldw<T, W>(yin + zz * pstride + off) : zero4;
  }
  int zn = z0 + 6; if (zn >= nz) zn -= nz;
  VecW<T, W> nxt = active ? ldw<T, W>(yin + zn * pstride + off) : zero4;
  constexpr bool PRE = MAXT <= 768;
  // the thread's halo item: row hr of the 12 halo rows, segment h_x0
  const bool one_halo = PRE && halo_items <= (int)blockDim.x;
  const bool has_halo = one_halo && t < halo_items;
  int h_base = 0, h_x0 = 0;
  long h_off = 0;
  if (has_halo) {
    const int hr = t / segs;
    h_x0 = W * (t - hr * segs);
    const int lrow = hr < 6 ? hr - 6 : ty + hr - 6;   // -6..-1, ty..ty+5
    int gy = y0 + lrow;
    gy = ((gy % ny) + ny) % ny;
    h_off = (long)nx * gy + h_x0;
    h_base = (lrow + 6) * pitch;
  }
  VecW<T, W> vv_n = zero4, pv_n = zero4, hv_n = zero4;
  if constexpr (PRE) {
    if (z0 < z1) {
      if (active) {
        vv_n = ldw<T, W>(veff + (long)z0 * pstride + off);
        if (yprev) pv_n = ldw<T, W>(yprev + (long)z0 * pstride + off);
      }
      if (has_halo) hv_n = ldw<T, W>(yin + (long)z0 * pstride + h_off);
    }
  }
  int buf = 0;
  for (int z = z0; z < z1; ++z) {
    q[12] = nxt;
    VecW<T, W> vv = vv_n, pv = pv_n;
    const VecW<T, W> hv = hv_n;
    int zl = z + 7; if (zl >= nz) zl -= nz;
    if (z + 1 < z1) {
      if (active) nxt = ldw<T, W>(yin + zl * pstride + off);
      if constexpr (PRE) {
        const long gn = (long)(z + 1) * pstride + off;
        if (active) {
          vv_n = ldw<T, W>(veff + gn);
          if (yprev) pv_n = ldw<T, W>(yprev + gn);
        }
        if (has_halo) hv_n = ldw<T, W>(yin + (long)(z + 1) * pstride + h_off);
      }
    }
    const long g = (long)z * pstride + off;
    if constexpr (!PRE) {
      if (active) {
        vv = ldw<T, W>(veff + g);
        if (yprev) pv = ldw<T, W>(yprev + g);
      }
    }
    T* P = lds + buf * plane_lds;
    if (active) {
      stw<T, W>(P + own, q[6]);
      if (copy_r >= 0) stw<T, W>(P + copy_r, q[6]);
      if (copy_l >= 0) stw<T, W>(P + copy_l, q[6]);
    }
    // halo rows of this plane: local rows -6..-1 and ty..ty+5 (periodic in y)
    if (one_halo) {
      if (has_halo) {
        stw<T, W>(P + h_base + kPad + h_x0, hv);
        if (h_x0 < kPad) stw<T, W>(P + h_base + kPad + nx + h_x0, hv);
        if (h_x0 >= nx - kPad) stw<T, W>(P + h_base + h_x0 - (nx - kPad), hv);
      }
    } else {
      for (int e = t; e < halo_items; e += blockDim.x) {
        const int hr = e / segs, hx0 = W * (e - hr * segs);
        const int lrow = hr < 6 ? hr - 6 : ty + hr - 6;
        int gy = y0 + lrow;
        gy = ((gy % ny) + ny) % ny;
        const VecW<T, W> hl = ldw<T, W>(yin + (long)z * pstride + (long)nx * gy + hx0);
        const int base = (lrow + 6) * pitch;
        stw<T, W>(P + base + kPad + hx0, hl);
        if (hx0 < kPad) stw<T, W>(P + base + kPad + nx + hx0, hl);
        if (hx0 >= nx - kPad) stw<T, W>(P + base + hx0 - (nx - kPad), hl);
      }
    }
    __syncthreads();
    if (active) {
      // x window x0-6 .. x0+W+5; the thread's own W values come from
      // registers, the six on each side from LDS
      T w[W + 12];
#pragma unroll
      for (int i = 0; i < W; ++i) w[6 + i] = q[6].v[i];
      if constexpr (W == 2) {
#pragma unroll
        for (int s2 = 0; s2 < 3; ++s2) {
          const VecW<T, 2> l = ldw<T, 2>(P + own - 6 + 2 * s2);
          const VecW<T, 2> r = ldw<T, 2>(P + own + 2 + 2 * s2);
          w[2 * s2] = l.v[0]; w[2 * s2 + 1] = l.v[1];
          w[8 + 2 * s2] = r.v[0]; w[8 + 2 * s2 + 1] = r.v[1];
        }
      } else {
        const VecW<T, 2> l2 = ldw<T, 2>(P + own - 6);
        const VecW<T, 4> l4 = ldw<T, 4>(P + own - 4);
        const VecW<T, 4> r4 = ldw<T, 4>(P + own + 4);
        const VecW<T, 2> r2 = ldw<T, 2>(P + own + 8);
        w[0] = l2.v[0]; w[1] = l2.v[1];
#pragma unroll
        for (int j = 0; j < 4; ++j) { w[2 + j] = l4.v[j]; w[10 + j] = r4.v[j]; }
        w[14] = r2.v[0]; w[15] = r2.v[1];
      }
      T acc[W];
#pragma unroll
      for (int i = 0; i < W; ++i) {
        acc[i] = 0;
#pragma unroll
        for (int k = 1; k <= 6; ++k) acc[i] += cx[k] * pair_d2(w[6 + i + k], w[6 + i - k], q[6].v[i]);
      }
#pragma unroll
      for (int k = 1; k <= 6; ++k) {
        const VecW<T, W> up = ldw<T, W>(P + own + k * pitch);
        const VecW<T, W> dn = ldw<T, W>(P + own - k * pitch);
#pragma unroll
        for (int i = 0; i < W; ++i)
          acc[i] += cy[k] * pair_d2(up.v[i], dn.v[i], q[6].v[i]) +
                    cz[k] * pair_d2(q[6 + k].v[i], q[6 - k].v[i], q[6].v[i]);
      }
      VecW<T, W> out;
#pragma unroll
      for (int i = 0; i < W; ++i)
        out.v[i] = alpha * (acc[i] + (vv.v[i] - vshift) * q[6].v[i]) +
                   (yprev ? beta * pv.v[i] : (T)0);
      stw<T, W>(yout + g, out);
    }
    buf ^= 1;
#pragma unroll
    for (int d = 0; d < 12; ++d) q[d] = q[d + 1];
  }
}

// Slab kernel for rows of any length: one column of the block, a slab of TY rows and a
// chunk of z-planes per workgroup.  A thread owns W consecutive points of a row (16
// bytes), the last segment of a row only its first R = nx % W (R = 0: all W).  Loads of
// that segment start at the last W points of the row, so that nothing past the row is
// read, and are shifted into place; its LDS and memory writes are element by element.
// All vectors need element alignment only, so nx, ld and the base may be anything.
//
// The z-queue lives in registers; the centre plane goes to one of two LDS buffers, rows
// of constant pitch with six periodic copies at either end, six rows above and six below
// (WHOLE: the slab is the plane and they are its own rows; otherwise they are read from
// memory).  Every LDS read is one base and a constant offset.  Idle threads of the last
// wave repeat thread 0 and write nothing, so no load is conditional.
//
// The bound is memory (three streams), closely followed by the VALU (18 neighbour pairs a
// point, three operations each).  What the time above the floor goes to is latency: one
// barrier per plane, and no prefetch beyond it, since at more than 128 VGPRs only 12 waves
// run on a CU (V_eff and Y_{k-1} loaded above the barrier, or the queue kept two planes
// long to halve its moves, spill and lose 20 to 60 %).  Measured against the kernels taken
// before (time of one application, memory floor at 4.7 TB/s):
//   FP32 72^3 x 2048    2.78 -> 2.38 ms (1.94)    FP32 45 x 40 x 54 x 203  215 -> 109 us (50)
//   FP32 64^3 x 256      231 -> 180 us (170)      FP32 50^3 x 300          434 -> 163 us (95)
//   FP64 48^3 x 512      430 -> 405 us (287)      FP64 71 x 67 x 70 x 150  750 -> 357 us (252)
//   FP64 24^3 x 64      20.5 -> 9.8 us (4.5)      FP32 24^3 x 512           38 -> 29 us (18)
// Rows that are no multiple of four run at 0.55 of the rate of those that are: 16-byte
// loads off their alignment are split.  (A thread owning four rows at one x, all accesses
// single elements, spilled: 255 us at 45 x 40 x 54 x 203.)
// LDS pitch of a row: its length, kPad copies at either end, a multiple that leaves sixteen
// waves of narrow planes room in LDS (nx <= 32: 48, <= 80: 96, else 128)
constexpr int rows_pitch(int nx) { return nx <= 32 ? 48 : nx <= 80 ? 96 : 128; }
constexpr int kRowsMaxNx = 112;

template <typename T, int W>
__device__ __forceinline__ VecW<T, W> ldu(const T* p) {
  typedef T vec __attribute__((ext_vector_type(W), aligned(sizeof(T))));
  const vec u = *reinterpret_cast<const vec*>(p);
  VecW<T, W> r;
#pragma unroll
  for (int i = 0; i < W; ++i) r.v[i] = u[i];
  return r;
}

template <typename T, int W>
__device__ __forceinline__ void stu(T* p, const VecW<T, W>& r) {
  typedef T vec __attribute__((ext_vector_type(W), aligned(sizeof(T))));
  vec u;
#pragma unroll
  for (int i = 0; i < W; ++i) u[i] = r.v[i];
  *reinterpret_cast<vec*>(p) = u;
}

template <typename T, int W, int R, bool WHOLE, int PITCH>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4)))
void stencil_rows_kernel(StencilArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  T* lds = reinterpret_cast<T*>(smem_raw);
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int y0 = WHOLE ? 0 : blockIdx.x * a.ty_tile;
  const int ty = WHOLE ? ny : min(a.ty_tile, ny - y0);
  const int plane_lds = (a.ty_tile + 12) * PITCH;
  const int pstride = nx * ny;
  const int col = blockIdx.z;
  const int z0 = blockIdx.y * a.zc;
  const int z1 = min(nz, z0 + a.zc);
  const int segs = (nx + W - 1) / W;
  const int t = threadIdx.x;
  const bool active = t < segs * ty;
  const int ly = active ? t / segs : 0;
  const int x0 = active ? W * (t - ly * segs) : 0;
  const bool last = R != 0 && x0 + W > nx;
  const int off = x0 + nx * (y0 + ly);
  // byte offsets within a plane: of the segment, and of where its vector loads start
  const unsigned ooff = off * (unsigned)sizeof(T);
  const unsigned loff = (last ? off - (W - R) : off) * (unsigned)sizeof(T);

  const T* __restrict__ yin = reinterpret_cast<const T*>(a.yin) + (long)col * a.ld;
  const T* __restrict__ yprev =
      a.yprev ? reinterpret_cast<const T*>(a.yprev) + (long)col * a.ld : nullptr;
  T* yout = reinterpret_cast<T*>(a.yout) + (long)col * a.ld;
  const T* __restrict__ veff = reinterpret_cast<const T*>(a.veff);
  auto cx = [&](int k) -> T { if constexpr (sizeof(T) == 4) return a.fcx[k]; else return a.cx[k]; };
  auto cy = [&](int k) -> T { if constexpr (sizeof(T) == 4) return a.fcy[k]; else return a.cy[k]; };
  auto cz = [&](int k) -> T { if constexpr (sizeof(T) == 4) return a.fcz[k]; else return a.cz[k]; };
  const T alpha = (T)a.alpha, beta = (T)a.beta, vshift = (T)a.shift;

  auto load = [&](const T* base, int z, unsigned o, bool shifted) {
    VecW<T, W> v = ldu<T, W>(
        reinterpret_cast<const T*>(reinterpret_cast<const char*>(base + (long)z * pstride) + o));
    if constexpr (R != 0) {
#pragma unroll
      for (int i = 0; i < R; ++i) v.v[i] = shifted ? v.v[i + W - R] : v.v[i];
    }
    return v;
  };
  // a segment starting at x of the LDS row at `row`: itself and, at the ends of the row,
  // its periodic copies
  auto put = [&](T* row, int x, bool part, const VecW<T, W>& v, bool copies) {
    T* o = row + kPad + x;
    if (!part) stw<T, W>(o, v);
    if constexpr (R != 0) {
      if (part)
#pragma unroll
        for (int i = 0; i < R; ++i) o[i] = v.v[i];
    }
    if (!copies) return;
    if (x < kPad) {
      if constexpr (R == 0) stw<T, W>(o + nx, v);
      else
#pragma unroll
        for (int i = 0; i < W; ++i) o[nx + i] = v.v[i];
    }
    if (x + W > nx - kFdRadius) {
      if constexpr (R == 0) stw<T, W>(o - nx, v);
      else
#pragma unroll
        for (int i = 0; i < W; ++i)
          if (x + i < nx && x + i >= nx - kPad) o[i - nx] = v.v[i];
    }
  };

  // halo rows from memory, one segment per thread (slabs have at least 12 rows): row
  // h_row of the slab, segment at h_x
  const int halo_items = 12 * segs;
  int h_row = 0, h_x = 0;
  unsigned h_off = 0;
  bool h_part = false;
  if constexpr (!WHOLE) {
    const int e = min(t, halo_items - 1), hr = e / segs;
    h_x = W * (e - hr * segs);
    h_part = R != 0 && h_x + W > nx;
    h_row = hr < 6 ? hr - 6 : ty + hr - 6;
    int gy = y0 + h_row;
    if (gy < 0) gy += ny;
    if (gy >= ny) gy -= ny;
    h_off = (unsigned)sizeof(T) * (nx * gy + (h_part ? nx - W : h_x));
  }

  const int base = ly * PITCH + x0;
  VecW<T, W> q[13];
#pragma unroll
  for (int d = 0; d < 12; ++d) {
    int zz = z0 - 6 + d;
    if (zz < 0) zz += nz;
    if (zz >= nz) zz -= nz;
    q[d] = load(yin, zz, loff, last);
  }
  VecW<T, W> hv;
  if constexpr (!WHOLE) hv = load(yin, z0, h_off, h_part);
  int buf = 0;
  for (int z = z0; z < z1; ++z) {
    int zl = z + 6;
    if (zl >= nz) zl -= nz;
    q[12] = load(yin, zl, loff, last);
    T* P = lds + buf * plane_lds;
    if (active) {
      put(P + (ly + 6) * PITCH, x0, last, q[6], true);
      if constexpr (WHOLE) {
        if (ly < 6) put(P + (ly + 6 + ny) * PITCH, x0, last, q[6], false);
        if (ly >= ny - 6) put(P + (ly + 6 - ny) * PITCH, x0, last, q[6], false);
      }
    }
    if constexpr (!WHOLE) {
      if (t < halo_items) put(P + (h_row + 6) * PITCH, h_x, h_part, hv, false);
    }
    __syncthreads();
    const T* B = P + base;
    T acc[W];
#pragma unroll
    for (int i = 0; i < W; ++i) acc[i] = (T)0;
    {
      // x neighbours x0 - 6 .. x0 + W + 5, the own W from registers
      const T* X = B + 6 * PITCH + kPad;
      T w[W + 12];
#pragma unroll
      for (int i = 0; i < W; ++i) w[6 + i] = q[6].v[i];
      if constexpr (W == 2) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const VecW<T, 2> l = ldw<T, 2>(X - 6 + 2 * s);
          const VecW<T, 2> r = ldw<T, 2>(X + 2 + 2 * s);
          w[2 * s] = l.v[0]; w[2 * s + 1] = l.v[1];
          w[8 + 2 * s] = r.v[0]; w[9 + 2 * s] = r.v[1];
        }
      } else {
        const VecW<T, 2> l2 = ldw<T, 2>(X - 6), r2 = ldw<T, 2>(X + 8);
        const VecW<T, 4> l4 = ldw<T, 4>(X - 4), r4 = ldw<T, 4>(X + 4);
        w[0] = l2.v[0]; w[1] = l2.v[1];
#pragma unroll
        for (int j = 0; j < 4; ++j) { w[2 + j] = l4.v[j]; w[10 + j] = r4.v[j]; }
        w[14] = r2.v[0]; w[15] = r2.v[1];
      }
      // in the row's last segment the points right of the row's end are its periodic
      // copies, not the (meaningless) rest of the own vector
      if constexpr (R != 0) {
        if (last) {
#pragma unroll
          for (int i = R; i < W; ++i) w[6 + i] = X[i];
        }
      }
#pragma unroll
      for (int i = 0; i < W; ++i)
#pragma unroll
        for (int k = 1; k <= kFdRadius; ++k)
          acc[i] += cx(k) * pair_d2(w[6 + i + k], w[6 + i - k], q[6].v[i]);
    }
    // (kept below the x part: loaded above it they cost registers that the occupancy needs)
    __builtin_amdgcn_sched_barrier(0);
    const VecW<T, W> vv = load(veff, z, loff, last);
    VecW<T, W> pv;
    if (yprev) {
      pv = load(yprev, z, loff, last);
    } else {
#pragma unroll
      for (int i = 0; i < W; ++i) pv.v[i] = (T)0;
    }
#pragma unroll
    for (int k = 1; k <= kFdRadius; ++k) {
      const VecW<T, W> up = ldw<T, W>(B + (6 + k) * PITCH + kPad);
      const VecW<T, W> dn = ldw<T, W>(B + (6 - k) * PITCH + kPad);
#pragma unroll
      for (int i = 0; i < W; ++i)
        acc[i] += cy(k) * pair_d2(up.v[i], dn.v[i], q[6].v[i]) +
                  cz(k) * pair_d2(q[6 + k].v[i], q[6 - k].v[i], q[6].v[i]);
    }
    VecW<T, W> out;
#pragma unroll
    for (int i = 0; i < W; ++i)
      out.v[i] = alpha * (acc[i] + (vv.v[i] - vshift) * q[6].v[i]) +
                 (yprev ? beta * pv.v[i] : (T)0);
    T* o = reinterpret_cast<T*>(reinterpret_cast<char*>(yout + (long)z * pstride) + ooff);
    if (active && !last) stu<T, W>(o, out);
    if constexpr (R != 0) {
      if (last)
#pragma unroll
        for (int i = 0; i < R; ++i) o[i] = out.v[i];
    }
    if constexpr (!WHOLE) {
      const int zh = min(z + 1, nz - 1);
      hv = load(yin, zh, h_off, h_part);
    }
    buf ^= 1;
#pragma unroll
    for (int d = 0; d < 12; ++d) q[d] = q[d + 1];
  }
}

static void fill_coeffs(const dk_ctx* c, StencilArgs& a) {
  // twelfth-order central second-derivative weights (closed form of the
  // order-12 Lagrange stencil): w_0 = -5369/1800, w_k = 2(-1)^{k+1}(6!)^2/(k^2(6-k)!(6+k)!)
  static const double w[7] = {-5369.0 / 1800.0, 12.0 / 7.0, -15.0 / 56.0, 10.0 / 189.0,
                              -1.0 / 112.0, 2.0 / 1925.0, -1.0 / 16632.0};
  const double ix = 1.0 / (c->hx * c->hx), iy = 1.0 / (c->hy * c->hy), iz = 1.0 / (c->hz * c->hz);
  for (int k = 0; k < 7; ++k) {
    a.cx[k] = -0.5 * w[k] * ix;
    a.cy[k] = -0.5 * w[k] * iy;
    a.cz[k] = -0.5 * w[k] * iz;
  }
  for (int k = 0; k < 7; ++k) {
    a.fcx[k] = (float)a.cx[k];
    a.fcy[k] = (float)a.cy[k];
    a.fcz[k] = (float)a.cz[k];
  }
  a.falpha = (float)a.alpha;
  a.fbeta = (float)a.beta;
  a.fshift = (float)a.shift;
}

// How the rows kernel cuts a block: slabs of equal height (of at least 12 rows, so that a
// thread has one halo segment) and z-chunks.  At most 16 waves run on a CU (104 to 125
// VGPRs), fewer where LDS or the size of a workgroup allows fewer.  The model of a cut:
// a workgroup costs its waves (partly: its points) x (planes + prologue), more for halo
// rows; m of them on a CU cost m (1 + share / m) of one, the share being what a lone
// workgroup loses at its barriers, more while wave slots are idle; and rounds of them
// follow each other, the last one partly filled.  The weights are fitted to the times of
// all cuts of 31 shapes in FP32 and 10 in FP64 (16^3 x 40 to 72^3 x 1024): the chosen
// cut is within 2 % of the best on average, 9 % at most.
struct RowsWeights { double waves, prologue, halo, whole, share, idle, tail; };
constexpr RowsWeights kRows32 = {0.37, 1.5, 0.12, 0.1, 0.75, 0.15, 0.33};
constexpr RowsWeights kRows64 = {0.6, 2.3, 0.2, 0.08, 0.0, 0.85, 0.2};
static size_t rows_lds_bytes(int nx, int ty, size_t elem) {
  return 2 * (size_t)(ty + 12) * rows_pitch(nx) * elem;
}

static RowsPlan plan_rows(int nx, int ny, int nz, int n_s, int W) {
  const RowsWeights& w = W == 4 ? kRows32 : kRows64;
  RowsPlan best;
  double least = 0.0;
  const int segs = ceil_div(nx, W);
  for (int slabs = 1; slabs <= ny; ++slabs) {
    const int ty = ceil_div(ny, slabs);
    if (slabs > 1 && ty < 12) break;
    if (ceil_div(ny, ty) != slabs) continue;
    const int threads = (ty * segs + 63) / 64 * 64;
    if (threads > 1024) continue;
    const size_t lds = rows_lds_bytes(nx, ty, 16 / W);
    if (lds > 160 * 1024) continue;
    const int waves = threads / 64;
    const int conc = std::max(1, std::min(16 / waves, (int)(160 * 1024 / lds)));
    for (int chunks = 1, zc = nz; chunks <= std::max(1, nz / 4);
         chunks = zc > 1 ? ceil_div(nz, zc - 1) : nz + 1, zc = ceil_div(nz, chunks)) {
      const double per = (w.waves * waves + (1.0 - w.waves) * ty * segs / 64.0) *
                         (zc + w.prologue) * (1.0 + (slabs == 1 ? w.whole : w.halo * 12 / ty));
      const double n = (double)slabs * chunks * n_s / 256;  // workgroups per CU
      auto round = [&](double m) {
        return (1.0 + w.idle * std::max(0.0, 1.0 - m * waves / 16)) * (m + w.share) * per;
      };
      const double full = std::floor(n / conc), rest = n - full * conc;
      double t = full * round(conc);
      if (rest > 1e-9) {
        const double part = round(std::ceil(rest));
        t += full > 0.0 ? w.tail * round(conc) * rest / conc + (1.0 - w.tail) * part : part;
      }
      if (best.slabs == 0 || t < least) {
        least = t;
        best = {slabs, ty, zc, chunks, threads};
      }
    }
  }
  return best;
}

template <typename T, int W, int R>
static hipError_t launch_rows(dk_ctx* c, StencilArgs a, const RowsPlan& p, int n_s) {
  a.ty_tile = p.ty;
  a.zc = p.zc;
  const size_t smem = rows_lds_bytes(a.nx, p.ty, sizeof(T));
  auto launch = [&](auto kernel) -> hipError_t {
    if (smem > 64 * 1024) {
      const hipError_t e = allow_lds(c, (const void*)kernel, 160 * 1024);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(p.slabs, p.chunks, n_s), dim3(p.threads), smem, c->stream, a);
    return hipGetLastError();
  };
  const int pitch = rows_pitch(a.nx);
  if (p.slabs == 1)
    return pitch == 48   ? launch(stencil_rows_kernel<T, W, R, true, 48>)
           : pitch == 96 ? launch(stencil_rows_kernel<T, W, R, true, 96>)
                         : launch(stencil_rows_kernel<T, W, R, true, 128>);
  return pitch == 48   ? launch(stencil_rows_kernel<T, W, R, false, 48>)
         : pitch == 96 ? launch(stencil_rows_kernel<T, W, R, false, 96>)
                       : launch(stencil_rows_kernel<T, W, R, false, 128>);
}

template <typename T, int PPT>
static hipError_t launch_stencil(StencilArgs a, int n_s, int n_ytiles, int n_zch, hipStream_t st) {
  size_t smem = (size_t)(a.ty_tile + 12) * a.nx * sizeof(T);
  dim3 grid(n_ytiles, n_zch, n_s);
  hipLaunchKernelGGL((stencil_kernel<T, PPT>), grid, dim3(256), smem, st, a);
  return hipGetLastError();
}

hipError_t stencil_step(dk_ctx* c, const void* yin, const void* yprev, void* yout, long ld,
                        int n_s, double alpha, double beta, double shift) {
  if (n_s <= 0) return hipSuccess;
  StencilArgs a{};
  a.yin = yin;
  a.yprev = (beta != 0.0) ? yprev : nullptr;
  a.yout = yout;
  a.ld = ld;
  a.nx = c->nx; a.ny = c->ny; a.nz = c->nz;
  a.alpha = alpha; a.beta = beta; a.shift = shift;
  fill_coeffs(c, a);
  // points per thread: enough rows for at least one full plane row per thread group
  int ppt = (int)((long)c->nx * c->ny + 255) / 256;
  if (ppt > 4) ppt = 4;
  if (ppt < 1) ppt = 1;
  int ty = (256 * ppt) / c->nx;
  if (ty > c->ny) ty = c->ny;
  if (ty < 1) return hipErrorInvalidValue;  // nx > 1024 is not supported
  a.ty_tile = ty;
  const int n_ytiles = ceil_div(c->ny, ty);
  int n_zch = ceil_div(2048, (long)n_ytiles * n_s);
  const int max_zch = c->nz / 12 > 0 ? c->nz / 12 : 1;
  if (n_zch > max_zch) n_zch = max_zch;
  if (n_zch < 1) n_zch = 1;
  a.zc = ceil_div(c->nz, n_zch);
  n_zch = ceil_div(c->nz, a.zc);
  const bool f64 = c->precision == DK_PREC_FP64;
  a.veff = f64 ? (const void*)c->veff64 : (const void*)c->veff32;
  KTimer kt(c, DK_K_STENCIL);
  const long plane = (long)c->nx * c->ny;
  // nx = 48 in FP32: one x-row per DPP row of 16 lanes, a whole plane per workgroup, two
  // workgroups per CU.  Where such workgroups fill the chip (to 95 %) it is ahead of the rows
  // kernel (H X without projectors, 48^3 x 512: 158 against 169 us, 48 x 24 x 48 x 512: 102
  // against 128; 24 filter steps over 128 projectors at 48^3 x 512: 7.97 against 8.12 ms),
  // elsewhere behind (48 x 40 x 54 x 203: 71 against 63 us)
  if (!f64 && c->nx == 48 && c->ny >= 6 && c->ny <= 48 && ld % 4 == 0) {
    int zch = ceil_div(512, (long)n_s);
    zch = std::max(1, std::min(zch, c->nz / 12));
    const int zc = ceil_div(c->nz, zch);
    zch = ceil_div(c->nz, zc);
    const long wgs = (long)n_s * zch, rounds = (wgs + 511) / 512;
    if (wgs >= 0.95 * 512 * rounds) {
      a.zc = zc;
      const size_t smem = 2 * (size_t)(c->ny + 12) * c->nx * sizeof(float);
      hipLaunchKernelGGL(stencil_dpp_kernel, dim3(1, zch, n_s), dim3(16 * c->ny), smem, c->stream,
                         a);
      return hipGetLastError();
    }
  }
  // Rows kernel up to 112 points a row.  Above 80, FP32 planes that need several of its
  // workgroups and that the slab kernel takes stay there: it loads the halo rows a plane
  // ahead (96^3 x 512: 1592 against 1829 us; 112 x 64 x 64 x 200: 388 and 384 us).  Planes
  // of one workgroup, rows off the vectors and FP64 gain (96 x 40 x 40 x 300: 188 -> 146 us;
  // 90^3 x 200: 1863 -> 783 us; 81 x 40 x 50 x 300: 662 -> 344 us; FP64 96^3 x 128: 890 ->
  // 687 us, 99 x 50 x 40 x 100: 302 -> 175 us; times of one application)
  // Of rows of at most ten points its vectors waste much where the length is no multiple of
  // them; in blocks large enough to hide latency one point a thread is faster, if the tiles
  // of that form are well filled (9 x 100 x 100 x 300: FP32 226 against 169 us, FP64 268
  // against 226; 7 x 100 x 100 x 300: 174 against 112 and 231 against 190).
  const int W = f64 ? 2 : 4;
  const bool short_rows = c->nx <= 10 && c->nx % W != 0 && c->ngrid * n_s >= 4000000 &&
                          plane >= 0.6 * n_ytiles * 256 * ppt;
  if (c->nx <= kRowsMaxNx && !short_rows) {
    // (the search over all cuts takes 1 us at 48^3 and 36 us at 7 x 1024 x 1024)
    if (c->rows_n_s != n_s) {
      c->rows_plan = plan_rows(c->nx, c->ny, c->nz, n_s, W);
      c->rows_n_s = n_s;
    }
    const RowsPlan p = c->rows_plan;
    const bool slab = !f64 && c->nx > 80 && p.slabs > 1 && c->nx % 4 == 0 && ld % 4 == 0;
    if (p.slabs > 0 && !slab) {
      const int R = c->nx % W;
      if (f64)
        return R == 0 ? launch_rows<double, 2, 0>(c, a, p, n_s)
                      : launch_rows<double, 2, 1>(c, a, p, n_s);
      switch (R) {
        case 0: return launch_rows<float, 4, 0>(c, a, p, n_s);
        case 1: return launch_rows<float, 4, 1>(c, a, p, n_s);
        case 2: return launch_rows<float, 4, 2>(c, a, p, n_s);
        default: return launch_rows<float, 4, 3>(c, a, p, n_s);
      }
    }
  }
  // longer rows: a whole FP32 plane of up to 4096 points in one workgroup (the FP64 queue
  // of 4-wide vectors costs ~180 VGPRs and ran slower than the row-tile kernel)
  if (!f64 && c->nx % 4 == 0 && plane <= 4096 && ld % 4 == 0) {
    // whole-plane workgroups: one per column and z-chunk
    const int threads = ((int)(plane / 4) + 63) / 64 * 64;
    // z-chunks only when there are too few columns to fill the GPU: every
    // chunk re-reads 12 planes
    int zch = ceil_div(512, (long)n_s);
    const int maxz = c->nz / 12 > 0 ? c->nz / 12 : 1;
    if (zch > maxz) zch = maxz;
    if (zch < 1) zch = 1;
    a.zc = ceil_div(c->nz, zch);
    zch = ceil_div(c->nz, a.zc);
    const size_t smem = 2 * (size_t)c->ny * (c->nx + 2 * kPad) * sizeof(float);
    dim3 grid(1, zch, n_s);
    if (smem <= 160 * 1024) {
      for (const void* f : {(const void*)stencil_plane_kernel<float, 640>,
                            (const void*)stencil_plane_kernel<float, 1024>}) {
        const hipError_t e = allow_lds(c, f, 160 * 1024);
        if (e != hipSuccess) return e;
      }
      if (threads <= 640)
        hipLaunchKernelGGL((stencil_plane_kernel<float, 640>), grid, dim3(threads), smem, c->stream, a);
      else
        hipLaunchKernelGGL((stencil_plane_kernel<float, 1024>), grid, dim3(threads), smem, c->stream, a);
      return hipGetLastError();
    }
  }
  // longer rows, slab kernel: FP32 planes larger than one workgroup (4-point vectors),
  // and FP64 planes (2-point vectors: the FP64 whole-plane form needs too many registers)
  {
    const int W = f64 ? 2 : 4;
    if (c->nx % W == 0 && (ld % W) == 0 && (f64 || plane > 4096) && c->nx <= W * 1024 / 7 &&
        c->ny >= 12) {
      const int segs = c->nx / W;
      // slabs of equal height with at most 1024 threads each
      const int max_ty = 1024 / segs;
      const int n_slabs = ceil_div(c->ny, max_ty);
      const int ty = ceil_div(c->ny, n_slabs);
      a.ty_tile = ty;
      const int threads = ((ty * segs) + 63) / 64 * 64;
      int zch = ceil_div(512, (long)n_slabs * n_s);
      const int maxz = c->nz / 12 > 0 ? c->nz / 12 : 1;
      if (zch > maxz) zch = maxz;
      if (zch < 1) zch = 1;
      a.zc = ceil_div(c->nz, zch);
      zch = ceil_div(c->nz, a.zc);
      const size_t smem = 2 * (size_t)(ty + 12) * (c->nx + 2 * kPad) * (f64 ? 8 : 4);
      if (smem <= 160 * 1024) {
        for (const void* f : {(const void*)stencil_slab_kernel<double, 2, 768>,
                              (const void*)stencil_slab_kernel<double, 2, 1024>,
                              (const void*)stencil_slab_kernel<float, 4, 768>,
                              (const void*)stencil_slab_kernel<float, 4, 1024>}) {
          const hipError_t e = allow_lds(c, f, 160 * 1024);
          if (e != hipSuccess) return e;
        }
        dim3 grid(n_slabs, zch, n_s);
        const bool small = threads <= 768;
        if (f64) {
          if (small)
            hipLaunchKernelGGL((stencil_slab_kernel<double, 2, 768>), grid, dim3(threads), smem, c->stream, a);
          else
            hipLaunchKernelGGL((stencil_slab_kernel<double, 2, 1024>), grid, dim3(threads), smem, c->stream, a);
        } else {
          if (small)
            hipLaunchKernelGGL((stencil_slab_kernel<float, 4, 768>), grid, dim3(threads), smem, c->stream, a);
          else
            hipLaunchKernelGGL((stencil_slab_kernel<float, 4, 1024>), grid, dim3(threads), smem, c->stream, a);
        }
        return hipGetLastError();
      }
    }
  }
  switch (ppt) {
    case 1: return f64 ? launch_stencil<double, 1>(a, n_s, n_ytiles, n_zch, c->stream)
                       : launch_stencil<float, 1>(a, n_s, n_ytiles, n_zch, c->stream);
    case 2: return f64 ? launch_stencil<double, 2>(a, n_s, n_ytiles, n_zch, c->stream)
                       : launch_stencil<float, 2>(a, n_s, n_ytiles, n_zch, c->stream);
    case 3: return f64 ? launch_stencil<double, 3>(a, n_s, n_ytiles, n_zch, c->stream)
                       : launch_stencil<float, 3>(a, n_s, n_ytiles, n_zch, c->stream);
    default: return f64 ? launch_stencil<double, 4>(a, n_s, n_ytiles, n_zch, c->stream)
                        : launch_stencil<float, 4>(a, n_s, n_ytiles, n_zch, c->stream);
  }
}

// grad_h of every projector table along x, y and z (twelfth-order central
// first difference a_k = (-1)^{k+1}(6!)^2/(k(6-k)!(6+k)!)), used by the
// nonlocal force in the transposed form <chi, grad_h f> = -<grad_h chi, f>.
template <typename T>
__global__ void fd_gradient_kernel(const T* __restrict__ chi, T* __restrict__ dchi, long ngrid,
                                   int n_proj, int nx, int ny, int nz, double ihx, double ihy,
                                   double ihz) {
  const double a[7] = {0.0, 6.0 / 7.0, -15.0 / 56.0, 5.0 / 63.0, -1.0 / 56.0, 1.0 / 385.0,
                       -1.0 / 5544.0};
  const long tot = ngrid * n_proj;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < tot;
       e += (long)gridDim.x * blockDim.x) {
    const int p = (int)(e / ngrid);
    const long g = e - (long)p * ngrid;
    const int x = (int)(g % nx);
    const int y = (int)((g / nx) % ny);
    const int z = (int)(g / ((long)nx * ny));
    const T* col = chi + (long)p * ngrid;
    double gx = 0, gy = 0, gz = 0;
    for (int k = 1; k <= kFdRadius; ++k) {
      int xp = (x + k) % nx, xm = (x - k + nx * 8) % nx;
      int yp = (y + k) % ny, ym = (y - k + ny * 8) % ny;
      int zp = (z + k) % nz, zm = (z - k + nz * 8) % nz;
      gx += a[k] * ((double)col[xp + (long)nx * (y + (long)ny * z)] - (double)col[xm + (long)nx * (y + (long)ny * z)]);
      gy += a[k] * ((double)col[x + (long)nx * (yp + (long)ny * z)] - (double)col[x + (long)nx * (ym + (long)ny * z)]);
      gz += a[k] * ((double)col[x + (long)nx * (y + (long)ny * zp)] - (double)col[x + (long)nx * (y + (long)ny * zm)]);
    }
    dchi[e] = (T)(gx * ihx);
    dchi[tot + e] = (T)(gy * ihy);
    dchi[2 * tot + e] = (T)(gz * ihz);
  }
}

hipError_t fd_gradient_tables(dk_ctx* c) {
  if (c->n_proj == 0) return hipSuccess;
  const long tot = c->ngrid * c->n_proj;
  int blocks = (int)((tot + 255) / 256);
  if (blocks > 65536) blocks = 65536;
  // FP64 tables in both precisions: the forces are accumulated in FP64
  hipLaunchKernelGGL(fd_gradient_kernel<double>, dim3(blocks), dim3(256), 0, c->stream,
                     c->chi64, c->dchi64, c->ngrid, c->n_proj, c->nx, c->ny, c->nz,
                     1.0 / c->hx, 1.0 / c->hy, 1.0 / c->hz);
  return hipGetLastError();
}

}  // namespace dk
