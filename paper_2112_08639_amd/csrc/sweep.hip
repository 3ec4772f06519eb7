// Kleinman-Bylander nonlocal operator over the atoms' compact supports (Eq.
// nonlocaloperator), as two passes over a block of grid vectors:
//   integrals  C = alpha gamma h^3 chi^T X   (N_proj x N_s)
//   scatter    Y += chi C
// Both run on MFMA over compact tables: blocks of 64 consecutive points, and in each the
// four-projector groups with a nonzero value there.
//
// Precision.  Mixed: the scatter is FP32 MFMA with the sum over projectors kept apart
// from Y and added once; the integrals are split-BF16 with FP32 accumulation over at
// most 64 blocks (three pieces, six products: FP32 level; two pieces, three products in
// the filter steps over more than kFullProj projectors).  FP64: FP64 MFMA throughout.
#include <algorithm>
#include <vector>

#include "ctx.h"
#include "gemm.h"
#include "sweep_kernels.h"

namespace dk {

namespace {

// FP32 accumulation.  Runs take at most 64 blocks of 64 points.  Each block's products are
// summed apart and added to the run's sum once (otherwise a sum that grows with the run is
// rounded 12 times per block: the error of H X over 128 projectors at 110592 x 2048, runs of
// 54 blocks, is 4.8e-7 of its rms where the nonlocal term dominates, against 1.8e-7).  Two
// pieces are off by 4e-6 there, and sums apart cost registers that their widest kernel does
// not have (2.70 against 2.79 ms for 8 filter steps at 110592 x 512): they sum straight on
// where runs are short, at most kPlainBlocks in equal shares and kMaxChunkBlocks over
// compact supports.
constexpr int kMaxRunBlocks = 64;
constexpr int kPlainBlocks = 14;
constexpr int kMaxChunkBlocks = 32;
// Up to this many projectors the filter steps take FP32-level products as well: two pieces
// are off by 2^-18 of each product (H X where the nonlocal term dominates: 4e-6 of its rms,
// three pieces 1e-7), and so few projectors are a small part of a step (16 atoms, 55296 x
// 512, 8 steps: 1.26 ms with two pieces, 1.38 with three, 1.60 on FP32 MFMA).
constexpr int kFullProj = 64;

// ------------------------------------------------------------- the tables --

// one workgroup per block, one wave per live group: entry e = eoff[block] + position in
// the block's list
template <bool MIXED>
__global__ __launch_bounds__(256) void sweep_table_kernel(
    const double* __restrict__ chi, long ngrid, int n_proj, int n_groups,
    const int* __restrict__ perm, const int* __restrict__ klist, const int* __restrict__ kcount,
    const int* __restrict__ eoff, float* __restrict__ stab, void* __restrict__ gtab) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, r16 = lane & 15;
  const long gb = blockIdx.x;
  const int cnt = kcount[gb];
  const long e0 = eoff[gb];
  for (int i = wave; i < cnt; i += 4) {
    const long e = e0 + i;
    const int grp = perm[klist[gb * n_groups + i]];
    auto val = [&](int p, int pt) -> double {
      const long x = gb * 64 + pt;
      const int proj = 4 * grp + p;
      return (x < ngrid && proj < n_proj) ? chi[(long)proj * ngrid + x] : 0.0;
    };
    if constexpr (MIXED) {
      // scatter operand: projector 3 - g, points 4 r16 ..
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
        stab[e * kScatFloats + lane * 4 + mb] = (float)val(3 - g, 4 * r16 + mb);
      // integral operand: projector r16 / 4, g = r16 % 4, the lane's g selecting ks and the
      // half of v
      __bf16* o = reinterpret_cast<__bf16*>(gtab) + e * kPieceElems;
      const int p = r16 >> 2, gg = r16 & 3, ks = g >> 1, v0 = 4 * (g & 1);
#pragma unroll
      for (int v = v0; v < v0 + 4; ++v) {
        __bf16 h, m, l;
        split3_bf16((float)val(p, 32 * ks + 8 * gg + v), h, m, l);
        o[piece_at(e, 0, ks, p, gg, v)] = h;
        o[piece_at(e, 1, ks, p, gg, v)] = m;
        o[piece_at(e, 2, ks, p, gg, v)] = l;
      }
    } else {
      double* o = reinterpret_cast<double*>(gtab) + e * kF64Elems;
      const int p = r16 >> 2, gg = r16 & 3;  // mb = g
#pragma unroll
      for (int r = 0; r < 4; ++r) o[f64_at(e, g, p, gg, r)] = val(p, f64_point(g, gg, r));
    }
  }
}

// --------------------------------------------------------------- integrals --
//
// A workgroup takes a run of blocks and 16 CB CW columns.  Up to 64 groups the runs are
// equal shares of the blocks with one slot per group, in FP64 beyond 32 groups two runs of
// half the groups each per share; beyond 64, runs of consecutive blocks whose live groups
// form a union of at most 64 (mixed) or 32 (FP64) slots.  (Unions for 33 to 64 groups in
// FP64 end after a few blocks where most groups are live: H X over 64 atoms at 32768 x 512
// 742 us, shares 451, the dense product before both 560; 48 atoms at 165888 x 1024 2615,
// 2475 and 4195; over 64 atoms at 221184 x 512, which read the block twice for little, 1537,
// 1575 and 2733.  And they make the workspace follow the atoms.)  Each of the CW
// consumer waves holds 16 CB columns of the current block in registers and accumulates the
// union's rows in registers; at the end of the run they go out as one partial row per
// projector, and a small kernel sums the runs.
//
// A block's table entries pass through LDS, in two buffers, one barrier per block.  Four
// further waves of the workgroup only move them, several stages ahead in registers: a
// wave's memory operations complete in order, so a consumer that loaded them would wait
// for its tile of the next block as well (373248 x 2048, 432 projectors, two pieces: 1.60
// against 1.16 ms).  Measured: 60 us at 110592 x 512 over 128 projectors (3.8 TB/s), before 80
// over the dense table; 1.11 against 1.72 ms at 373248 x 2048; FP64 186 against 342 us
// at 110592 x 512.  In the mixed kernel the feeding waves run at the highest priority
// (64.6 -> 62.8 us and, over 432 projectors, 1.23 -> 1.17 ms); in FP64, where they share
// SIMDs whose matrix pipes are full, at the same as the others (higher: 186 -> 208 us).

constexpr int kFeedWaves = 4;
constexpr int kFeedDepth = 2;

// UNITS 16-byte units of each entry's SRC_UNITS are taken.  Loads are unconditional (the
// entry clamped), so that the waits count exactly.
template <int UNITS, int SRC_UNITS>
struct SweepFeed {
  static constexpr int T = 64 * kFeedWaves;
  static constexpr int N = UNITS * kStageEntries / T;
  static_assert(UNITS * kStageEntries % T == 0, "whole rounds of the feeding waves");
  const f32x4* tab;
  StageCursor cur;
  int tid;
  int fetched = 0;
  f32x4 v[kFeedDepth][N];

  __device__ __forceinline__ void fetch(int d) {
    const f32x4* const src = tab + (long)(cur.valid() ? cur.first_entry() : 0) * SRC_UNITS;
    const int last = cur.valid() ? cur.entries() - 1 : 0;
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const unsigned i = tid + T * r;
      v[d][r] = src[min((int)(i / UNITS), last) * SRC_UNITS + (int)(i % UNITS)];
    }
    if (cur.valid()) {
      cur.next();
      ++fetched;
    }
  }
  __device__ __forceinline__ void put(int d, f32x4* buf) const {
#pragma unroll
    for (int r = 0; r < N; ++r) buf[tid + T * r] = v[d][r];
  }
  // All stages of the run: stage k in buffer k % 2 from barrier k on.  The barriers are
  // rounded up to whole rounds of kFeedDepth (the consumers do the same): a condition
  // inside the round would make every wait one for all loads in flight.
  __device__ __forceinline__ void run(f32x4* ring) {
#pragma unroll
    for (int d = 0; d < kFeedDepth; ++d) fetch(d);
    for (int k = 0; cur.valid() || k < fetched + 1; k += kFeedDepth) {
#pragma unroll
      for (int d = 0; d < kFeedDepth; ++d) {
        put(d, ring + ((k + d) & 1) * (UNITS * kStageEntries));
        fetch(d);
        __syncthreads();  // barrier k + d
      }
    }
  }
};

// bf16 per column of a staged tile: 64 points and 8 more, so that the 16 columns of a
// fragment start at different banks
constexpr int kTilePitch = 72;

// 16-byte units taken of an entry
constexpr int piece_units(int NP) { return 32 * NP; }
constexpr int kF64Units = kF64Elems / 2;

// RB: 16-projector row blocks of the run's union (4 slots each), CB: 16-column blocks per
// wave, CW consumer waves, NP bf16 pieces; APART: each block's sum apart from the run's.
template <int RB, int CB, int CW, int NP, bool APART>
__global__ __launch_bounds__(64 * (CW + kFeedWaves), (CW + kFeedWaves) / 4)
void integrals_mixed_kernel(SweepArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char sweep_lds[];
  constexpr int BUF = piece_units(NP) * kStageEntries;
  f32x4* const ring = reinterpret_cast<f32x4*>(sweep_lds);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c16 = lane & 15;
  const unsigned slot_bit = 1u << (c16 >> 2), slot_below = slot_bit - 1;
  // the column tiles of a run run one after another on one XCD and share its table
  // entries in that XCD's L2
  const long w = xcd_work_item(blockIdx.x, (long)gridDim.x);
  const SweepRun run(a, (int)(w / a.ntiles));
  if (wave >= CW) {
    __builtin_amdgcn_s_setprio(3);  // few instructions, and the others wait for them
    SweepFeed<piece_units(NP), 96> feed{(const f32x4*)a.tab, StageCursor(run),
                                        (int)threadIdx.x - 64 * CW};
    feed.run(ring);
    return;
  }
  const int n0 = ((int)(w % a.ntiles) * CW + wave) * 16 * CB;
  const bool active = n0 < a.n_s;
  // The tile is read along the columns (16 lanes x 16 bytes each) and turned into the MFMA
  // operand through the wave's own slice of LDS: [column block][piece][column][point].
  __bf16* const xs = reinterpret_cast<__bf16*>(ring + 2 * BUF) + wave * (CB * NP * 16 * kTilePitch);
  const float* xp[CB][4];  // columns 16 cb + 4 i + g (past the last column: the last)
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      xp[cb][i] =
          (const float*)a.x + (long)min(n0 + 16 * cb + 4 * i + g, a.n_s - 1) * a.ld + 4 * c16;
  f32x4 x[CB][4];
  const int full_blocks = (int)(a.ngrid / 64) - run.b0;  // blocks of the run before a ragged one
  auto load_x = [&](int t) {
    const long base = (long)(run.b0 + t) * 64;
    if (t < full_blocks) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          x[cb][i] = *reinterpret_cast<const f32x4_u*>(xp[cb][i] + base);
    } else {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            x[cb][i][r] = (base + 4 * c16 + r < a.ngrid) ? xp[cb][i][base + r] : 0.f;
    }
  };
  // the first block with a live slot from t on (run.nb: none), and its row
  unsigned long long live = 0;
  int e0 = 0;
  auto next_live = [&](int t) {
    for (; t < run.nb; ++t) {
      live = run.rows[t].live;
      e0 = run.rows[t].entry0;
      if (live != 0) break;
    }
    return t;
  };
  int t = next_live(0);
  if (active && t < run.nb) load_x(t);
  f32x4 acc[RB][CB];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[b][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // an all-zero entry, for the dead slots of a row block
  constexpr int ZERO = 2 * BUF + CW * CB * NP * 16 * kTilePitch / 8;  // in units of 16 bytes
  if (wave == 0)
    for (int i = lane; i < piece_units(NP); i += 64) ring[ZERO + i] = f32x4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();  // barrier 0: the first stage's entries
  int buf = 0, barriers = 1;
  auto next_stage = [&]() {
    buf ^= 1;
    ++barriers;
    __syncthreads();
  };
  while (t < run.nb) {
    bf16x8 xb[NP][2][CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        bf16x4 pc[NP];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          __bf16 p0, p1, p2;
          if constexpr (NP == 3) {
            split3_bf16(x[cb][i][r], p0, p1, p2);
            pc[NP - 1][r] = p2;
          } else {
            split_bf16(x[cb][i][r], p0, p1);
          }
          pc[0][r] = p0;
          pc[1][r] = p1;
        }
#pragma unroll
        for (int p = 0; p < NP; ++p)
          *reinterpret_cast<bf16x4*>(xs + ((cb * NP + p) * 16 + 4 * i + g) * kTilePitch + 4 * c16) =
              pc[p];
      }
    }
    // other lanes of the wave read them: ordered here, and against the next tile by the
    // barriers of the stages
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
          xb[p][ks][cb] = *reinterpret_cast<const bf16x8*>(
              xs + ((cb * NP + p) * 16 + c16) * kTilePitch + 32 * ks + 8 * g);
    const unsigned long long now = live;
    const int entry0 = e0;
    // the next block's tile, in flight while this one is multiplied
    t = next_live(t + 1);
    if (active && t < run.nb) load_x(t);
    const bool split = RB * 4 > kStageEntries && split_stage(now);
    const int lower = split ? (int)__popcll(now & 0xffffffffull) : 0;
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      if (4 * b == kStageEntries && split) next_stage();
      // this lane's table row: slot 4 b + c16 / 4, if live the at-th entry of the block
      const unsigned nib = (unsigned)(now >> (4 * b)) & 15u;
      if (nib == 0 || !active) continue;
      const int at = (int)__popcll(now & ((1ull << (4 * b)) - 1)) + (int)__popc(nib & slot_below);
      const int first = 4 * b >= kStageEntries ? lower : 0;
      const int row = (nib & slot_bit) ? buf * BUF + (at - first) * piece_units(NP) : ZERO;
      const __bf16* tp = reinterpret_cast<const __bf16*>(ring + row) +
                         piece_at(entry0 + at, 0, 0, c16 & 3, g, 0);
      bf16x8 tv[NP][2];
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
          tv[p][ks] = *reinterpret_cast<const bf16x8*>(tp + 256 * p + 128 * ks);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        // smallest products first
        f32x4 v = APART ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[b][cb];
        if constexpr (NP == 3) {
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            v = mfma_bf16(tv[NP - 1][ks], xb[0][ks][cb], v);
            v = mfma_bf16(tv[1][ks], xb[1][ks][cb], v);
            v = mfma_bf16(tv[0][ks], xb[NP - 1][ks][cb], v);
          }
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          v = mfma_bf16(tv[1][ks], xb[0][ks][cb], v);
          v = mfma_bf16(tv[0][ks], xb[1][ks][cb], v);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) v = mfma_bf16(tv[0][ks], xb[0][ks][cb], v);
        acc[b][cb] = APART ? acc[b][cb] + v : v;
      }
    }
    next_stage();
  }
  for (; barriers % kFeedDepth != 0; ++barriers) __syncthreads();
  if (!active) return;
  float* __restrict__ part = (float*)a.part + (long)4 * run.uoff * a.n_s;
  const int rows = 4 * run.ulen;
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 16 * b + 4 * g + i;
        const int col = n0 + 16 * cb + c16;
        if (r < rows && col < a.n_s) part[(long)r * a.n_s + col] = acc[b][cb][i];
      }
}

// FP64, one 16-column block per wave, one product of four projectors at a time: the four
// 4x4x4 blocks of the MFMA are four columns each, with the same projectors.  Only live
// slots are multiplied, where 16x16x4 works on four slots as soon as one is live (6.4 of 8
// row blocks at 48^3 over 32 groups, of which 16 are live); both forms run at the same
// rate (65 and 66 TFLOP/s from registers).  110592 x 512: 254 -> 186 us, 373248 x 512 over
// 432 projectors 1.10 -> 0.91 ms, 64000 x 300: 139 -> 120 us.  What bounds it now is the LDS
// path as much as the products (156 us with multiply-adds in their place): a lane needs
// all 16 points of its projector and k for every 16 columns.  Lane (g, column c16):
// SLOTS accumulators, acc[s] projector g of slot s.
template <int SLOTS, int CW>
__global__ __launch_bounds__(64 * (CW + kFeedWaves), (CW + kFeedWaves) / 4)
void integrals_f64_kernel(SweepArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char sweep_lds[];
  constexpr int BUF = kF64Units * kStageEntries;
  static_assert(SLOTS <= kStageEntries && SLOTS <= 32, "one stage per block");
  f32x4* const ring = reinterpret_cast<f32x4*>(sweep_lds);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c16 = lane & 15;
  const long w = xcd_work_item(blockIdx.x, (long)gridDim.x);
  const SweepRun run(a, (int)(w / a.ntiles));
  if (wave >= CW) {
    SweepFeed<kF64Units, kF64Units> feed{(const f32x4*)a.tab, StageCursor(run),
                                         (int)threadIdx.x - 64 * CW};
    feed.run(ring);
    return;
  }
  const int n0 = ((int)(w % a.ntiles) * CW + wave) * 16;
  const bool active = n0 < a.n_s;
  const int col = min(n0 + c16, a.n_s - 1);
  const double* const xp = (const double*)a.x + (long)col * a.ld + 2 * g;
  double x[4][4];
  const int full_blocks = (int)(a.ngrid / 64) - run.b0;
  auto load_x = [&](int t) {
    const long base = (long)(run.b0 + t) * 64;
    if (t < full_blocks) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f64x2_u v = *reinterpret_cast<const f64x2_u*>(xp + base + 16 * mb + 8 * h);
          x[mb][2 * h] = v[0];
          x[mb][2 * h + 1] = v[1];
        }
    } else {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const long o = base + f64_point(mb, 0, r);
          x[mb][r] = (o + 2 * g < a.ngrid) ? xp[o] : 0.0;
        }
    }
  };
  auto next_live = [&](int t) {
    while (t < run.nb && run.rows[t].live == 0) ++t;
    return t;
  };
  const int first = next_live(0);
  if (active && first < run.nb) load_x(first);
  double acc[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) acc[s] = 0.0;
  __syncthreads();
  int buf = 0, barriers = 1;
  for (int t = first; t < run.nb;) {
    const unsigned live = (unsigned)run.rows[t].live;
    const long e0 = run.rows[t].entry0;
    double z[4][4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) z[mb][r] = x[mb][r];
    const int tn = next_live(t + 1);
    if (active && tn < run.nb) load_x(tn);
    if (active) {
      const double* const tab = reinterpret_cast<const double*>(ring + buf * BUF);
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        if (((live >> s) & 1u) == 0) continue;
        const int at = (int)__popc(live & ((1u << s) - 1));
        const double* const tp = tab + min(at, kStageEntries - 1) * kF64Elems +
                                 f64_at(e0 + at, 0, c16 & 3, g, 0);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
          f64x2_t tv[2];
#pragma unroll
          for (int h = 0; h < 2; ++h)
            tv[h] = *reinterpret_cast<const f64x2_t*>(tp + 64 * mb + 32 * h);
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[s] = mfma_f64_4(tv[r >> 1][r & 1], z[mb][r], acc[s]);
        }
      }
    }
    buf ^= 1;
    ++barriers;
    __syncthreads();
    t = tn;
  }
  for (; barriers % kFeedDepth != 0; ++barriers) __syncthreads();
  if (!active) return;
  double* __restrict__ part = (double*)a.part + (long)4 * run.uoff * a.n_s;
#pragma unroll
  for (int s = 0; s < SLOTS; ++s)
    if (s < run.ulen) part[(long)(4 * s + g) * a.n_s + col] = acc[s];
}

// ----------------------------------------------------------------- scatter --
//
// A wave holds the table values of its points and of up to 32 live groups in registers
// (FP64: 24) and walks over the columns, 16 at a time: the coefficients of a tile come as
// one 16-byte (FP64: 32-byte) load per four groups (lane group g takes group 4 q + g, and k
// step j one projector of each), the tile of Y is read one tile ahead, the coefficients of
// the next tile replace this one's as they are used, and nothing passes through LDS.  The
// four waves of a workgroup take consecutive points of the same columns.  The grid is two
// waves per SIMD, every workgroup with an equal share of the tiles, points outermost.
// (Shares by the cost of their blocks instead of equal ones change nothing.)
//
// MFMA alone takes half of the time and memory alone two thirds (72^3 x 2048, 432
// projectors: 1.1 and 1.24 of 2.0 ms), and what the two waves of a SIMD overlap depends on
// their priorities: highest while a wave multiplies, lowest while it issues the next
// tile's loads: 122 -> 112 us at 110592 x 512 over 128 projectors, 2.02 -> 1.94 ms at
// 373248 x 2048, FP64 214 -> 206 us at 110592 x 512.  (The reverse order: 145 us, 2.96
// ms.)

// The columns are the rows of the MFMA and the points its columns, the lane's points of
// the row blocks being consecutive: the 16 lanes of a column then move 256 consecutive
// bytes per access.  (With the points as rows each 16-lane pass touched 16 columns, 16 or
// 32 bytes each: 140 against 119 us at 110592 x 512 over 128 projectors, 2.14 against
// 1.79 ms at 373248 x 2048 over 432, FP64 256 against 216 us at 110592 x 512.)

template <typename T> struct ScatterTraits;
template <> struct ScatterTraits<float> {
  static constexpr int MB = 4;  // 16-point row blocks per wave: all of a block's 64 points
  using Acc = f32x4;
  using Vec = f32x4;            // the lane's MB points
  using VecU = f32x4_u;
};
template <> struct ScatterTraits<double> {
  static constexpr int MB = 2;  // half a block
  using Acc = f64x4;
  using Vec = f64x2_t;
  using VecU = f64x2_u;
};
__device__ __forceinline__ f32x4 mfma_t(float a, float b, f32x4 c) { return mfma_f32(a, b, c); }
__device__ __forceinline__ f64x4 mfma_t(double a, double b, f64x4 c) { return mfma_f64(a, b, c); }

__device__ __forceinline__ void load4(float (&v)[4], const float* p) {
  const f32x4 u = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = u[j];
}
__device__ __forceinline__ void load4(double (&v)[4], const double* p) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const f64x2_t u = *reinterpret_cast<const f64x2_t*>(p + 2 * h);
    v[2 * h] = u[0];
    v[2 * h + 1] = u[1];
  }
}

// k step j sums over projector 3 - j (FP64: j) of four groups.  The s projectors come first
// in a group and have the largest integrals; summed last, the three steps before them round
// a small sum (H X of positive columns over 16 projectors: error 1.03e-7 against 6.2e-8 of
// its rms where the nonlocal term dominates).
//
// Tiles [t0, t1) of the columns for the 16 MB points from `base` on (row blocks mb0 .. of
// block b), live groups s0 .. s0 + n - 1 of the block, n <= 4 NQ.
template <typename T, int NQ, bool FULL>
__device__ __forceinline__ void scatter_tiles(const ScatterArgs& a, int b, int mb0, int s0, int n,
                                              int t0, int t1) {
  using Tr = ScatterTraits<T>;
  using Acc = typename Tr::Acc;
  using Vec = typename Tr::Vec;
  using VecU = typename Tr::VecU;
  constexpr int MB = Tr::MB;
  const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
  const long base = (long)b * 64 + 16 * mb0 + MB * c16;  // the lane's first point
  T av[NQ][4][MB];
  const T* cp[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = min(4 * q + g, n - 1);
    const bool on = 4 * q + g < n;
    const long e = a.eoff[b] + s0 + i;
    cp[q] = (const T*)a.coef + (long)a.klist[(long)b * a.n_groups + s0 + i] * a.n_s * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Vec u;
      if constexpr (sizeof(T) == 4) {
        u = ((const Vec*)a.tab)[e * (kScatFloats / 4) + j * 16 + c16];
      } else {
        const int p = 16 * mb0 + MB * c16;  // even: its register is 2 (p / 8 % 2)
        u = *(const Vec*)((const double*)a.tab + e * kF64Elems +
                          f64_at(e, p >> 4, j, (p >> 1) & 3, (p >> 2) & 2));
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) av[q][j][mb] = on ? u[mb] : (T)0;
    }
  }
  // register r: column 4 g + r (FP32) or g + 4 r (FP64) of a tile
  auto y_at = [&](int t, int r) -> T* {
    const int col = 16 * t + (sizeof(T) == 4 ? 4 * g + r : g + 4 * r);
    return (T*)a.y + (long)min(col, a.n_s - 1) * a.ld + base;
  };
  auto load_tile = [&](Vec (&y)[4], int t) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const T* p = y_at(t, r);
      if constexpr (FULL) {
        y[r] = *reinterpret_cast<const VecU*>(p);
      } else {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) y[r][mb] = base + mb < a.ngrid ? p[mb] : (T)0;
      }
    }
  };
  T cv[NQ][4];
  Vec ya[4], yb[4];
#pragma unroll
  for (int q = 0; q < NQ; ++q) load4(cv[q], cp[q] + (long)min(16 * t0 + c16, a.n_s - 1) * 4);
  load_tile(ya, t0);
  auto tile = [&](int t, Vec (&y)[4], Vec (&yn)[4]) {
    const int tn = min(t + 1, t1 - 1);
    __builtin_amdgcn_s_setprio(0);
    load_tile(yn, tn);
    __builtin_amdgcn_s_setprio(3);
    const long next = min(16 * tn + c16, a.n_s - 1);
    Acc s[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) s[mb] = Acc{0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) s[mb] = mfma_t(cv[q][j], av[q][j][mb], s[mb]);
      load4(cv[q], cp[q] + next * 4);
    }
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      T* p = y_at(t, r);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) y[r][mb] += s[mb][r];
      if constexpr (FULL) {
        *reinterpret_cast<VecU*>(p) = y[r];
      } else {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          if (base + mb < a.ngrid) p[mb] = y[r][mb];
      }
    }
  };
  for (int t = t0; t < t1; t += 2) {
    tile(t, ya, yb);
    if (t + 1 < t1) tile(t + 1, yb, ya);
  }
}

// MAXQ: groups of four live groups taken at once (a block with more takes several passes)
template <typename T, int MAXQ, int NQ>
__device__ __forceinline__ void scatter_dispatch(const ScatterArgs& a, int b, int mb0, int s0, int n,
                                                 int t0, int t1) {
  if constexpr (NQ > 1)
    if (n <= 4 * (NQ - 1)) {
      scatter_dispatch<T, MAXQ, NQ - 1>(a, b, mb0, s0, n, t0, t1);
      return;
    }
  scatter_tiles<T, NQ, true>(a, b, mb0, s0, n, t0, t1);
}

template <typename T, int MAXQ, int OCC>
__global__ __launch_bounds__(256, OCC) void scatter_kernel(ScatterArgs a) {
  constexpr int MB = ScatterTraits<T>::MB;
  constexpr int WB = 4 * MB / 4;  // blocks of 64 points per workgroup
  const int wave = threadIdx.x >> 6;
  const long total = (long)((a.nblocks + WB - 1) / WB) * a.ntiles;
  const long w = xcd_work_item(blockIdx.x, (long)gridDim.x);
  long i = total * w / gridDim.x;
  const long i1 = total * (w + 1) / gridDim.x;
  while (i < i1) {
    const int quad = (int)(i / a.ntiles);
    const int t0 = (int)(i - (long)quad * a.ntiles);
    const int t1 = (int)min((long)a.ntiles, t0 + (i1 - i));
    i += t1 - t0;
    const int b = __builtin_amdgcn_readfirstlane(quad * WB + wave * MB / 4);
    const int mb0 = __builtin_amdgcn_readfirstlane((wave * MB) & 3);
    if (b >= a.nblocks) continue;
    const bool full = (long)b * 64 + 16 * (mb0 + MB) <= a.ngrid;
    if ((long)b * 64 + 16 * mb0 >= a.ngrid) continue;
    const int cnt = const_ints(a.kcount)[b];
    for (int s0 = 0; s0 < cnt; s0 += 4 * MAXQ) {
      const int n = min(cnt - s0, 4 * MAXQ);
      if (full) scatter_dispatch<T, MAXQ, MAXQ>(a, b, mb0, s0, n, t0, t1);
      else scatter_tiles<T, MAXQ, false>(a, b, mb0, s0, n, t0, t1);
    }
  }
}

// --------------------------------------------------------------- reduction --

// coef[(group n_s + col) 4 + q] = scale rowscale[4 group + p] sum over the runs that hold
// the group of the partial row (4 occ + p); zero past the last projector.  q = 3 - p in
// FP32, p in FP64.  A workgroup
// takes one projector and 64 columns; its W waves sum interleaved shares of the
// occurrences, kReduceDepth loads in flight each, which is what the time goes by
// (two in flight: 12 us at 24^3 x 64 in FP64, 10 at 48^3 x 512 mixed; now 4 and 7; at 72^3 x
// 2048 mixed, 108 groups, 141, bound by the partials).  occ null: the dense runs,
// occurrence o of group g = o n_groups + g.
constexpr int kReduceDepth = 16;
template <typename PT, int W>
__global__ __launch_bounds__(64 * W) void sweep_reduce_kernel(const PT* __restrict__ part, int n_s,
                                                           int n_proj, int n_groups, int n_runs,
                                                           const int* __restrict__ occ_off,
                                                           const int* __restrict__ occ,
                                                           const int* __restrict__ perm,
                                                           double scale,
                                                           const double* __restrict__ rowscale,
                                                           PT* __restrict__ out) {
  __shared__ double sh[W][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int grp = blockIdx.x >> 2, p = blockIdx.x & 3;
  const int proj = 4 * perm[grp] + p;
  const double rs = rowscale[blockIdx.x];
  const int col = blockIdx.y * 64 + lane;
  const int o0 = occ ? occ_off[grp] : 0, o1 = occ ? occ_off[grp + 1] : n_runs;
  double acc = 0.0;
  if (col < n_s) {
    for (int o = o0 + wv; o < o1; o += W * kReduceDepth) {
      PT v[kReduceDepth];
#pragma unroll
      for (int i = 0; i < kReduceDepth; ++i) {
        const int oi = min(o + W * i, o1 - 1);
        v[i] = part[(4L * (occ ? occ[oi] : (long)oi * n_groups + grp) + p) * n_s + col];
      }
#pragma unroll
      for (int i = 0; i < kReduceDepth; ++i)
        if (o + W * i < o1) acc += (double)v[i];
    }
  }
  sh[wv][lane] = acc;
  __syncthreads();
  if (wv == 0 && col < n_s) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; w += 4)
      s += (sh[w][lane] + sh[w + 1][lane]) + (sh[w + 2][lane] + sh[w + 3][lane]);
    const int q = sizeof(PT) == 4 ? 3 - p : p;
    out[((long)grp * n_s + col) * 4 + q] = proj < n_proj ? (PT)(s * scale * rs) : (PT)0;
  }
}

// One wave per 64-point block: lane i looks at point 64 gb + i of the four
// projectors of each group; the groups where any lane sees a nonzero are
// listed in increasing order.  Clears the sums of group_centres_kernel.
__global__ __launch_bounds__(256) void group_lists_kernel(const double* __restrict__ chi, long ng,
                                                          int n_proj, long gblocks, int n_groups,
                                                          int* __restrict__ list,
                                                          int* __restrict__ count,
                                                          unsigned long long* __restrict__ sums) {
  const int lane = threadIdx.x & 63;
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < 4 * n_groups; i += 256) sums[i] = 0;
  const long nwaves = ((long)gridDim.x * blockDim.x) >> 6;
  for (long gb = (blockIdx.x * (long)blockDim.x + threadIdx.x) >> 6; gb < gblocks; gb += nwaves) {
    const long x = gb * 64 + lane;
    int cnt = 0;
    for (int gr = 0; gr < n_groups; ++gr) {
      bool nz = false;
      if (x < ng)
        for (int p = 4 * gr; p < 4 * gr + 4 && p < n_proj; ++p)
          nz = nz || chi[(long)p * ng + x] != 0.0;
      if (__any(nz)) {
        if (lane == 0) list[gb * n_groups + cnt] = gr;
        ++cnt;
      }
    }
    if (lane == 0) count[gb] = cnt;
  }
}

// Order of the groups.  The mixed integrals work on row blocks of four consecutive groups,
// all of it if one of them is live, so groups that are live in the same blocks are put next
// to each other: a block is (part of) an x-row, so they are sorted by the z of their centre
// in layers of kLayer bohr, then by y.  With atoms in the order of cubic cells 6.7 of 8 row
// blocks are live at 48^3 over 32 groups and 9.9 of 16 at 72^3 over 108; sorted, 5.3 and
// 7.5, and the integrals of 2048 columns took 1.10 instead of 1.17 ms.
// From here on a group is its place in that order, perm[place] the four projectors and
// ggamma their energies.
constexpr double kLayer = 4.0;
constexpr int kOrderMax = 1024;  // groups; beyond, the order stays as it is

// centres (circular means over the live blocks) as fixed-point sums, whose order does not
// matter: sums[4 g + {0, 1}] of cos, sin of z, {2, 3} of y.  At most kOrderMax groups; each
// workgroup sums in LDS first (every wave adding to the same few counters in memory: 118 us
// at 48^3 over 32 groups)
__global__ __launch_bounds__(256) void group_centres_kernel(const int* __restrict__ klist,
                                                            const int* __restrict__ kcount,
                                                            int nblocks, int n_groups, int nx,
                                                            int ny, int nz,
                                                            unsigned long long* __restrict__ sums) {
  __shared__ unsigned long long own[4 * kOrderMax];
  const int lane = threadIdx.x & 63;
  const int nwaves = (gridDim.x * 256) >> 6;
  for (int i = threadIdx.x; i < 4 * n_groups; i += 256) own[i] = 0;
  __syncthreads();
  for (int b = (blockIdx.x * 256 + threadIdx.x) >> 6; b < nblocks; b += nwaves) {
    const long e = min((long)b * 64 + 32, (long)nx * ny * nz - 1);
    const int y = (int)((e / nx) % ny), z = (int)(e / ((long)nx * ny));
    double v[4];
    sincospi(2.0 * z / nz, &v[1], &v[0]);
    sincospi(2.0 * y / ny, &v[3], &v[2]);
    for (int i = lane; i < kcount[b]; i += 64)
      for (int k = 0; k < 4; ++k)
        atomicAdd(own + 4 * klist[(long)b * n_groups + i] + k,
                  (unsigned long long)(long long)rint(v[k] * (1 << 20)));
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 4 * n_groups; i += 256)
    if (own[i] != 0) atomicAdd(sums + i, own[i]);
}

// the order (sort: by centre; otherwise as it is)
__device__ void group_order(const unsigned long long* __restrict__ sums, int n_groups, bool sort,
                            double ly, double lz, const double* __restrict__ gamma, int n_proj,
                            int sets, int* __restrict__ perm, int* __restrict__ rank,
                            double* __restrict__ ggamma) {
  __shared__ double layer[kOrderMax], along[kOrderMax];
  const int t = threadIdx.x;
  auto place = [&](int g, int r) {
    perm[r] = g;
    rank[g] = r;
    for (int p = 0; p < 4; ++p) ggamma[4 * r + p] = 4 * g + p < n_proj ? gamma[4 * g + p] : 0.0;
  };
  if (!sort) {
    for (int g = t; g < n_groups; g += 1024) place(g, g);
    return;
  }
  if (t < n_groups) {
    auto centre = [&](int k, double len) {
      const double turn = atan2((double)(long long)sums[4 * t + k + 1],
                                (double)(long long)sums[4 * t + k]) / (2.0 * M_PI);
      return (turn < 0.0 ? turn + 1.0 : turn) * len;
    };
    layer[t] = floor(centre(0, lz) / kLayer + 0.5);
    along[t] = centre(2, ly);
  }
  __syncthreads();
  if (t >= n_groups) return;
  int r = 0;
  for (int g = 0; g < n_groups; ++g)
    if (layer[g] != layer[t] ? layer[g] < layer[t]
                             : (along[g] != along[t] ? along[g] < along[t] : g < t))
      ++r;
  // alternately to the sets, so that their runs are live in the same blocks and take equal time
  // (48 atoms, 165888 x 512: 1330 -> 1204 us)
  place(t, (r % sets) * ((n_groups + sets - 1) / sets) + r / sets);
}

// eoff[b] = sum of kcount[0..b), eoff[nblocks] the total
__device__ void entry_offsets(const int* __restrict__ kcount, int nblocks, int* __restrict__ eoff) {
  __shared__ int sh[1024];
  __shared__ int base;
  const int t = threadIdx.x;
  if (t == 0) base = 0;
  for (int b0 = 0; b0 < nblocks; b0 += 1024) {
    const int v = (b0 + t < nblocks) ? kcount[b0 + t] : 0;
    sh[t] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int u = t >= o ? sh[t - o] : 0;
      __syncthreads();
      sh[t] += u;
      __syncthreads();
    }
    if (b0 + t < nblocks) eoff[b0 + t] = base + sh[t] - v;
    __syncthreads();
    if (t == 0) base += sh[1023];
    __syncthreads();
  }
  if (t == 0) eoff[nblocks] = base;
}

// the two jobs of one workgroup, side by side
__global__ __launch_bounds__(1024) void order_offsets_kernel(
    const unsigned long long* __restrict__ sums, int n_groups, bool sort, double ly, double lz,
    const double* __restrict__ gamma, int n_proj, int sets, int* __restrict__ perm,
    int* __restrict__ rank, double* __restrict__ ggamma, const int* __restrict__ kcount,
    int nblocks, int* __restrict__ eoff) {
  if (blockIdx.x == 0)
    group_order(sums, n_groups, sort, ly, lz, gamma, n_proj, sets, perm, rank, ggamma);
  else
    entry_offsets(kcount, nblocks, eoff);
}

// the lists in the new order, increasing; one wave per block.  rows not null: the rows of the
// equal shares, the live ones of `slots` consecutive groups per set, set after set
__global__ __launch_bounds__(64) void relabel_kernel(int* __restrict__ klist,
                                                     const int* __restrict__ kcount, int n_groups,
                                                     const int* __restrict__ rank,
                                                     const int* __restrict__ eoff, int sets,
                                                     int slots, SweepRow* __restrict__ rows) {
  __shared__ int r[kOrderMax];
  const int b = blockIdx.x, lane = threadIdx.x;
  int* const list = klist + (long)b * n_groups;
  const int cnt = kcount[b];
  for (int i = lane; i < cnt; i += 64) r[i] = rank[list[i]];
  __syncthreads();
  for (int i = lane; i < cnt; i += 64) {
    int at = 0;
    for (int j = 0; j < cnt; ++j) at += r[j] < r[i] ? 1 : 0;
    list[at] = r[i];
  }
  if (!rows) return;
  unsigned long long m = lane < cnt ? 1ull << r[lane] : 0ull;  // at most 64 groups
  for (int o = 32; o > 0; o >>= 1) m |= __shfl_xor(m, o);
  if (lane >= sets) return;
  const int first = lane * slots;
  const unsigned long long below = m & ((1ull << first) - 1);
  unsigned long long live = m >> first;
  if (sets > 1) live &= (1ull << slots) - 1;
  rows[(long)lane * gridDim.x + b] = SweepRow{live, eoff[b] + (int)__popcll(below), 0};
}

// Slots a run may have: 4 per row block of the kernels' accumulators.
int max_slots(const dk_ctx* c) { return c->precision == DK_PREC_MIXED ? 64 : 32; }

// Equal shares of the blocks for every run, with as many sets of groups as the slots take
// (FP64 beyond 32 groups: two), or chunks.
bool dense_runs(const dk_ctx* c) { return c->n_groups <= 64; }
int run_sets(const dk_ctx* c) { return ceil_div(c->n_groups, max_slots(c)); }
int set_slots(const dk_ctx* c) { return ceil_div(c->n_groups, run_sets(c)); }

// How the integrals are cut: the kernel's row blocks and column blocks per wave, and the
// runs.
constexpr int kConsumers = 8;
struct SweepPlan {
  int rb = 8, cb = 1;
  int n_runs = 0, run_len = 0, ntiles = 0;
  int sets = 1;
  long rows = 0;  // partial rows
  bool apart = false;  // two pieces: sums apart
};

SweepPlan plan_sweep(const dk_ctx* c, int n_s, bool two_piece) {
  SweepPlan p;
  const long nb = (c->ngrid + 63) / 64;
  if (c->precision == DK_PREC_MIXED) {
    if (c->n_groups > 32) p.rb = 16;
    else if (two_piece && nb * ceil_div(n_s, 256) >= 8L * 256) p.cb = 2;
  }
  p.ntiles = ceil_div(n_s, 16 * p.cb * kConsumers);
  if (!dense_runs(c)) {
    p.n_runs = c->n_gchunks;
    p.rows = 4 * c->g_rows;
    return p;
  }
  // one workgroup per CU, or as many whole rounds as keep the runs within kMaxRunBlocks
  p.sets = run_sets(c);
  long len = nb;
  for (int rounds = 1; rounds == 1 || len > kMaxRunBlocks; ++rounds) {
    const long runs = std::max(1L, 256L * rounds / (p.ntiles * p.sets));
    len = (nb + runs - 1) / runs;
  }
  p.apart = len > kPlainBlocks;
  p.run_len = (int)len;
  p.n_runs = (int)((nb + len - 1) / len);
  p.rows = 4L * c->n_groups * p.n_runs;
  return p;
}

size_t elem_bytes(const dk_ctx* c) {
  return c->precision == DK_PREC_MIXED ? sizeof(float) : sizeof(double);
}

size_t partial_bytes(const dk_ctx* c, int n_s) {
  const long rows = std::max(plan_sweep(c, n_s, false).rows, plan_sweep(c, n_s, true).rows);
  return ws_slice((size_t)rows * n_s * elem_bytes(c));
}

template <typename K>
hipError_t launch_integrals(dk_ctx* c, K kernel, const SweepArgs& a, const SweepPlan& p, int units,
                            size_t tiles) {
  if (p.n_runs == 0) return hipSuccess;
  // two buffers of table entries, and what the consumers keep
  const size_t lds = 2 * (size_t)units * kStageEntries * sizeof(f32x4) + tiles;
  if (lds > 64 * 1024) {
    const hipError_t e = allow_lds(c, (const void*)kernel, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)((long)p.n_runs * p.sets * p.ntiles)),
                     dim3(64 * (kConsumers + kFeedWaves)), lds, c->stream, a);
  return hipGetLastError();
}

template <int NP>
hipError_t integrals_mixed(dk_ctx* c, const SweepArgs& a, const SweepPlan& p) {
  const int units = piece_units(NP);
  // the consumers' tiles and the zero entry
  const size_t tiles = (size_t)kConsumers * p.cb * NP * 16 * kTilePitch * sizeof(__bf16) +
                       units * sizeof(f32x4);
  auto go = [&](auto kernel) { return launch_integrals(c, kernel, a, p, units, tiles); };
  if constexpr (NP == 3) {
    return p.rb == 16 ? go(integrals_mixed_kernel<16, 1, kConsumers, 3, true>)
                      : go(integrals_mixed_kernel<8, 1, kConsumers, 3, true>);
  } else {
    if (p.rb == 16)
      return p.apart ? go(integrals_mixed_kernel<16, 1, kConsumers, 2, true>)
                     : go(integrals_mixed_kernel<16, 1, kConsumers, 2, false>);
    if (p.cb == 2)
      return p.apart ? go(integrals_mixed_kernel<8, 2, kConsumers, 2, true>)
                     : go(integrals_mixed_kernel<8, 2, kConsumers, 2, false>);
    return p.apart ? go(integrals_mixed_kernel<8, 1, kConsumers, 2, true>)
                   : go(integrals_mixed_kernel<8, 1, kConsumers, 2, false>);
  }
}

struct SweepWs {
  void* part;
  void* coef;
  bool ok;
};
SweepWs sweep_ws(const dk_ctx* c, int n_s, void* ws) {
  WsCursor cur((char*)ws, nonlocal_ws_bytes(c, n_s));
  SweepWs s;
  s.part = cur.take<char>(partial_bytes(c, n_s));
  s.coef = cur.take<char>((size_t)4 * c->n_groups * n_s * elem_bytes(c));
  s.ok = cur.ok;
  return s;
}

}  // namespace

void free_sweep_tables(dk_ctx* c) {
  hipFree(c->klist); c->klist = nullptr;
  hipFree(c->kcount); c->kcount = nullptr;
  hipFree(c->geoff); c->geoff = nullptr;
  hipFree(c->gperm); c->gperm = nullptr;
  hipFree(c->gcentre); c->gcentre = nullptr;
  hipFree(c->ggamma); c->ggamma = nullptr;
  hipFree(c->growrec); c->growrec = nullptr;
  hipFree(c->gchunk); c->gchunk = nullptr;
  hipFree(c->gqoff); c->gqoff = nullptr;
  hipFree(c->gocc_off); c->gocc_off = nullptr;
  hipFree(c->gocc); c->gocc = nullptr;
  hipFree(c->gtab); c->gtab = nullptr;
  hipFree(c->stab); c->stab = nullptr;
  c->g_capacity = 0;
  c->n_groups = 0;
  c->n_gchunks = 0;
  c->g_rows = 0;
}

namespace {

// Compact supports: chunks, union maps and occurrences from the per-block group lists.
// Host work: one copy of the lists and a linear pass over the blocks.
hipError_t build_chunks(dk_ctx* c) {
  const int umax = max_slots(c);
  const long nb = (c->ngrid + 63) / 64;
  const int ng = c->n_groups;
  std::vector<int> kc(nb), kl((size_t)nb * ng);
  hipError_t e;
  if ((e = hipMemcpyAsync(kc.data(), c->kcount, nb * sizeof(int), hipMemcpyDeviceToHost,
                          c->stream)) != hipSuccess)
    return e;
  if ((e = hipMemcpyAsync(kl.data(), c->klist, (size_t)nb * ng * sizeof(int),
                          hipMemcpyDeviceToHost, c->stream)) != hipSuccess)
    return e;
  if ((e = hipStreamSynchronize(c->stream)) != hipSuccess) return e;
  std::vector<long> eoff(nb + 1, 0);
  for (long b = 0; b < nb; ++b) eoff[b + 1] = eoff[b] + kc[b];
  // chunks: runs of blocks whose union stays within umax groups (a block with
  // more live groups than umax is split into several single-block chunks)
  std::vector<int4> chunks;
  std::vector<int> uni;        // union groups of every chunk, chunk after chunk
  std::vector<int> slot_of(ng, -1);
  int cur_begin = 0, cur_n = 0;
  long uoff = 0;
  auto close = [&]() {
    if (cur_n == 0) return;
    const int len = (int)(uni.size() - uoff);
    std::sort(uni.begin() + uoff, uni.end());  // slots in the order of the blocks' entries
    chunks.push_back(make_int4(cur_begin, cur_n, (int)uoff, len));
    for (size_t s = uoff; s < uni.size(); ++s) slot_of[uni[s]] = -1;
    uoff = (long)uni.size();
    cur_n = 0;
  };
  for (long b = 0; b < nb; ++b) {
    const int* live = &kl[(size_t)b * ng];
    const int n = kc[b];
    if (n > umax) {
      close();
      for (int s0 = 0; s0 < n; s0 += umax) {
        cur_begin = (int)b;
        cur_n = 1;
        for (int i = s0; i < n && i < s0 + umax; ++i) {
          slot_of[live[i]] = (int)(uni.size() - uoff);
          uni.push_back(live[i]);
        }
        close();
      }
      continue;
    }
    int fresh = 0;
    for (int i = 0; i < n; ++i) fresh += slot_of[live[i]] < 0;
    if (cur_n > 0 && ((long)(uni.size() - uoff) + fresh > umax || cur_n >= kMaxChunkBlocks)) close();
    if (cur_n == 0) cur_begin = (int)b;
    for (int i = 0; i < n; ++i)
      if (slot_of[live[i]] < 0) {
        slot_of[live[i]] = (int)(uni.size() - uoff);
        uni.push_back(live[i]);
      }
    ++cur_n;
  }
  close();
  const int nch = (int)chunks.size();
  // per (chunk, block): the live slots and the entry of the first
  std::vector<int> qoff(nch + 1, 0);
  for (int k = 0; k < nch; ++k) qoff[k + 1] = qoff[k] + chunks[k].y;
  const long nq = qoff[nch];
  std::vector<SweepRow> rows(nq > 0 ? nq : 1, SweepRow{0, 0, 0});
  for (int k = 0; k < nch; ++k) {
    const int4 ch = chunks[k];
    for (int s = 0; s < ch.w; ++s) slot_of[uni[(size_t)ch.z + s]] = s;
    for (int t = 0; t < ch.y; ++t) {
      const long b = (long)ch.x + t;
      SweepRow& r = rows[qoff[k] + t];
      for (int i = kc[b] - 1; i >= 0; --i) {
        const int s = slot_of[kl[(size_t)b * ng + i]];
        if (s < 0) continue;
        r.live |= 1ull << s;
        r.entry0 = (int)(eoff[b] + i);
      }
    }
    for (int s = 0; s < ch.w; ++s) slot_of[uni[(size_t)ch.z + s]] = -1;
  }
  // occurrences of every group among the unions, in chunk order
  std::vector<int> occ_off(ng + 1, 0);
  for (size_t s = 0; s < uni.size(); ++s) ++occ_off[uni[s] + 1];
  for (int g = 0; g < ng; ++g) occ_off[g + 1] += occ_off[g];
  std::vector<int> occ(uni.size() > 0 ? uni.size() : 1), fill(occ_off.begin(), occ_off.end() - 1);
  for (size_t s = 0; s < uni.size(); ++s) occ[fill[uni[s]]++] = (int)s;
  auto up = [&](int** dst, const void* src, size_t bytes) -> hipError_t {
    hipFree(*dst);
    *dst = nullptr;
    hipError_t r = hipMalloc((void**)dst, bytes > 0 ? bytes : 16);
    if (r != hipSuccess) return r;
    if (bytes == 0) return hipSuccess;
    return hipMemcpy(*dst, src, bytes, hipMemcpyHostToDevice);
  };
  if ((e = up(&c->gchunk, chunks.data(), chunks.size() * sizeof(int4))) != hipSuccess) return e;
  if ((e = up(&c->gqoff, qoff.data(), qoff.size() * sizeof(int))) != hipSuccess) return e;
  if ((e = up((int**)&c->growrec, rows.data(), rows.size() * sizeof(SweepRow))) != hipSuccess) return e;
  if ((e = up(&c->gocc_off, occ_off.data(), occ_off.size() * sizeof(int))) != hipSuccess) return e;
  if ((e = up(&c->gocc, occ.data(), occ.size() * sizeof(int))) != hipSuccess) return e;
  c->n_gchunks = nch;
  c->g_rows = (long)uni.size();
  return hipSuccess;
}

}  // namespace

// Lists, maps and compact tables from the dense table chi64 (rebuilt for every set of
// projectors; buffers of the previous set are kept where they are large enough).
hipError_t build_sweep_tables(dk_ctx* c) {
  if (c->n_proj == 0) return hipSuccess;
  const bool mixed = c->precision == DK_PREC_MIXED;
  const long nb = (c->ngrid + 63) / 64;
  const int n_groups = (c->n_proj + 3) / 4;
  hipError_t e;
  if (!c->klist || c->n_groups != n_groups) {
    free_sweep_tables(c);
    if ((e = hipMalloc(&c->klist, (size_t)nb * n_groups * sizeof(int))) != hipSuccess) return e;
    if ((e = hipMalloc(&c->kcount, (size_t)nb * sizeof(int))) != hipSuccess) return e;
    if ((e = hipMalloc(&c->geoff, (size_t)(nb + 1) * sizeof(int))) != hipSuccess) return e;
    if ((e = hipMalloc(&c->ggamma, 4 * (size_t)n_groups * sizeof(double))) != hipSuccess) return e;
    if ((e = hipMalloc(&c->gperm, 2 * (size_t)n_groups * sizeof(int))) != hipSuccess) return e;
    if ((e = hipMalloc(&c->gcentre, 4 * (size_t)n_groups * sizeof(unsigned long long))) !=
        hipSuccess)
      return e;
    c->n_groups = n_groups;
  }
  long blocks = (nb * 64 + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(group_lists_kernel, dim3((int)blocks), dim3(256), 0, c->stream, c->chi64,
                     c->ngrid, c->n_proj, nb, n_groups, c->klist, c->kcount, c->gcentre);
  // the order matters to row blocks of four groups (mixed) and to two sets (FP64)
  const bool dense = dense_runs(c);
  const int sets = dense ? run_sets(c) : 1;
  const bool sort = n_groups <= kOrderMax && (mixed ? n_groups > 4 : sets > 1);
  int* const rank = c->gperm + n_groups;
  if (sort)
    hipLaunchKernelGGL(group_centres_kernel, dim3(64), dim3(256), 0, c->stream, c->klist,
                       c->kcount, (int)nb, n_groups, c->nx, c->ny, c->nz, c->gcentre);
  hipLaunchKernelGGL(order_offsets_kernel, dim3(2), dim3(1024), 0, c->stream, c->gcentre, n_groups,
                     sort, c->ly, c->lz, c->gamma_dev, c->n_proj, sets, c->gperm, rank, c->ggamma,
                     c->kcount, (int)nb, c->geoff);
  if (dense && !c->growrec &&
      (e = hipMalloc(&c->growrec, (size_t)sets * nb * sizeof(SweepRow))) != hipSuccess)
    return e;
  if (sort || dense)
    hipLaunchKernelGGL(relabel_kernel, dim3((unsigned)nb), dim3(64), 0, c->stream, c->klist,
                       c->kcount, n_groups, rank, c->geoff, sets, set_slots(c),
                       dense ? (SweepRow*)c->growrec : nullptr);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // Room for the entries: beyond 64 groups as many as there are, which has to be read back;
  // up to 64, a quarter of the dense table at most, for all (a wait of 15 us saved where the
  // whole call takes 100)
  long entries = nb * n_groups;
  if (!dense) {
    int live = 0;
    if ((e = hipMemcpyAsync(&live, c->geoff + nb, sizeof live, hipMemcpyDeviceToHost,
                            c->stream)) != hipSuccess)
      return e;
    if ((e = hipStreamSynchronize(c->stream)) != hipSuccess) return e;
    entries = live;
  }
  if (entries > c->g_capacity || !c->gtab) {
    hipFree(c->gtab); c->gtab = nullptr;
    hipFree(c->stab); c->stab = nullptr;
    c->g_capacity = 0;
    const size_t cap = (size_t)entries + 1;  // (never empty)
    const size_t per = mixed ? kPieceElems * sizeof(__bf16) : kF64Elems * sizeof(double);
    if ((e = hipMalloc(&c->gtab, cap * per)) != hipSuccess) return e;
    if (mixed && (e = hipMalloc(&c->stab, cap * kScatFloats * sizeof(float))) != hipSuccess) return e;
    c->g_capacity = (long)cap;
  }
  if (mixed)
    hipLaunchKernelGGL(sweep_table_kernel<true>, dim3((unsigned)nb), dim3(256), 0, c->stream,
                       c->chi64, c->ngrid, c->n_proj, n_groups, c->gperm, c->klist, c->kcount,
                       c->geoff, c->stab, c->gtab);
  else
    hipLaunchKernelGGL(sweep_table_kernel<false>, dim3((unsigned)nb), dim3(256), 0, c->stream,
                       c->chi64, c->ngrid, c->n_proj, n_groups, c->gperm, c->klist, c->kcount,
                       c->geoff, c->stab, c->gtab);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return dense ? hipSuccess : build_chunks(c);
}

// integral partials and the coefficients alpha gamma h^3 chi^T X
size_t nonlocal_ws_bytes(const dk_ctx* c, int n_s) {
  if (c->n_proj == 0) return 0;
  return partial_bytes(c, n_s) + ws_slice((size_t)4 * c->n_groups * n_s * elem_bytes(c));
}

hipError_t nonlocal_integrals(dk_ctx* c, const void* x, long ld, int n_s, double alpha, void* ws,
                              bool subspace) {
  if (c->n_proj == 0 || n_s <= 0) return hipSuccess;
  const SweepWs w = sweep_ws(c, n_s, ws);
  if (!w.ok) return hipErrorInvalidValue;
  const bool two_piece = subspace && c->n_proj > kFullProj;
  const SweepPlan p = plan_sweep(c, n_s, two_piece);
  const bool dense = dense_runs(c);
  SweepArgs a{};
  a.x = x;
  a.ld = ld;
  a.n_s = n_s;
  a.ngrid = c->ngrid;
  a.ntiles = p.ntiles;
  if (!dense) {
    a.chunks = (const int4*)c->gchunk;
    a.qoff = c->gqoff;
  }
  a.nblocks = (int)((c->ngrid + 63) / 64);
  a.run_len = p.run_len;
  a.n_groups = c->n_groups;
  a.sets = p.sets;
  a.slots = set_slots(c);
  a.rows = (const SweepRow*)c->growrec;
  a.tab = c->gtab;
  a.part = w.part;
  KTimer kt(c, DK_K_NL_GATHER);
  hipError_t e;
  if (c->precision == DK_PREC_FP64)
    e = launch_integrals(c, integrals_f64_kernel<32, kConsumers>, a, p, kF64Units, 0);
  else if (two_piece) e = integrals_mixed<2>(c, a, p);
  else e = integrals_mixed<3>(c, a, p);
  if (e != hipSuccess) return e;
  const dim3 grid(4 * c->n_groups, ceil_div(n_s, 64));
  const int* off = dense ? nullptr : c->gocc_off;
  const int* occ = dense ? nullptr : c->gocc;
  const double scale = c->dv * alpha;
  auto reduce = [&](auto kernel, auto* part, auto* out, int waves) {
    hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), 0, c->stream, part, n_s, c->n_proj,
                       c->n_groups, p.n_runs, off, occ, c->gperm, scale, c->ggamma, out);
  };
  // sixteen waves where four need more than one round of loads and the workgroups leave a
  // CU each (216 runs, 16 workgroups: 6.0 -> 4.1 us; with 512 workgroups over 128 runs the
  // second round of workgroups takes back what the round of loads gave)
  const long occurrences = dense ? p.n_runs : c->g_rows / c->n_groups;
  const bool wide = occurrences > 4 * kReduceDepth && (long)grid.x * grid.y <= 256;
  if (c->precision == DK_PREC_MIXED) {
    const float* part = (const float*)w.part;
    if (wide) reduce(sweep_reduce_kernel<float, 16>, part, (float*)w.coef, 16);
    else reduce(sweep_reduce_kernel<float, 4>, part, (float*)w.coef, 4);
  } else {
    const double* part = (const double*)w.part;
    if (wide) reduce(sweep_reduce_kernel<double, 16>, part, (double*)w.coef, 16);
    else reduce(sweep_reduce_kernel<double, 4>, part, (double*)w.coef, 4);
  }
  return hipGetLastError();
}

hipError_t nonlocal_scatter(dk_ctx* c, void* y, long ld, int n_s, void* ws) {
  if (c->n_proj == 0 || n_s <= 0) return hipSuccess;
  const SweepWs w = sweep_ws(c, n_s, ws);
  if (!w.ok) return hipErrorInvalidValue;
  const bool mixed = c->precision == DK_PREC_MIXED;
  ScatterArgs a{};
  a.y = y;
  a.ld = ld;
  a.n_s = n_s;
  a.ngrid = c->ngrid;
  a.ntiles = ceil_div(n_s, 16);
  a.nblocks = (int)((c->ngrid + 63) / 64);
  a.n_groups = c->n_groups;
  a.klist = c->klist;
  a.kcount = c->kcount;
  a.eoff = c->geoff;
  a.tab = mixed ? (const void*)c->stab : c->gtab;
  a.coef = w.coef;
  const long items = (long)ceil_div(a.nblocks, mixed ? 4 : 2) * a.ntiles;
  KTimer kt(c, DK_K_NL_SCATTER);
  auto go = [&](auto kernel, int occ) {
    const dim3 grid((unsigned)std::min(items, 256L * occ));
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, c->stream, a);
  };
  if (mixed) {
    go(scatter_kernel<float, 8, 2>, 2);
  } else {
    go(scatter_kernel<double, 6, 2>, 2);
  }
  return hipGetLastError();
}

}  // namespace dk
