// Tables and run order of the nonlocal term's kernels (sweep.hip).
#pragma once

#include "common.h"

namespace dk {

// Grid blocks of 64 consecutive points; one table entry per (block, live group), a group
// being four consecutive projectors with a nonzero value in the block.  The entries of a
// block are consecutive, in the order of its groups.
//   mixed: the scatter operand, FP32 [3 - projector][point] (1 KB), and the integral operand,
//          three bf16 pieces of 512 bytes
//   FP64:  one operand for both, 2 KB
constexpr int kScatFloats = 256;    // floats per mixed scatter entry
constexpr int kPieceElems = 768;    // bf16 per mixed integral entry
constexpr int kF64Elems = 256;      // doubles per FP64 entry

// FP64 integrals: point of a 64-point block that register r of access mb of lane
// (g, column) holds; k = g of MFMA step (mb, r).
__host__ __device__ constexpr int f64_point(int mb, int g, int r) {
  return 16 * mb + 8 * (r >> 1) + 2 * g + (r & 1);
}

// Element of an entry.  The 16-byte units of a 256-byte row are permuted by the entry's
// number, so that the four entries that a wave reads for one 16-projector row block start
// at different LDS banks.
//   mixed: piece p, projector pr, point 32 ks + 8 g + v
__host__ __device__ constexpr int piece_at(long e, int p, int ks, int pr, int g, int v) {
  return 256 * p + 128 * ks + (((g ^ (int)(e & 3)) * 4 + pr) * 8) + v;
}
//   FP64: projector pr, point f64_point(mb, g, r)
__host__ __device__ constexpr int f64_at(long e, int mb, int pr, int g, int r) {
  return 64 * mb + 32 * (r >> 1) + (((g ^ (int)(e & 3)) * 4 + pr) * 2) + (r & 1);
}

// vectors at element alignment (columns may start anywhere)
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef double f64x2_t __attribute__((ext_vector_type(2)));
typedef double f64x2_u __attribute__((ext_vector_type(2), aligned(8)));

// Read-only tables that steer a wave are read through the constant address space: uniform
// scalar loads, counted apart from its vector memory operations.  (As vector loads each
// one waited for every store and load of the wave.)
typedef const __attribute__((address_space(4))) int ConstInt;
__device__ __forceinline__ ConstInt* const_ints(const int* p) { return (ConstInt*)(uintptr_t)p; }

// One (run, block): the union slots that are live there, the table entry of the first.
struct SweepRow {
  unsigned long long live;
  int entry0;
  int pad;
};
typedef const __attribute__((address_space(4))) SweepRow ConstRow;

struct SweepArgs {
  const void* x;       // block
  long ld;
  int n_s;
  long ngrid;
  int ntiles;          // column tiles per run
  // runs of consecutive blocks: {first block, blocks, union offset, union length} and
  // the row of the first block (compact supports), or (chunks null) equal shares of run_len
  // blocks, `sets` (1 or 2) runs of `slots` consecutive groups each (the last one the rest)
  const int4* chunks;
  const int* qoff;
  int nblocks, run_len, n_groups, sets, slots;
  const SweepRow* rows;
  const void* tab;
  void* part;          // integral partials: row (4 * union offset + r), columns contiguous
};

struct SweepRun {
  int b0, nb, uoff, ulen;
  ConstRow* rows;
  __device__ __forceinline__ SweepRun(const SweepArgs& a, int run) {
    rows = (ConstRow*)(uintptr_t)a.rows;
    if (a.chunks) {
      ConstInt* ch = const_ints((const int*)(a.chunks + run));
      b0 = ch[0]; nb = ch[1]; uoff = ch[2]; ulen = ch[3];
      rows += const_ints(a.qoff)[run];
    } else {
      const int share = run >> (a.sets - 1), set = run & (a.sets - 1);
      b0 = share * a.run_len;
      nb = min(a.run_len, a.nblocks - b0);
      uoff = share * a.n_groups + set * a.slots;
      ulen = min(a.slots, a.n_groups - set * a.slots);
      rows += (long)set * a.nblocks + b0;
    }
  }
};

// The stages of a run, in order: every block with a live slot is one stage, or, with more
// than 32 live slots (of at most 64), one per half of the slots.
constexpr int kStageEntries = 32;
__device__ __forceinline__ bool split_stage(unsigned long long live) {
  return (int)__popcll(live) > kStageEntries;
}
struct StageCursor {
  ConstRow* rows;
  int nb;
  int t = -1;  // block of the run; nb: past the end
  unsigned long long live = 0;
  int entry0 = 0;
  bool upper = false;  // the second stage of a split block

  __device__ __forceinline__ StageCursor(const SweepRun& r) : rows(r.rows), nb(r.nb) { next_block(); }
  __device__ __forceinline__ bool valid() const { return t < nb; }
  __device__ __forceinline__ int lower() const { return (int)__popcll(live & 0xffffffffull); }
  __device__ __forceinline__ int first_entry() const { return entry0 + (upper ? lower() : 0); }
  __device__ __forceinline__ int entries() const {
    if (upper) return (int)__popcll(live >> 32);
    return split_stage(live) ? lower() : (int)__popcll(live);
  }
  __device__ __forceinline__ void next_block() {
    upper = false;
    do {
      ++t;
      if (t >= nb) return;
      live = rows[t].live;
    } while (live == 0);
    entry0 = rows[t].entry0;
  }
  __device__ __forceinline__ void next() {
    if (!upper && split_stage(live)) upper = true;
    else next_block();
  }
};

struct ScatterArgs {
  void* y;
  long ld;
  int n_s;
  long ngrid;
  int ntiles;          // tiles of 16 columns
  int nblocks, n_groups;
  const int* klist;    // groups of every block: klist[b * n_groups + i], i < kcount[b]
  const int* kcount;
  const int* eoff;     // entry of a block's first group
  const void* tab;
  const void* coef;    // [group][column][4 projectors, in FP32 the last first]
};

}  // namespace dk
