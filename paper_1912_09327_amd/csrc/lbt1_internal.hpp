// Host-side declarations shared by the runtime and the kernel table.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace lbt1 {

enum : int { KIND_GATHER = 1, KIND_STRIP = 2, KIND_BGK = 3, KIND_TILE = 4, KIND_BGK_TILE = 5, KIND_SC_TILE = 6 };

// One built step kernel.  Gather kernels take (StepArgs); strip kernels take
// (StepArgs, StripMap); tile kernels take (StepArgs, TileMap); population (BGK)
// kernels take (BgkArgs).
struct StepKernel {
  int prec, haswall, wall, kind, vec, rows;
  const void *fn;
  const char *name;
  int steps;  // time steps one launch advances (fused strip kernels: 2; tile kernels: any)
  int sc;     // multiphase (Shan-Chen force) kernel
  int threads = 256;  // tile kernels: threads of a block (vec: columns, rows: rows of its region)
  // tile kernels, measured: us of a launch, and of each block that falls to one CU, per
  // step and once
  double us_launch = 0, us_step = 0, us_block = 0;
};

// The kernels of one storage precision (lbt1_step_kernels.hip and
// lbt1_batch_step_kernels.hip, each compiled once per precision).
struct PrecKernels {
  const StepKernel *steps;
  int count;
  const void *reduce_partial, *bgk_psi, *bgk_reduce_partial;
};
struct BatchTileKernel {  // regions of vec columns by `rows` rows on `threads` threads
  int vec, rows, threads;
  const void *fn;
};
constexpr int kBatchTiles = 3;
struct BatchKernels {
  const void *step[3][3];  // [strips of 6, 14, 30 rows][1, 2, 4 columns per lane]
  const void *fused[4];    // strips of 2, 6, 14, 30 rows
  const void *lds[2];      // strips of 6, 14 rows
  BatchTileKernel tile[kBatchTiles];
  const void *reduce;
};
template <int P> const PrecKernels &prec_kernels();
template <int P> const BatchKernels &batch_kernels();
template <int P> const StepKernel *tile_kernels(int *count);
template <> const StepKernel *tile_kernels<0>(int *count);
template <> const StepKernel *tile_kernels<1>(int *count);
template <> const StepKernel *tile_kernels<2>(int *count);
template <> const StepKernel *tile_kernels<3>(int *count);
template <> const PrecKernels &prec_kernels<0>();
template <> const PrecKernels &prec_kernels<1>();
template <> const PrecKernels &prec_kernels<2>();
template <> const PrecKernels &prec_kernels<3>();
template <> const BatchKernels &batch_kernels<0>();
template <> const BatchKernels &batch_kernels<1>();
template <> const BatchKernels &batch_kernels<2>();
template <> const BatchKernels &batch_kernels<3>();

const StepKernel *step_kernels(int *count);
const void *reduce_partial_kernel(int prec);
const void *reduce_final_kernel();
const void *reduce_final_out_kernel();  // final pass writing the user-facing slots
const void *bgk_reduce_partial_kernel(int prec);
const void *bgk_psi_kernel(int prec);
const void *batch_step_kernel(int prec, int vec_class, int rows);
const void *batch_fused_kernel(int prec, int rows);  // two steps per launch, two columns per lane
const void *batch_lds_kernel(int prec, int rows);    // grids resident in LDS for a burst
const BatchTileKernel *batch_tile_kernel(int prec, int i);  // regions held in registers; NULL past the last
const void *batch_reduce_kernel(int prec);
const void *batch_classify_kernel(int vec);          // strip kinds of a work list, once per list
const void *batch_reduce_final_kernel();

}  // namespace lbt1
