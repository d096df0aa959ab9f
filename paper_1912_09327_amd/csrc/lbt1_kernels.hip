// The final reduction passes, and the selectors over the kernels that
// lbt1_step_kernels.hip and lbt1_batch_step_kernels.hip instantiate per precision.
#include <vector>

#include "lbt1_batch_kernels.hpp"
#include "lbt1_internal.hpp"
#include "lbt1_step.hpp"

namespace lbt1 {

// one wavefront: lane l combines partial rows l, l + 64, ... in index order, then
// a fixed butterfly over the lanes (slot 3 is a maximum, the others sums)
__device__ __forceinline__ void reduce_rows(const double *partials, int nparts, double (&acc)[6]) {
  const int l = threadIdx.x;
#pragma unroll
  for (int q = 0; q < 6; ++q) acc[q] = 0.0;
  for (int b = l; b < nparts; b += 64) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const double x = partials[b * 6 + q];
      acc[q] = q == 3 ? __builtin_fmax(acc[q], x) : acc[q] + x;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const double o = __shfl_xor(acc[q], off);
      acc[q] = q == 3 ? __builtin_fmax(acc[q], o) : acc[q] + o;
    }
  }
}

// lane 0 writes the six raw slots (0 sum of rho - 1, 1-2 momentum, 3 residual,
// 4 non-finite count, 5 FLUID count)
__global__ void __launch_bounds__(64) k_reduce_final(const double *partials, int nparts, double *out) {
  double acc[6];
  reduce_rows(partials, nparts, acc);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < 6; ++q) out[q] = acc[q];
  }
}

// The same combination, written as lbt1_reduce reports it: slot 0 the mass
// (FLUID count + sum of rho - 1, the same FP64 addition the host makes), the
// slots of `what` (LBT1_REDUCE_* bits), and slot 5 always.
__global__ void __launch_bounds__(64) k_reduce_final_out(const double *partials, int nparts, uint32_t what,
                                                         double *out) {
  double acc[6];
  reduce_rows(partials, nparts, acc);
  if (threadIdx.x == 0) {
    if (what & 1u) out[0] = acc[5] + acc[0];
    if (what & 2u) {
      out[1] = acc[1];
      out[2] = acc[2];
    }
    if (what & 4u) out[3] = acc[3];
    if (what & 8u) out[4] = acc[4];
    out[5] = acc[5];
  }
}

// The partials of each active grid (fixed order: lane-strided, then a butterfly)
// into out[slot * 6 + q].
__global__ void __launch_bounds__(64) k_reduce_batch_final(BatchReduceArgs b) {
  const int n = *b.nactive;
  for (int k = blockIdx.x; k < n; k += gridDim.x) {
    const int slot = b.active[k];
    const int2 r = b.ranges[slot];
    // lane l: partial rows l, l + 64, ... of the grid in order, then a fixed butterfly
    const int l = threadIdx.x;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int i = l; i < r.y; i += 64) {
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        const double x = b.partials[(long)(r.x + i) * 6 + q];
        acc[q] = q == 3 ? __builtin_fmax(acc[q], x) : acc[q] + x;
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        const double o = __shfl_xor(acc[q], off);
        acc[q] = q == 3 ? __builtin_fmax(acc[q], o) : acc[q] + o;
      }
    }
    if (l == 0) {
#pragma unroll
      for (int q = 0; q < 6; ++q) b.out[slot * 6 + q] = acc[q];
    }
  }
}

static const PrecKernels *of_prec(int prec) {
  switch (prec) {
    case P_F64: return &prec_kernels<P_F64>();
    case P_F32: return &prec_kernels<P_F32>();
    case P_F16S: return &prec_kernels<P_F16S>();
    case P_BF16S: return &prec_kernels<P_BF16S>();
  }
  return nullptr;
}

const StepKernel *step_kernels(int *count) {
  static const std::vector<StepKernel> all = [] {
    std::vector<StepKernel> t;
    for (int p = P_F64; p <= P_BF16S; ++p) t.insert(t.end(), of_prec(p)->steps, of_prec(p)->steps + of_prec(p)->count);
    for (auto tiles : {tile_kernels<P_F64>, tile_kernels<P_F32>, tile_kernels<P_F16S>, tile_kernels<P_BF16S>}) {
      int n = 0;
      const StepKernel *k = tiles(&n);
      t.insert(t.end(), k, k + n);
    }
    return t;
  }();
  *count = (int)all.size();
  return all.data();
}

const void *reduce_partial_kernel(int prec) { return of_prec(prec) ? of_prec(prec)->reduce_partial : nullptr; }
const void *bgk_psi_kernel(int prec) { return of_prec(prec) ? of_prec(prec)->bgk_psi : nullptr; }
const void *bgk_reduce_partial_kernel(int prec) { return of_prec(prec) ? of_prec(prec)->bgk_reduce_partial : nullptr; }

const void *reduce_final_kernel() { return (const void *)&k_reduce_final; }
const void *reduce_final_out_kernel() { return (const void *)&k_reduce_final_out; }

static const BatchKernels *batch_of_prec(int prec) {
  switch (prec) {
    case P_F64: return &batch_kernels<P_F64>();
    case P_F32: return &batch_kernels<P_F32>();
    case P_F16S: return &batch_kernels<P_F16S>();
    case P_BF16S: return &batch_kernels<P_BF16S>();
  }
  return nullptr;
}

const void *batch_step_kernel(int prec, int vec_class, int rows) {
  const BatchKernels *k = batch_of_prec(prec);
  if (!k || vec_class < 0 || vec_class > 2) return nullptr;
  return rows == 6 ? k->step[0][vec_class] : rows == 14 ? k->step[1][vec_class] : rows == 30 ? k->step[2][vec_class] : nullptr;
}

// Two steps per launch, two columns per lane
const void *batch_fused_kernel(int prec, int rows) {
  const BatchKernels *k = batch_of_prec(prec);
  if (!k) return nullptr;
  return rows == 2 ? k->fused[0] : rows == 6 ? k->fused[1] : rows == 14 ? k->fused[2] : rows == 30 ? k->fused[3] : nullptr;
}

// Grids resident in LDS for a burst: two columns per lane
const void *batch_lds_kernel(int prec, int rows) {
  const BatchKernels *k = batch_of_prec(prec);
  if (!k) return nullptr;
  return rows == 6 ? k->lds[0] : rows == 14 ? k->lds[1] : nullptr;
}

const BatchTileKernel *batch_tile_kernel(int prec, int i) {
  const BatchKernels *k = batch_of_prec(prec);
  return k && i >= 0 && i < kBatchTiles && k->tile[i].fn ? &k->tile[i] : nullptr;
}

const void *batch_reduce_kernel(int prec) { return batch_of_prec(prec) ? batch_of_prec(prec)->reduce : nullptr; }

const void *batch_classify_kernel(int vec) {
  switch (vec) {
    case 1: return (const void *)&k_batch_classify<1>;
    case 2: return (const void *)&k_batch_classify<2>;
    case 4: return (const void *)&k_batch_classify<4>;
  }
  return nullptr;
}

const void *batch_reduce_final_kernel() { return (const void *)&k_reduce_batch_final; }

}  // namespace lbt1
