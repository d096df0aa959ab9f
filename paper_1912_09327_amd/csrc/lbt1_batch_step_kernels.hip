// Batched kernels of one storage precision (always wall-aware).  Compiled once per
// precision (LBT1_PREC).
#include "lbt1_batch_kernels.hpp"
#include "lbt1_internal.hpp"

#ifndef LBT1_PREC
#error "compile with -DLBT1_PREC=0..3 (P_F64 ... P_BF16S)"
#endif

namespace lbt1 {

#define BATCH_STEP(V, R) (const void *)&k_step_batch<LBT1_PREC, V, R>
#define BATCH_FUSED(R) (const void *)&k_step_batch_fused<LBT1_PREC, R>

template <>
const BatchKernels &batch_kernels<LBT1_PREC>() {
  static const BatchKernels k = {
#if LBT1_PREC == 0
      // FP64: up to 2 columns per lane; 30-row strips would spill, and the LDS-resident
      // kernel would spill scalar registers (only grids of about 32 x 32 would fit)
      {{BATCH_STEP(1, 6), BATCH_STEP(2, 6), nullptr},
       {BATCH_STEP(1, 14), BATCH_STEP(2, 14), nullptr},
       {nullptr, nullptr, nullptr}},
      {BATCH_FUSED(2), BATCH_FUSED(6), BATCH_FUSED(14), nullptr},
      {nullptr, nullptr},
      {{32, 32, 512, (const void *)&k_step_batch_tile<LBT1_PREC, 32, 1, 2, 512>},
       {64, 32, 512, (const void *)&k_step_batch_tile<LBT1_PREC, 64, 1, 4, 512>},
       {0, 0, 0, nullptr}},
#else
      // strips of 6 rows (short: half the serial latency of a strip, for classes with
      // too few strips to fill the device), 14 rows (tall) and 30 rows (fewer, longer
      // walks per item)
      {{BATCH_STEP(1, 6), BATCH_STEP(2, 6), BATCH_STEP(4, 6)},
       {BATCH_STEP(1, 14), BATCH_STEP(2, 14), BATCH_STEP(4, 14)},
       {BATCH_STEP(1, 30), BATCH_STEP(2, 30), BATCH_STEP(4, 30)}},
      {BATCH_FUSED(2), BATCH_FUSED(6), BATCH_FUSED(14), BATCH_FUSED(30)},
      {(const void *)&k_step_batch_lds<LBT1_PREC, 2, 6>, (const void *)&k_step_batch_lds<LBT1_PREC, 2, 14>},
      {{32, 32, 1024, (const void *)&k_step_batch_tile<LBT1_PREC, 32, 1, 1, 1024>},
       {64, 32, 1024, (const void *)&k_step_batch_tile<LBT1_PREC, 64, 1, 2, 1024>},
       {64, 64, 512, (const void *)&k_step_batch_tile<LBT1_PREC, 64, 1, 8, 512>}},
#endif
      (const void *)&k_reduce_batch<LBT1_PREC>};
  return k;
}

}  // namespace lbt1
