// Step and reduction kernels of one storage precision and the part of the kernel
// table the runtime selects from.  Compiled once per precision (LBT1_PREC).
#include "lbt1_bgk.hpp"
#include "lbt1_fused.hpp"
#include "lbt1_fused_wall.hpp"
#include "lbt1_internal.hpp"
#include "lbt1_multiphase.hpp"
#include "lbt1_step.hpp"

#ifndef LBT1_PREC
#error "compile with -DLBT1_PREC=0..3 (P_F64 ... P_BF16S)"
#endif

namespace lbt1 {

#define GATHER(P, HW, W) \
  {P, HW, W, KIND_GATHER, 0, 0, (const void *)&k_step_gather<P, HW, W>, "k_step_gather<" #P "," #HW "," #W ">", 1, 0}
#define STRIP(P, HW, W, V, R)                                                    \
  {P, HW, W, KIND_STRIP, V, R, (const void *)&k_step_strip<P, HW, W, V, R>, \
   "k_step_strip<" #P "," #HW "," #W "," #V "," #R ">", 1, 0}
// K steps per launch, fully periodic grids without wall or fixed nodes
#define FUSED(P, V, R, K)                                                        \
  {P, false, 0, KIND_STRIP, V, R, (const void *)&k_step_fused<P, V, R, K>, \
   "k_step_fused<" #P "," #V "," #R "," #K ">", K, 0}
#define FUSED_ROWS(P, V, K) FUSED(P, V, 6, K), FUSED(P, V, 14, K)
// two steps per launch on grids with walls, fixed nodes or non-periodic axes
#define FUSED_WALL(P, W, V, R)                                                              \
  {P, true, W, KIND_STRIP, V, R, (const void *)&k_step_fused_wall<P, W, V, R>,           \
   "k_step_fused_wall<" #P "," #W "," #V "," #R ">", 2, 0}
// (2-row strips: the shortest walk, for small grids bound by its latency)
#define FUSED_WALL_ALL(P)                                                                       \
  FUSED_WALL(P, 0, 2, 2), FUSED_WALL(P, 0, 2, 6), FUSED_WALL(P, 0, 2, 14), FUSED_WALL(P, 1, 2, 2), \
      FUSED_WALL(P, 1, 2, 6), FUSED_WALL(P, 1, 2, 14)
// 30 rows: fewer rounds of resident wavefronts on the largest grids (FP64 at 30
// rows would spill a scalar register)
#define FUSED_WALL_TALL(P) FUSED_WALL(P, 0, 2, 30), FUSED_WALL(P, 1, 2, 30)
#define FUSED_TALL(P, V, K) FUSED(P, V, 22, K), FUSED(P, V, 30, K)
#define STRIP_WALLS(P, V, R) STRIP(P, false, 0, V, R), STRIP(P, true, 0, V, R), STRIP(P, true, 1, V, R)
#define STRIP_ROWS(P, V) STRIP_WALLS(P, V, 6), STRIP_WALLS(P, V, 14)
// 8 columns per lane only without walls: the wall-aware variants at that width
// need more registers than a wavefront has and spill (the build refuses any
// kernel that spills or uses scratch memory)
#define STRIP_ROWS_NOWALL(P, V) STRIP(P, false, 0, V, 6), STRIP(P, false, 0, V, 14)
#define GATHER_ALL(P) GATHER(P, false, 0), GATHER(P, true, 0), GATHER(P, true, 1)
// population grids one step at a time: multiphase ones, and short calls on the others
#define BGK(P, HW, W, SC) \
  {P, HW, W, KIND_BGK, 0, 0, (const void *)&k_bgk_step<P, HW, W, SC>, "k_bgk_step<" #P "," #HW "," #W "," #SC ">", 1, SC}
#define BGK_ALL(P)                                                                            \
  BGK(P, false, 0, false), BGK(P, true, 0, false), BGK(P, true, 1, false), BGK(P, false, 0, true), \
      BGK(P, true, 0, true), BGK(P, true, 1, true)
// multiphase LBMTau1: gather for any geometry, strips for periodic grids without walls
#define SC_GATHER(P, HW, W) \
  {P, HW, W, KIND_GATHER, 0, 0, (const void *)&k_step_sc_gather<P, HW, W>, "k_step_sc_gather<" #P "," #HW "," #W ">", 1, 1}
#define SC_STRIP(P, V, R) \
  {P, false, 0, KIND_STRIP, V, R, (const void *)&k_step_sc_strip<P, V, R>, "k_step_sc_strip<" #P "," #V "," #R ">", 1, 1}
// two multiphase steps per launch (4 columns per lane: each step widens the
// wrong halo columns by two); 22 rows measured fastest on large drops, 30
// would spill
#define SC_FUSED(P, V, R) \
  {P, false, 0, KIND_STRIP, V, R, (const void *)&k_step_sc_fused<P, V, R>, "k_step_sc_fused<" #P "," #V "," #R ">", 2, 1}
#define SC_ALL(P, V)                                                                                \
  SC_GATHER(P, false, 0), SC_GATHER(P, true, 0), SC_GATHER(P, true, 1), SC_STRIP(P, V, 6), SC_STRIP(P, V, 14)

#define TABLE_COMMON(P) \
  GATHER_ALL(P), STRIP_ROWS(P, 1), STRIP_ROWS(P, 2), FUSED_ROWS(P, 2, 2), FUSED_WALL_ALL(P), BGK_ALL(P), SC_ALL(P, 2)
// 16-bit storage: strips up to 8 columns per lane, taller two-step strips (fewer
// redundant halo rows per stored row)
#define TABLE_HALF(P)                                                                                  \
  TABLE_COMMON(P), STRIP_ROWS(P, 4), STRIP_ROWS_NOWALL(P, 8), FUSED_ROWS(P, 4, 2), FUSED_TALL(P, 2, 2), \
      FUSED_WALL_TALL(P)

static const StepKernel kTable[] = {
#if LBT1_PREC == 0
    TABLE_COMMON(P_F64),
#elif LBT1_PREC == 1
    TABLE_COMMON(P_F32), STRIP_ROWS(P_F32, 4), FUSED_ROWS(P_F32, 4, 2), FUSED_WALL_TALL(P_F32),
    // three steps per launch at 4 columns per lane (built for two wavefronts per
    // SIMD: FP64, and 16-bit storage with its codec, would need scratch memory);
    // four would need more registers than a wavefront has
    FUSED_ROWS(P_F32, 4, 3),
    // 22 and 28 rows: the runtime picks the height whose strip count best fills the
    // last round of resident wavefronts (each with its two-step companion)
    FUSED(P_F32, 4, 22, 3), FUSED(P_F32, 4, 22, 2), FUSED(P_F32, 4, 28, 3), FUSED(P_F32, 4, 28, 2),
    SC_STRIP(P_F32, 4, 6), SC_STRIP(P_F32, 4, 14),
    SC_FUSED(P_F32, 4, 6), SC_FUSED(P_F32, 4, 14), SC_FUSED(P_F32, 4, 22),
#elif LBT1_PREC == 2
    TABLE_HALF(P_F16S),
#else
    TABLE_HALF(P_BF16S),
#endif
};

template <>
const PrecKernels &prec_kernels<LBT1_PREC>() {
  static const PrecKernels k = {kTable, (int)(sizeof(kTable) / sizeof(kTable[0])),
                                (const void *)&k_reduce_partial<LBT1_PREC>, (const void *)&k_bgk_psi<LBT1_PREC>,
                                (const void *)&k_bgk_reduce_partial<LBT1_PREC>};
  return k;
}

}  // namespace lbt1
