// The tile kernels (several steps per launch on small grids) of one storage precision.
// Compiled once per precision (LBT1_PREC).
#include "lbt1_bgk_tile.hpp"
#include "lbt1_internal.hpp"
#include "lbt1_sc_tile.hpp"
#include "lbt1_tile.hpp"

#ifndef LBT1_PREC
#error "compile with -DLBT1_PREC=0..3 (P_F64 ... P_BF16S)"
#endif

namespace lbt1 {

#define LBT1_STR2(x) #x
#define LBT1_STR(x) LBT1_STR2(x)

#define TILE(P, HW, WL, W, CPL, RPT, TH, ...)                                                        \
  {P, HW, WL, KIND_TILE, W * CPL, TH / W * RPT, (const void *)&k_step_tile<P, HW, WL, W, CPL, RPT, TH>, \
   "k_step_tile<" LBT1_STR(P) "," #HW "," #WL "," #W "," #CPL "," #RPT "," #TH ">", 1, 0, TH, __VA_ARGS__}
#define TILE_WALLED(...) TILE_WALLED_(__VA_ARGS__)
#define TILE_WALLED_(P, W, CPL, RPT, TH, ...) \
  TILE(P, true, 0, W, CPL, RPT, TH, __VA_ARGS__), TILE(P, true, 1, W, CPL, RPT, TH, __VA_ARGS__)
#define TILE_FREE(P, W, CPL, RPT, TH, ...) TILE(P, false, 0, W, CPL, RPT, TH, __VA_ARGS__)

// Two blocks of every shape fit a CU (with one, loads and stores are not overlapped with
// another block's steps: 128 x 128 regions on 1024 threads take 18 % longer at 4096^2
// FP32 than 128 x 64 on 512).  Small regions for grids bound by latency, large ones
// for less halo; with walls the masks take registers, so the largest are smaller.
// The three figures are the times the runtime's choice is made by, fitted to grids of
// 48^2 to 8192^2 (see default_config and sc_choice).
#define BGK_TILE(P, HW, WL, W, RPT, TH, ...)                                                        \
  {P, HW, WL, KIND_BGK_TILE, W, TH / W * RPT, (const void *)&k_bgk_tile<P, HW, WL, W, RPT, TH>,     \
   "k_bgk_tile<" LBT1_STR(P) "," #HW "," #WL "," #W "," #RPT "," #TH ">", 1, 0, TH, __VA_ARGS__}
#define BGK_FREE(P, W, RPT, TH, ...) BGK_TILE(P, false, 0, W, RPT, TH, __VA_ARGS__)
#define BGK_WALLED(...) BGK_WALLED_(__VA_ARGS__)
#define BGK_WALLED_(P, W, RPT, TH, ...) \
  BGK_TILE(P, true, 0, W, RPT, TH, __VA_ARGS__), BGK_TILE(P, true, 1, W, RPT, TH, __VA_ARGS__)

#define SC_TILE(P, HW, WL, W, RPT, TH, ...)                                                         \
  {P, HW, WL, KIND_SC_TILE, W, TH / W * RPT, (const void *)&k_sc_tile<P, HW, WL, W, RPT, TH>,       \
   "k_sc_tile<" LBT1_STR(P) "," #HW "," #WL "," #W "," #RPT "," #TH ">", 1, 1, TH, __VA_ARGS__}
#define SC_FREE(P, W, RPT, TH, ...) SC_TILE(P, false, 0, W, RPT, TH, __VA_ARGS__)
#define SC_WALLED(...) SC_WALLED_(__VA_ARGS__)
#define SC_WALLED_(P, W, RPT, TH, ...) \
  SC_TILE(P, true, 0, W, RPT, TH, __VA_ARGS__), SC_TILE(P, true, 1, W, RPT, TH, __VA_ARGS__)

static const StepKernel kTable[] = {
#if LBT1_PREC == 0
    TILE_FREE(P_F64, 32, 1, 2, 512, 3.7, 0.442, 0.73), TILE_WALLED(P_F64, 32, 1, 2, 512, 6.6, 0.569, 0.37),
    TILE_FREE(P_F64, 64, 1, 4, 512, 3.5, 0.972, 0.83), TILE_WALLED(P_F64, 64, 1, 4, 512, 7.8, 1.261, 0.0),
    TILE_FREE(P_F64, 64, 1, 8, 512, 3.2, 2.056, 1.51),
    BGK_FREE(P_F64, 32, 2, 512, 4.2, 0.522, 2.95), BGK_WALLED(P_F64, 32, 2, 512, 8.3, 0.679, 1.82),
    BGK_FREE(P_F64, 64, 4, 512, 3.4, 1.150, 5.33), BGK_WALLED(P_F64, 64, 4, 512, 6.4, 1.588, 6.24),
    SC_FREE(P_F64, 32, 2, 512, 3.1, 0.756, 0.59), SC_WALLED(P_F64, 32, 2, 512, 5.0, 0.868, 0.89),
    SC_FREE(P_F64, 64, 4, 512, 3.4, 1.472, 0.99), SC_WALLED(P_F64, 64, 4, 512, 7.4, 1.864, 0.07),
    SC_FREE(P_F64, 64, 8, 512, 3.4, 3.022, 2.07),
#elif LBT1_PREC == 1
    TILE_FREE(P_F32, 32, 1, 1, 1024, 3.1, 0.235, 0.69), TILE_WALLED(P_F32, 32, 1, 1, 1024, 4.5, 0.350, 0.67),
    TILE_FREE(P_F32, 64, 1, 2, 1024, 3.2, 0.528, 0.48), TILE_WALLED(P_F32, 64, 1, 2, 1024, 5.6, 0.655, 0.19),
    TILE_FREE(P_F32, 64, 1, 4, 1024, 3.3, 1.100, 1.20), TILE_WALLED(P_F32, 64, 1, 8, 512, 14.0, 1.200, 1.10),
    TILE_FREE(P_F32, 64, 2, 8, 512, 6.5, 1.930, 3.00),
    BGK_FREE(P_F32, 32, 2, 512, 4.2, 0.276, 1.92), BGK_WALLED(P_F32, 32, 2, 512, 6.8, 0.356, 1.36),
    BGK_FREE(P_F32, 64, 4, 512, 4.1, 0.752, 3.20), BGK_WALLED(P_F32, 64, 4, 512, 7.7, 0.953, 1.40),
    BGK_FREE(P_F32, 64, 8, 512, 2.9, 1.897, 4.96),
    SC_FREE(P_F32, 32, 2, 512, 3.3, 0.414, 0.35), SC_WALLED(P_F32, 32, 2, 512, 4.6, 0.549, 0.36),
    SC_FREE(P_F32, 64, 4, 512, 3.4, 0.912, 0.35), SC_WALLED(P_F32, 64, 4, 512, 6.1, 1.139, 0.00),
    SC_FREE(P_F32, 64, 8, 512, 3.6, 2.098, 0.52),
#else
#if LBT1_PREC == 2
#define P_HALF P_F16S
#else
#define P_HALF P_BF16S
#endif
    TILE_FREE(P_HALF, 32, 1, 1, 1024, 3.3, 0.311, 0.41), TILE_WALLED(P_HALF, 32, 1, 1, 1024, 4.6, 0.360, 0.57),
    TILE_FREE(P_HALF, 64, 1, 2, 1024, 3.3, 0.579, 0.36), TILE_WALLED(P_HALF, 64, 1, 2, 1024, 5.5, 0.681, 0.15),
    TILE_FREE(P_HALF, 64, 1, 4, 1024, 3.6, 1.368, 0.0), TILE_WALLED(P_HALF, 64, 1, 8, 512, 14.0, 1.400, 0.90),
    TILE_FREE(P_HALF, 64, 2, 8, 512, 5.9, 2.733, 0.0),
    BGK_FREE(P_HALF, 32, 2, 512, 4.7, 0.632, 0.72), BGK_WALLED(P_HALF, 32, 2, 512, 7.4, 0.770, 0.00),
    BGK_FREE(P_HALF, 64, 4, 512, 5.4, 1.333, 0.64), BGK_WALLED(P_HALF, 64, 4, 512, 9.4, 1.512, 0.00),
    BGK_FREE(P_HALF, 64, 8, 512, 5.4, 2.841, 1.41),
    SC_FREE(P_HALF, 32, 2, 512, 3.2, 0.560, 0.16), SC_WALLED(P_HALF, 32, 2, 512, 4.7, 0.658, 0.12),
    SC_FREE(P_HALF, 64, 4, 512, 3.5, 1.160, 0.01), SC_WALLED(P_HALF, 64, 4, 512, 6.5, 1.279, 0.00),
    SC_FREE(P_HALF, 64, 8, 512, 3.8, 2.472, 0.00),
#endif
};

template <>
const StepKernel *tile_kernels<LBT1_PREC>(int *count) {
  *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}

}  // namespace lbt1
