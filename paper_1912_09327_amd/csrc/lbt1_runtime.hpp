// Host-side state of grids and batches (shared by the runtime sources).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <initializer_list>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "../../include/lbt1.h"
#include "lbt1_internal.hpp"
#include "lbt1_tile_args.hpp"

namespace lbt1 {

constexpr int kReduceBlocks = 1024;  // most partial rows a reduction writes

struct Layout {
  int pitch;          // values per row of one field (nx rounded up to 64)
  int nfield;         // fields per parity: 3 moments, or 9 populations
  int rs;             // field row stride in values: pitch (planar) or nfield * pitch
  bool interleaved;   // the field rows of a lattice row are adjacent
  size_t field_off[9];  // byte offset of field q inside a parity block
  size_t state;       // bytes of one parity block (all fields, 256-byte multiple)
  size_t flags_off, flags_bytes;
  size_t snap_off;    // 0 without LBT1_OPT_SNAPSHOT
  int snap_rs;        // row stride of the snapshot's three moment fields
  size_t snap_field_off[3];
  size_t psi_off;     // multiphase population grids: psi of every node, 0 otherwise
  int nparts;
  size_t part_off, out_off, trash_off;
  size_t total;
};

Layout layout_of(int nx, int ny, int prec, uint32_t options);
size_t value_bytes(int prec);
lbt1_status fail(lbt1_status st, const char *fmt, ...);
lbt1_status check_device(int *dev_out, int *cus);
void encode_values(int prec, const double *in, size_t n, double inv_scale, void *out);
void decode_values(int prec, const void *in, size_t n, double scale, double *out);
lbt1_status hip_fail(hipError_t e, const char *what);
void clear_error();
hipError_t upload(void *dst, const void *host, size_t bytes, std::initializer_list<void *> more, hipStream_t s);

// Rows of stored values in device memory: row r of field q starts r * stride + q * field values
// of c bytes after src.  scratch: device memory of the grid that a readout may overwrite.
struct RowSource {
  const char *src;
  size_t c, stride, field;
  void *scratch;
  size_t scratch_bytes;
  hipStream_t stream;
};
hipError_t pack_rows(const RowSource &s, size_t row0, size_t rows, size_t w, uint32_t fields);

// take(q, r, row) with the w stored values of row r of each field q of the bits `fields`.  One of
// three ways, by an estimate of its time (measured: 8 bytes a nanosecond, 10 us a copy, and as
// much for each row of a strided copy, 22 us for a launch that packs and its copy):
//   whole rows of all the fields between, kReadStage bytes at a time, which the conversion then
//   finds in the cache (8192^2 FP32: 92 ms, in one piece 255; box of 200 x 180 x 150: 10 ms);
//   rows one by one, a strided copy, where rows are long and most of the fields are not wanted;
//   packed on the device into `scratch` first, where the window is narrow: a column of an
//   8192^2 FP32 grid in 0.1 ms, where whole rows move and stage 805 MB in 280 ms.
constexpr size_t kReadStage = 1u << 20;
template <typename F>
lbt1_status read_rows(const RowSource &s, uint32_t fields, size_t w, size_t rows, const F &take) {
  if (!fields) return LBT1_OK;
  int q[32], n_ = 0;
  for (int k = 0; k < 32; ++k)
    if (fields >> k & 1u) q[n_++] = k;
  const size_t n = (size_t)n_, first = (size_t)q[0], line = w * s.c;
  const bool adjacent = s.field < s.stride;  // the rows of all fields of a lattice row
  const size_t span = adjacent ? ((size_t)q[n - 1] - first) * s.field + w : w, passes = adjacent ? 1 : n;
  const size_t fit = s.scratch_bytes / (n * line);  // rows of a launch that packs
  const size_t wanted = n * rows * line, all = passes * ((rows - 1) * s.stride + span) * s.c;
  const double whole = (passes + (double)all / kReadStage) * 1e4 + all / 8.0;
  const double strided = n * rows * 1e4 + wanted / 8.0;
  const double packed = fit ? ((rows + fit - 1) / fit) * 2.2e4 + wanted / 8.0 : 1e300;
  enum { WHOLE, STRIDED, PACKED } how = packed < whole && packed < strided ? PACKED : strided < whole ? STRIDED : WHOLE;
  const size_t few = how == PACKED    ? fit
                     : how == STRIDED ? kReadStage / line
                                      : kReadStage / (s.stride * s.c);
  const size_t block = std::min(rows, std::max<size_t>(1, few));  // rows at a time
  const size_t bytes = how == PACKED ? block * n * line : how == STRIDED ? block * line : ((block - 1) * s.stride + span) * s.c;
  const std::unique_ptr<char[]> stage(new (std::nothrow) char[bytes]);
  if (!stage) return fail(LBT1_ENOMEM, "host staging");
  hipError_t e = hipSuccess;
  const size_t turns = how == STRIDED ? n : how == WHOLE ? passes : 1;
  for (size_t t = 0; t < turns; ++t)
    for (size_t r = 0; r < rows; r += block) {
      const size_t h = std::min(block, rows - r), from = how == WHOLE && adjacent ? first : (size_t)q[t];
      const char *const src = s.src + (r * s.stride + from * s.field) * s.c;
      if (how == PACKED) {
        if ((e = pack_rows(s, r, h, w, fields)) == hipSuccess)
          e = hipMemcpyAsync(stage.get(), s.scratch, h * n * line, hipMemcpyDeviceToHost, s.stream);
        if (e == hipSuccess) e = hipStreamSynchronize(s.stream);
      } else if (how == STRIDED) {
        e = hipMemcpy2D(stage.get(), line, src, s.stride * s.c, line, h, hipMemcpyDeviceToHost);
      } else {
        e = hipMemcpy(stage.get(), src, ((h - 1) * s.stride + span) * s.c, hipMemcpyDeviceToHost);
      }
      if (e != hipSuccess) return hip_fail(e, "copy to the host");
      const size_t k1 = how == PACKED || (how == WHOLE && adjacent) ? n : t + 1;
      for (size_t y = 0; y < h; ++y)
        for (size_t k = t; k < k1; ++k)
          take(q[k], r + y,
               stage.get() + (how == PACKED    ? (k * h + y) * line
                              : how == STRIDED ? y * line
                                               : (y * s.stride + ((size_t)q[k] - from) * s.field) * s.c));
    }
  return LBT1_OK;
}

}  // namespace lbt1

namespace lbt1 {
// How a call of very few steps runs where the library chose the grid's kernel and another one
// takes them in less time: `times` launches of kern, which together advance them.
struct Brief {
  const StepKernel *kern = nullptr;
  int times = 0;
  StripMap map{};
  dim3 grid{1, 1, 1}, block{1, 1, 1};
};
constexpr int kBrief = 3;  // most steps of such a call
}  // namespace lbt1

struct lbt1_grid {
  int device = 0, cus = 0;
  int nx = 0, ny = 0;
  uint32_t periodic = 0;
  int prec = 0, wall = 0;
  uint32_t options = 0;
  bool pop = false;       // LBT1_OPT_POPULATIONS: stored-population BGK
  double tau = 1.0;
  bool mp = false;        // LBT1_OPT_MULTIPHASE: Shan-Chen force
  double sc_G = 0.0, sc_rho0 = 1.0;
  void *psi = nullptr;    // population grids with sc: psi field
  double F[2] = {0, 0};
  double sc[2] = {1, 1};  // decode scales of d and j
  lbt1::Layout L{};
  hipStream_t stream = nullptr;
  bool own_stream = false;
  char *base = nullptr;
  bool own_mem = false;
  void *plane[2][9] = {};
  uint8_t *flags = nullptr;
  void *snap[3] = {};
  double *partials = nullptr;
  double *red_out = nullptr;
  double *red_host = nullptr;  // pinned
  int parity = 0;
  int64_t steps = 0;
  bool geometry = false;
  bool haswall = false;
  int64_t fluid = 0;
  // population grids: moments given to set_geometry for SOLID and FIXED nodes
  // (reported by the readout), node index and (rho, jx, jy)
  std::vector<size_t> given_idx;
  std::vector<double> given_val;
  // step kernel
  lbt1_kernel_config cfg{};
  bool user_cfg = false;
  const lbt1::StepKernel *kern = nullptr;   // advances kern->steps steps per launch
  const lbt1::StepKernel *kern1 = nullptr;  // single-step kernel of the same launch shape
  const lbt1::StepKernel *kern2 = nullptr;  // two-step kernel of the same strip shape, when kern takes three
  lbt1::StripMap map{};
  int launch_steps = 1;  // steps one launch of kern takes
  lbt1::Brief brief[lbt1::kBrief];  // by steps - 1
  dim3 grid{1, 1, 1}, block{1, 1, 1};
  dim3 grid1{1, 1, 1}, block1{1, 1, 1};  // launch shape of kern1
  hipGraphExec_t burst[2] = {nullptr, nullptr};
  bool graph_valid = false;
  // batch residency
  lbt1_batch *batch = nullptr;
  int slot = -1;
};

namespace lbt1 {
lbt1_status bind_config(lbt1_grid *g, const lbt1_kernel_config &want, int cus);
StepArgs step_args(const lbt1_grid *g, int src_parity);
lbt1_status enqueue_steps(lbt1_grid *g, int64_t n, hipStream_t s, bool use_graph);
lbt1_status enqueue_reduce(lbt1_grid *g, uint32_t what, hipStream_t s);
// tile kernels (lbt1_tile.hpp, lbt1_bgk_tile.hpp): most steps of one launch, the kernel of a
// shape, the tiles of a grid, the modelled time of a step
constexpr int kMaxTileSteps = 64;
const StepKernel *find_tile(int kind, int prec, bool haswall, int wall, int w, int rows, int waves);
bool tile_map(int nx, int ny, uint32_t periodic, const lbt1_kernel_config &c, int steps, TileMap *m, int reach = 1);
double tile_us(const StepKernel &k, int steps, long tiles, int cus);
}  // namespace lbt1
