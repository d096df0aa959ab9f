// Host runtime and C ABI of liblbt1 (see include/lbt1.h).
//
// A grid owns (or borrows) one device allocation laid out as
//   planes[parity 0][d, jx, jy] planes[parity 1][d, jx, jy] flags [snapshot d, jx, jy]
//   reduction partials, reduction result
// Each plane is ny rows of `pitch` values (pitch = nx rounded up to 64), the
// structure-of-arrays form of the paper's R, U, V tables (Algorithm 1), with
// x fastest so a wavefront's loads of one row are contiguous.  The two
// parities are the paper's ping-pong copies; lbt1_step flips between them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

#include "../../include/lbt1.h"
#include "lbt1_internal.hpp"
#include "lbt1_runtime.hpp"

namespace lbt1 {

// ----------------------------------------------------------------- errors
static thread_local std::string g_err;

lbt1_status fail(lbt1_status st, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return st;
}

lbt1_status hip_fail(hipError_t e, const char *what) {
  return fail(LBT1_EDEVICE, "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
}

void clear_error() { g_err.clear(); }

// ----------------------------------------------------------------- layout
size_t value_bytes(int prec) {
  switch (prec) {
    case LBT1_F64: return 8;
    case LBT1_F32: return 4;
    case LBT1_F16S:
    case LBT1_BF16S: return 2;
  }
  return 0;
}

static size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

Layout layout_of(int nx, int ny, int prec, uint32_t options) {
  Layout L{};
  const size_t c = value_bytes(prec);
  L.pitch = (int)round_up((size_t)nx, 64);
  L.interleaved = !(options & LBT1_OPT_PLANAR);
  const bool pop = options & LBT1_OPT_POPULATIONS;
  const int nf = pop ? 9 : 3;
  L.nfield = nf;
  const size_t plane = round_up((size_t)L.pitch * ny * c, 256);
  if (L.interleaved) {
    // [ny][nf][pitch]: a wavefront reading (writing) one lattice row touches one
    // contiguous stretch of the parity block
    L.rs = nf * L.pitch;
    for (int q = 0; q < nf; ++q) L.field_off[q] = (size_t)q * L.pitch * c;
    L.state = round_up((size_t)nf * L.pitch * ny * c, 256);
  } else {
    // [nf][ny][pitch]: separate planes
    L.rs = L.pitch;
    for (int q = 0; q < nf; ++q) L.field_off[q] = (size_t)q * plane;
    L.state = nf * plane;
  }
  L.flags_off = 2 * L.state;
  L.flags_bytes = round_up((size_t)L.pitch * ny, 256);
  size_t off = L.flags_off + L.flags_bytes;
  L.snap_off = 0;
  L.snap_rs = L.rs;
  for (int q = 0; q < 3; ++q) L.snap_field_off[q] = L.field_off[q];
  if (options & LBT1_OPT_SNAPSHOT) {
    L.snap_off = off;
    if (pop) {
      // the residual compares moments: three planes of rho - 1, jx, jy
      L.snap_rs = L.pitch;
      for (int q = 0; q < 3; ++q) L.snap_field_off[q] = (size_t)q * plane;
      off += 3 * plane;
    } else {
      off += L.state;
    }
  }
  L.psi_off = 0;
  if (pop && (options & LBT1_OPT_MULTIPHASE)) {
    L.psi_off = off;
    off += round_up((size_t)L.pitch * ny * (prec == LBT1_F64 ? 8 : 4), 256);
  }
  L.nparts = kReduceBlocks;
  L.part_off = off;
  off += round_up((size_t)L.nparts * 6 * sizeof(double), 256);
  L.out_off = off;
  off += 256;
  L.trash_off = off;  // 3 KiB: stores of lanes / rows outside the grid land here (one region per field)
  off += 3 * kTrashRegion;
  L.total = off;
  return L;
}

static bool valid_shape(int nx, int ny) { return nx >= 3 && ny >= 3 && nx <= 65536 && ny <= 65536; }
static bool valid_prec(int p) { return p >= LBT1_F64 && p <= LBT1_BF16S; }

static bool pow2_or_zero(double s) {
  if (s == 0.0) return true;
  if (!(s > 0.0) || !std::isfinite(s)) return false;
  int e;
  double m = std::frexp(s, &e);
  return m == 0.5;
}

// ----------------------------------------------------------------- host codecs
// The conversions below are written without branches and library calls, so that the loops
// of encode_values and decode_values run several values at a time: one rounding from the
// 64-bit value, half to even, gradual underflow, infinity above the largest value.
//
// A double rounded to MANT significand bits (at most 11) for exponents from EMIN up, to
// the quantum of EMIN below: integer rounding of the fraction, or the addition of a number
// whose unit in the last place is that quantum.
constexpr double pow2(int e) { return e < 0 ? 0.5 * pow2(e + 1) : e > 0 ? 2.0 * pow2(e - 1) : 1.0; }
template <int MANT, int EMIN>
static inline double round_bits(double x) {
  uint64_t u;
  std::memcpy(&u, &x, 8);
  constexpr int drop = 53 - MANT;
  const uint64_t r = (u + (((u >> drop) & 1) + ((1ull << (drop - 1)) - 1))) & ~((1ull << drop) - 1);
  double big;
  std::memcpy(&big, &r, 8);
  constexpr double magic = 1.5 * pow2(EMIN - (MANT - 1) + 52), least = pow2(EMIN);
  const double tiny = (x + magic) - magic;
  return std::fabs(x) < least ? tiny : big;
}

static inline uint16_t encode_half(double v) {
  const double r = round_bits<11, -14>(v);
  uint64_t u, uv;
  std::memcpy(&u, &r, 8);
  std::memcpy(&uv, &v, 8);
  const uint16_t sign = (uint16_t)(uv >> 48) & 0x8000;
  const double a = std::fabs(r);
  const uint16_t normal = (uint16_t)((u >> 42) - (uint64_t)((1023 - 15) << 10)) & 0x7fff;
  constexpr double least = 6.103515625e-05;  // 2^-14
  const uint16_t sub = (uint16_t)(int32_t)((a < least ? a : 0.0) * 16777216.0);  // in units of 2^-24
  uint16_t h = a < least ? sub : normal;
  h = a > 65504.0 ? (uint16_t)0x7c00 : h;
  h = v != v ? (uint16_t)0x7e00 : h;
  return sign | h;
}
static inline uint16_t encode_bf16(double v) {
  const double r = round_bits<8, -126>(v);
  const float f = (float)r;  // exact, or infinite where r is past the largest value
  uint32_t u;
  uint64_t uv;
  std::memcpy(&u, &f, 4);
  std::memcpy(&uv, &v, 8);
  const uint16_t sign = (uint16_t)(uv >> 48) & 0x8000;  // (a negative value that rounds to zero keeps it)
  return v != v ? (uint16_t)0x7fc0 : (uint16_t)((u >> 16 & 0x7fff) | sign);
}
// (no subnormal float on the way: a host thread may flush those to zero)
static inline double decode_half(uint16_t b) {
  const uint32_t m = b & 0x7fff;
  // normal: the exponent moved from bias 15 to 127; 31 becomes 255
  const uint32_t normal = ((m << 13) + (112u << 23)) | (m >= 0x7c00 ? 0x7f800000u : 0u);
  const float small = (float)(int32_t)m * 5.9604644775390625e-08f;  // m < 2^10: in units of 2^-24
  uint32_t u;
  std::memcpy(&u, &small, 4);
  u = (m < 0x400 ? u : normal) | (uint32_t)(b & 0x8000) << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return (double)f;
}
static inline double decode_bf16(uint16_t b) {
  uint32_t u = (uint32_t)b << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return (double)f;
}

void encode_values(int prec, const double *in, size_t n, double inv_scale, void *out) {
  switch (prec) {
    case LBT1_F64: {
      double *o = (double *)out;
      for (size_t i = 0; i < n; ++i) o[i] = in[i];
      break;
    }
    case LBT1_F32: {
      float *o = (float *)out;
      for (size_t i = 0; i < n; ++i) o[i] = (float)in[i];
      break;
    }
    case LBT1_F16S: {
      uint16_t *o = (uint16_t *)out;
      for (size_t i = 0; i < n; ++i) o[i] = encode_half(in[i] * inv_scale);
      break;
    }
    case LBT1_BF16S: {
      uint16_t *o = (uint16_t *)out;
      for (size_t i = 0; i < n; ++i) o[i] = encode_bf16(in[i] * inv_scale);
      break;
    }
  }
}

void decode_values(int prec, const void *in, size_t n, double scale, double *out) {
  switch (prec) {
    case LBT1_F64: {
      const double *s = (const double *)in;
      for (size_t i = 0; i < n; ++i) out[i] = s[i];
      break;
    }
    case LBT1_F32: {
      const float *s = (const float *)in;
      for (size_t i = 0; i < n; ++i) out[i] = s[i];
      break;
    }
    case LBT1_F16S: {
      const uint16_t *s = (const uint16_t *)in;
      for (size_t i = 0; i < n; ++i) out[i] = decode_half(s[i]) * scale;
      break;
    }
    case LBT1_BF16S: {
      const uint16_t *s = (const uint16_t *)in;
      for (size_t i = 0; i < n; ++i) out[i] = decode_bf16(s[i]) * scale;
      break;
    }
  }
}

// ----------------------------------------------------------------- host copies
// `bytes` from host memory to `dst` and, on the device, to each of the `more` places after
// it (host memory crosses the bus once).
hipError_t upload(void *dst, const void *host, size_t bytes, std::initializer_list<void *> more, hipStream_t s) {
  hipError_t e = hipMemcpy(dst, host, bytes, hipMemcpyHostToDevice);
  for (void *p : more)
    if (e == hipSuccess && p) e = hipMemcpyAsync(p, dst, bytes, hipMemcpyDeviceToDevice, s);
  return e == hipSuccess ? hipStreamSynchronize(s) : e;
}

// Windows too narrow for whole rows, [field][row][w] (read_rows; the copy to the host bounds it)
struct PackArgs {
  const void *src;
  void *dst;
  unsigned long long stride, field;
  unsigned int w, rows, n;
  unsigned int which;  // bit q: field q is wanted
};
template <typename S>
__global__ void __launch_bounds__(256) k_pack_rows(PackArgs a) {
  const unsigned int total = a.n * a.rows * a.w;
  for (unsigned int i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const unsigned int x = i % a.w, kr = i / a.w, r = kr % a.rows;
    unsigned int which = a.which;
    for (unsigned int k = kr / a.rows; k > 0; --k) which &= which - 1;
    const unsigned int q = __builtin_ctz(which);
    static_cast<S *>(a.dst)[i] = static_cast<const S *>(a.src)[r * a.stride + q * a.field + x];
  }
}

// Rows row0 ... row0 + rows - 1 of the fields into the scratch, which holds them.
hipError_t pack_rows(const RowSource &s, size_t row0, size_t rows, size_t w, uint32_t fields) {
  PackArgs a{};
  a.src = s.src + row0 * s.stride * s.c;
  a.dst = s.scratch;
  a.stride = s.stride;
  a.field = s.field;
  a.w = (unsigned int)w;
  a.rows = (unsigned int)rows;
  a.n = (unsigned int)__builtin_popcount(fields);
  a.which = fields;
  const void *fn = s.c == 8   ? (const void *)&k_pack_rows<uint64_t>
                   : s.c == 4 ? (const void *)&k_pack_rows<uint32_t>
                              : (const void *)&k_pack_rows<uint16_t>;
  void *args[] = {&a};
  const size_t total = a.n * rows * w;
  return hipLaunchKernel(fn, dim3((unsigned int)std::min<size_t>(96, (total + 255) / 256)), dim3(256), args, 0, s.stream);
}

// ----------------------------------------------------------------- device check
lbt1_status check_device(int *dev_out, int *cus) {
  int ndev = 0;
  hipError_t e = hipGetDeviceCount(&ndev);
  if (e != hipSuccess) return fail(LBT1_EDEVICE, "no HIP device is visible: hipGetDeviceCount: %s (%d)", hipGetErrorString(e), (int)e);
  if (ndev <= 0) return fail(LBT1_EDEVICE, "no HIP device is visible");
  int dev = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return hip_fail(e, "hipGetDevice");
  hipDeviceProp_t prop;
  if ((e = hipGetDeviceProperties(&prop, dev)) != hipSuccess) return hip_fail(e, "hipGetDeviceProperties");
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return fail(LBT1_EDEVICE, "device %d is %s; this library is built for gfx950", dev, prop.gcnArchName);
  *dev_out = dev;
  if (cus) *cus = prop.multiProcessorCount;
  return LBT1_OK;
}

// ----------------------------------------------------------------- kernel selection
// A strip kernel with vec columns per lane fits a grid when vec divides nx, or
// when x is not periodic: then the last chunk of a row runs past nx into the
// row padding (pitch is nx rounded up to 64, a multiple of vec), whose flags
// are SOLID, exactly like the outside of a non-periodic axis.
static bool strip_fits(int nx, int vec, bool periodic_x) { return vec >= 1 && (nx % vec == 0 || !periodic_x); }
static int chunks_of(int nx, int vec) { return (nx + vec - 1) / vec; }

// The tile kernel of a kind with regions of w columns and `rows` rows on `waves` wavefronts.
const StepKernel *find_tile(int kind, int prec, bool haswall, int wall, int w, int rows, int waves) {
  int n = 0;
  const StepKernel *t = step_kernels(&n);
  for (int i = 0; i < n; ++i) {
    const StepKernel &k = t[i];
    if (k.kind == kind && k.prec == prec && (k.haswall != 0) == haswall && (!haswall || k.wall == wall) &&
        k.vec == w && k.rows == rows && k.threads == 64 * waves)
      return &k;
  }
  return nullptr;
}

const StepKernel *find_kernel(int prec, bool haswall, int wall, int kind, int vec, int rows, int fuse, bool sc) {
  int n = 0;
  const StepKernel *t = step_kernels(&n);
  for (int i = 0; i < n; ++i) {
    const StepKernel &k = t[i];
    if (k.prec != prec || k.kind != kind || (k.haswall != 0) != haswall || (k.sc != 0) != sc) continue;
    if (haswall && k.wall != wall) continue;
    if (kind == KIND_STRIP && (k.vec != vec || k.rows != rows || k.steps != fuse)) continue;
    return &k;
  }
  return nullptr;
}

static std::mutex g_tune_mu;
static std::map<std::tuple<int, int, int, int, int, int>, lbt1_kernel_config> g_tuned;

static std::tuple<int, int, int, int, int, int> tune_key(const lbt1_grid *g) {
  // multiphase grids tune separately (precision code offset by 8); the periodic
  // bits take part because a strip shape that fits a walled grid of odd width
  // does not fit one periodic in x
  return std::make_tuple(g->prec + (g->mp ? 8 : 0), (int)g->haswall, g->haswall ? g->wall : 0, (int)(g->periodic & 3u),
                         g->nx, g->ny);
}

// A strip configuration of 32 columns or more is a tile kernel's: vec columns and `rows`
// rows of the region, `waves` wavefronts of a block, `fuse` steps of a launch.
static bool is_tile(const lbt1_kernel_config &c) { return c.kernel == LBT1_KERNEL_STRIP && c.vec >= 32; }


// Tiles of configuration c on an nx x ny grid for a launch of `steps` steps: a halo
// of that many nodes (`reach` times as many) on each side of an axis, none on an axis that is not periodic and
// fits the region whole.  False when the halo leaves nothing to store, or when the launch would
// have 2^32 threads or more, which is past what a launch takes (the count wraps, without an
// error, and most tiles are not run: 65536 x 4100 nodes in regions of 32 x 32 at 12 steps).
bool tile_map(int nx, int ny, uint32_t periodic, const lbt1_kernel_config &c, int steps, TileMap *m, int reach) {
  m->steps = steps;
  const int halo = steps * reach, even = (halo + 1) / 2 * 2;  // chunks of two columns start at even columns
  m->hx = !(periodic & 1u) && nx <= c.vec ? 0 : c.vec > 64 ? even : halo;
  m->hy = !(periodic & 2u) && ny <= c.rows ? 0 : halo;
  m->ox = c.vec - 2 * m->hx;
  m->oy = c.rows - 2 * m->hy;
  if (m->ox < 1 || m->oy < 1) return false;
  m->tiles_x = (nx + m->ox - 1) / m->ox;
  m->tiles = m->tiles_x * ((ny + m->oy - 1) / m->oy);
  m->per_xcd = (m->tiles + 7) / 8;
  return 8ll * m->per_xcd * 64 * c.waves < 1ll << 32;
}
static bool is_tile_kind(const StepKernel *k) { return k->kind >= KIND_TILE; }
// nodes of a region's halo that a step of the kind uses up
static int reach_of(int kind) { return kind == KIND_SC_TILE ? 2 : 1; }
static dim3 tile_grid(const TileMap &m) { return dim3(8 * (unsigned)m.per_xcd, 1, 1); }

// Steps of a launch the choice is made over (and the autotuner's candidates).  Single-phase
// grids take four or more (three and fewer measured slower on each); a multiphase step
// uses up two nodes of the halo.
static const int kTileSteps[] = {2, 3, 4, 6, 8, 10, 12, 16, kMaxTileSteps};

// Modelled us per step of a tile kernel on `tiles` blocks: a launch takes us_launch and, for
// each block that falls to the busiest CU (past eight rounds the average: blocks end at
// different times), us_step per step and us_block.
double tile_us(const StepKernel &k, int steps, long tiles, int cus) {
  const double per_cu = (double)tiles / cus;
  const double rounds = per_cu <= 8 ? std::ceil(per_cu) : per_cu + 0.5;
  return (k.us_launch + rounds * (steps * k.us_step + k.us_block)) / steps;
}

// The tile kernel of a kind and the steps per launch with the least modelled time per
// step (tile_us), which goes to *us_out.  On 80 grids of 48^2 to 8192^2, periodic and cavities, FP64,
// FP32 and FP16S, what it picks is within 2 % of the fastest shape on average.
static lbt1_kernel_config tile_choice(int kind, int prec, bool haswall, int wall, int nx, int ny, uint32_t periodic, int cus,
                                      double *us_out) {
  lbt1_kernel_config best{};
  best.kernel = LBT1_KERNEL_GATHER;
  double best_us = 1e300;
  int n = 0;
  const StepKernel *t = step_kernels(&n);
  for (int i = 0; i < n; ++i) {
    const StepKernel &k = t[i];
    if (k.kind != kind || k.prec != prec || (k.haswall != 0) != haswall || (haswall && k.wall != wall)) continue;
    for (int steps : kTileSteps) {
      if (steps < 4 && kind != KIND_SC_TILE) continue;
      lbt1_kernel_config c{};
      c.kernel = LBT1_KERNEL_STRIP;
      c.vec = k.vec;
      c.rows = k.rows;
      c.waves = k.threads / 64;
      c.fuse = steps;
      TileMap m;
      if (!tile_map(nx, ny, periodic, c, steps, &m, reach_of(kind))) continue;
      const double us = tile_us(k, steps, m.tiles, cus);
      if (us < best_us) {
        best_us = us;
        best = c;
      }
    }
  }
  *us_out = best_us;
  return best;
}

// Default without a tuned entry: the tile kernel tile_choice finds.
//
// In FP32 and FP64 that beat every strip and gather kernel at each size (us per step,
// tile against the best of those: FP32 periodic 256^2 0.77 / 3.4, 1024^2 3.1 / 7.1,
// 4096^2 29.0 / 31.1, 8192^2 107 / 108.5; FP32 cavity 256^2 0.91 / 2.85, 1024^2 4.6 /
// 6.5, 8192^2 125 / 168; FP64 periodic 8192^2 224 / 302, cavity 274 / 540).  16-bit
// storage pays its codec once per step either way, and the strips exchange columns off
// the vector ALU: on large grids whose width they take, two-step strips of 14 rows are
// the faster (FP16S periodic 2700 x 2500 11.7 against 13.3, 4096^2 24.6 / 30.7, 8192^2
// 104.9 / 108.3, cavity 8192^2 116 / 133; but 2400 x 2200 11.7 / 10.6, cavity 2048^2 14.1 /
// 10.7), and strips of 6 rows where two or three rounds of them (eight wavefronts a CU) are
// what a periodic grid takes (BF16S 2048^2 8.55 / 9.21, FP16S 9.05 / 9.18).  Their times, in
// us, were fitted to grids of 1200^2 to 12288^2.
static lbt1_kernel_config default_config(int prec, bool haswall, int wall, int nx, int ny, uint32_t periodic, int cus) {
  double best_us;
  lbt1_kernel_config best = tile_choice(KIND_TILE, prec, haswall, wall, nx, ny, periodic, cus, &best_us);
  if ((prec != LBT1_F16S && prec != LBT1_BF16S) || !strip_fits(nx, 2, periodic & 1u)) return best;
  const double nodes = (double)nx * ny;
  const auto take = [&](int rows, double us) {
    if (us >= best_us || !find_kernel(prec, haswall, wall, KIND_STRIP, 2, rows, 2, false)) return;
    best_us = us;
    best = lbt1_kernel_config{};
    best.kernel = LBT1_KERNEL_STRIP;
    best.vec = 2;
    best.rows = rows;
    best.fuse = 2;
  };
  if (haswall) {
    take(14, 1.70e-6 * nodes + 5.0);
  } else {
    if (nodes >= 6e6) take(14, 1.47e-6 * nodes + 2.6);
    const long strips = (long)((chunks_of(nx, 2) + 61) / 62) * ((ny + 5) / 6), rounds = (strips + 8L * cus - 1) / (8L * cus);
    if (rounds == 2 || rounds == 3) take(6, 1.6 + (prec == LBT1_F16S ? 2.45 : 2.3) * rounds);
  }
  return best;
}

// Default without a tuned entry for a multiphase grid: the tile kernel too (us per step on
// drop fields, tile against the best of the strips: FP32 128^2 1.2 / 5.1, 1024^2 5.7 / 7.8,
// 4096^2 54.7 / 67; FP64 1024^2 8.3 / 12.1, 4096^2 100 / 149; with walls, where only the
// gather kernel applied, FP32 128^2 1.8 / 24.8, 1024^2 7.2 / 109).  16-bit storage on large
// periodic grids takes one-step strips of 14 rows (FP16S 4096^2 50.5 against 55; 2048^2 19.4
// against 17.1).
static lbt1_kernel_config sc_choice(int prec, bool haswall, int wall, int nx, int ny, uint32_t periodic, int cus) {
  double best_us;
  lbt1_kernel_config best = tile_choice(KIND_SC_TILE, prec, haswall, wall, nx, ny, periodic, cus, &best_us);
  if ((prec == LBT1_F16S || prec == LBT1_BF16S) && !haswall && nx % 2 == 0 && 2.85e-6 * nx * ny + 6.0 < best_us) {
    best = lbt1_kernel_config{};
    best.kernel = LBT1_KERNEL_STRIP;
    best.vec = 2;
    best.rows = 14;
    best.fuse = 1;
  }
  return best;
}

// Strips of vec columns per lane and `rows` rows of a grid, and their launch size.
static dim3 strip_launch(int nx, int ny, int vec, int rows, int waves, int cus, StripMap *map) {
  StripMap &m = *map;
  m.strips_x = (chunks_of(nx, vec) + 61) / 62;  // 62 chunks of vec columns per strip
  m.strips_y = (ny + rows - 1) / rows;
  const int strips = m.strips_x * m.strips_y;
  m.units = (strips + 3) / 4;
  int blocks;
  if (waves > 0) {
    // `waves` wavefronts per CU, 4 per block, a multiple of 8 blocks (one range per XCD)
    blocks = std::max(8, (cus * waves / 4) / 8 * 8);
    blocks = std::min(blocks, (m.units + 7) / 8 * 8);
    m.persistent = 1;
  } else {
    blocks = (m.units + 7) / 8 * 8;
    m.persistent = 0;
  }
  m.per_xcd = (m.units + 7) / 8;
  return dim3(blocks, 1, 1);
}

// Calls of up to three steps on periodic grids without walls, where the library chose a tile
// kernel: strips, one launch for all the steps.  A tile's rows do not start at cache lines, and
// few steps do not make up for it (us of a call, strips / tile): FP32 1024^2 one step 6.4 / 9.2,
// two 8.9 / 11.5; 8192^2 one 298 / 338, two 290 / 352, three 323 / 372; FP64 1024^2 one 9.5 /
// 12.4, two 12.8 / 15.5, 4096^2 155 / 164, 149 / 164; multiphase one step only, FP64 1024^2 11.8
// / 14.9.  Strips of 6 rows and 2 columns a lane are the fastest, or within 2 % of it, from about
// 700^2 nodes (16-bit storage 950^2; below, the tile kernel: FP32 512^2 two steps 5.8 / 5.9), of
// 4 columns from 12 million nodes in FP32 and, for one step, 20 million in 16-bit storage;
// three steps gain from 12 million nodes only.  With walls the tile kernel is the faster.
static void brief_strips(lbt1_grid *g, int cus) {
  const double nodes = (double)g->nx * g->ny;
  const bool half = g->prec == LBT1_F16S || g->prec == LBT1_BF16S, f32 = g->prec == LBT1_F32;
  if (g->haswall || nodes < (half ? 9e5 : 5e5)) return;
  for (int n = 1; n <= (g->mp ? 1 : kBrief); ++n) {
    const bool wide = !g->mp && nodes >= (half ? 2e7 : 1.2e7) && g->nx % 4 == 0 && (f32 || (half && n == 1));
    if (n == 3 && !(wide && f32)) continue;
    const int vec = wide ? 4 : 2, rows = n == 3 ? 14 : 6;
    const StepKernel *k = find_kernel(g->prec, false, 0, KIND_STRIP, vec, rows, n, g->mp);
    if (!k || !strip_fits(g->nx, vec, true)) continue;
    Brief &b = g->brief[n - 1];
    b.kern = k;
    b.times = 1;
    b.block = dim3(256, 1, 1);
    b.grid = strip_launch(g->nx, g->ny, vec, rows, 0, cus, &b.map);
  }
}

// The launch shape of a thread per node on population grids.
static dim3 push_grid(const lbt1_grid *g) {
  const int tiles = ((g->nx + 63) / 64) * ((g->ny + 3) / 4);
  return dim3((tiles + 7) / 8 * 8, 1, 1);
}

// Calls of one or two steps on population grids: k_bgk_step, a launch a step, where the tile
// kernel takes longer for so few (us of a call, k_bgk_step / k_bgk_tile: periodic FP32 64^2 one
// step 3.3 / 4.8, 512^2 one 4.4 / 9.2, two 9.0 / 11.3, three 13.3 / 13.0; 2048^2 one 55 / 70, two
// 110 / 68; FP64 cavity 384^2 one 7.5 / 11.0, two 14 / 12.5).  Periodic grids take it for every
// single step; otherwise its time is modelled as a launch and the bytes at the rate of the last
// cache level, lower with walls, whose flags are read for each neighbour, and two launches are
// not worth it on the smallest grids (FP64 64^2: 7.5 / 6.0).
static void brief_populations(lbt1_grid *g, int cus) {
  const double nodes = (double)g->nx * g->ny, bytes = nodes * 18 * value_bytes(g->prec);
  const double push = g->haswall ? 5.0 + (bytes + nodes) / 5e6 : 3.0 + bytes / 7e6;
  const dim3 grid = push_grid(g);
  if ((double)grid.x * 256 >= 4294967296.0) return;  // past what a launch takes
  for (int n = 1; n <= 2; ++n) {
    TileMap m;
    if (!tile_map(g->nx, g->ny, g->periodic, g->cfg, n, &m)) continue;
    const bool less = push < tile_us(*g->kern, n, m.tiles, cus) && (n == 1 || nodes >= 2e5);
    if (!less && (n > 1 || g->haswall)) continue;
    Brief &b = g->brief[n - 1];
    b.kern = find_kernel(g->prec, g->haswall, g->wall, KIND_BGK, 0, 0, 1, false);
    b.times = n;
    b.grid = grid;
    b.block = dim3(256, 1, 1);
  }
}

// Resolve a configuration into a kernel and launch shape for grid g.
lbt1_status bind_config(lbt1_grid *g, const lbt1_kernel_config &want, int cus) {
  for (Brief &b : g->brief) b = Brief{};
  if (g->pop) {
    g->kern2 = nullptr;
    g->graph_valid = false;
    if (!g->mp) {
      double us;
      g->cfg = tile_choice(KIND_BGK_TILE, g->prec, g->haswall, g->wall, g->nx, g->ny, g->periodic, cus, &us);
      const StepKernel *k =
          find_tile(KIND_BGK_TILE, g->prec, g->haswall, g->wall, g->cfg.vec, g->cfg.rows, g->cfg.waves);
      if (!k) return fail(LBT1_EINVAL, "no built population kernel at this precision");
      g->kern = g->kern1 = k;
      g->launch_steps = g->cfg.fuse;
      g->block = g->block1 = dim3(k->threads, 1, 1);
      brief_populations(g, cus);
      return LBT1_OK;
    }
    // multiphase: one step at a time, a thread per node (the gather launch shape)
    const StepKernel *k = find_kernel(g->prec, g->haswall, g->wall, KIND_BGK, 0, 0, 1, g->mp);
    if (!k) return fail(LBT1_EINVAL, "no built population kernel at this precision");
    g->kern = g->kern1 = k;
    g->launch_steps = 1;
    g->cfg = lbt1_kernel_config{};
    g->cfg.kernel = LBT1_KERNEL_GATHER;
    g->cfg.fuse = 1;
    g->block = g->block1 = dim3(256, 1, 1);
    g->grid = g->grid1 = push_grid(g);
    return LBT1_OK;
  }
  lbt1_kernel_config c = want;
  if (c.kernel == LBT1_KERNEL_AUTO) {
    lbt1_kernel_config tuned{};
    bool have = false;
    {
      std::lock_guard<std::mutex> lk(g_tune_mu);
      auto it = g_tuned.find(tune_key(g));
      if (it != g_tuned.end()) tuned = it->second, have = true;
    }
    // a tuned entry that does not bind this grid (it should always, being keyed on
    // everything bind_config checks) yields to the heuristic rather than failing
    if (have && bind_config(g, tuned, cus) == LBT1_OK) return LBT1_OK;
    if (have) clear_error();
    c = g->mp ? sc_choice(g->prec, g->haswall, g->wall, g->nx, g->ny, g->periodic, cus)
              : default_config(g->prec, g->haswall, g->wall, g->nx, g->ny, g->periodic, cus);
    if (is_tile(c)) brief_strips(g, cus);
  }
  const StepKernel *k = nullptr, *k1 = nullptr, *k2 = nullptr;
  if (c.kernel == LBT1_KERNEL_GATHER) {
    k = k1 = find_kernel(g->prec, g->haswall, g->wall, KIND_GATHER, 0, 0, 1, g->mp);
    k2 = nullptr;
    c.vec = c.rows = c.waves = 0;
    c.fuse = 1;
  } else if (c.kernel == LBT1_KERNEL_STRIP && !is_tile(c)) {
    if (!strip_fits(g->nx, c.vec, g->periodic & 1u))
      return fail(LBT1_EINVAL, "strip kernel: vec %d does not divide nx %d on a grid periodic in x", c.vec, g->nx);
    if ((long)chunks_of(g->nx, c.vec) * c.vec > g->L.pitch)
      return fail(LBT1_EINVAL, "strip kernel: vec %d chunks overrun the row pitch %d", c.vec, g->L.pitch);
    if (c.waves < 0 || c.waves > 32) return fail(LBT1_EINVAL, "waves %d out of range", c.waves);
    if (c.fuse == 0) c.fuse = 1;
    if (c.fuse < 1 || c.fuse > c.vec) return fail(LBT1_EINVAL, "fuse %d must be between 1 and vec %d", c.fuse, c.vec);
    if (c.fuse > 2 && g->haswall)
      return fail(LBT1_EINVAL, "three fused steps need a grid periodic in x and y without SOLID or FIXED nodes");
    if (c.fuse > 2 && g->mp) return fail(LBT1_EINVAL, "multiphase grids take one or two steps per launch");
    if (g->mp && g->haswall)
      return fail(LBT1_EINVAL, "multiphase strips need a grid periodic in x and y without SOLID nodes (use gather)");
    k = find_kernel(g->prec, g->haswall, g->wall, KIND_STRIP, c.vec, c.rows, c.fuse, g->mp);
    k1 = find_kernel(g->prec, g->haswall, g->wall, KIND_STRIP, c.vec, c.rows, 1, g->mp);
    // a fused shape with no single-step strip of its height finishes odd step
    // counts with the gather kernel (same arithmetic, own launch shape)
    if (k && !k1 && c.fuse > 1) k1 = find_kernel(g->prec, g->haswall, g->wall, KIND_GATHER, 0, 0, 1, g->mp);
    // three steps per launch: remainders of two steps take the two-step kernel of
    // the same strip shape where one is built
    if (c.fuse == 3) k2 = find_kernel(g->prec, g->haswall, g->wall, KIND_STRIP, c.vec, c.rows, 2, g->mp);
  } else if (is_tile(c)) {
    const int kind = g->mp ? KIND_SC_TILE : KIND_TILE;
    if (c.fuse < 1 || c.fuse > kMaxTileSteps)
      return fail(LBT1_EINVAL, "tile kernel: fuse %d must be between 1 and %d", c.fuse, kMaxTileSteps);
    k = k1 = find_tile(kind, g->prec, g->haswall, g->wall, c.vec, c.rows, c.waves);
    TileMap m;
    if (k && !tile_map(g->nx, g->ny, g->periodic, c, c.fuse, &m, reach_of(kind)))
      return fail(LBT1_EINVAL, "tile kernel: a halo of %d steps leaves too little of a %d x %d region", c.fuse, c.vec, c.rows);
  } else {
    return fail(LBT1_EINVAL, "unknown kernel family %d", c.kernel);
  }
  if (!k || !k1)
    return fail(LBT1_EINVAL, "no built kernel for vec %d rows %d fuse %d at this precision", c.vec, c.rows, c.fuse);
  g->kern = k;
  g->kern1 = k1;
  g->kern2 = k2;
  g->cfg = c;
  g->launch_steps = is_tile_kind(k) ? c.fuse : k->steps;
  if (is_tile_kind(k)) {
    g->block = dim3(k->threads, 1, 1);  // (its grid depends on the steps of a launch)
  } else if (k->kind == KIND_GATHER) {
    g->block = dim3(64, 4, 1);
    g->grid = dim3((g->nx + 63) / 64, (g->ny + 3) / 4, 1);
  } else {
    g->block = dim3(256, 1, 1);
    g->grid = strip_launch(g->nx, g->ny, c.vec, c.rows, c.waves, cus, &g->map);
  }
  g->block1 = g->block;
  g->grid1 = g->grid;
  if (k1->kind == KIND_GATHER && k->kind != KIND_GATHER) {
    g->block1 = dim3(64, 4, 1);
    g->grid1 = dim3((g->nx + 63) / 64, (g->ny + 3) / 4, 1);
  }
  g->graph_valid = false;
  return LBT1_OK;
}

StepArgs step_args(const lbt1_grid *g, int src_parity) {
  StepArgs a{};
  for (int q = 0; q < 3; ++q) {
    a.src[q] = g->plane[src_parity][q];
    a.dst[q] = g->plane[1 - src_parity][q];
  }
  a.flags = g->haswall ? g->flags : nullptr;
  a.nx = g->nx;
  a.ny = g->ny;
  a.pitch = g->L.pitch;
  a.rs = g->L.rs;
  a.periodic = g->periodic;
  a.fx = g->F[0];
  a.fy = g->F[1];
  a.sc_d = g->sc[0];
  a.sc_j = g->sc[1];
  a.is_d = 1.0 / g->sc[0];
  a.is_j = 1.0 / g->sc[1];
  a.trash = g->base + g->L.trash_off;
  a.sc_G = g->sc_G;
  a.sc_rho0 = g->sc_rho0;
  return a;
}

BgkArgs bgk_args(const lbt1_grid *g, int src_parity) {
  BgkArgs a{};
  for (int q = 0; q < 9; ++q) {
    a.src[q] = g->plane[src_parity][q];
    a.dst[q] = g->plane[1 - src_parity][q];
  }
  a.flags = g->haswall ? g->flags : nullptr;
  a.nx = g->nx;
  a.ny = g->ny;
  a.pitch = g->L.pitch;
  a.rs = g->L.rs;
  a.periodic = g->periodic;
  a.fx = g->tau * g->F[0];
  a.fy = g->tau * g->F[1];
  a.omega = 1.0 / g->tau;
  a.sc = g->sc[0];
  a.is = 1.0 / g->sc[0];
  a.tiles_x = (g->nx + 63) / 64;
  a.tiles = a.tiles_x * ((g->ny + 3) / 4);
  a.per_xcd = (a.tiles + 7) / 8;
  a.psi = g->psi;
  a.sc_G = g->sc_G;
  a.sc_rho0 = g->sc_rho0;
  a.tau = g->tau;
  a.bfx = g->F[0];
  a.bfy = g->F[1];
  return a;
}

// One launch of kernel k (g->kern, or its single-step companion g->kern1,
// which has the same launch shape) reading parity src_parity; a tile kernel takes
// `steps` steps.
hipError_t launch_step(lbt1_grid *g, const StepKernel *k, int src_parity, hipStream_t s, int steps = 1) {
  if (k->kind == KIND_BGK) {
    BgkArgs b = bgk_args(g, src_parity);
    void *args[] = {&b};
    hipError_t e = hipLaunchKernel(bgk_psi_kernel(g->prec), g->grid, g->block, args, 0, s);
    if (e != hipSuccess) return e;
    return hipLaunchKernel(k->fn, g->grid, g->block, args, 0, s);
  }
  if (is_tile_kind(k)) {
    TileMap t;
    if (!tile_map(g->nx, g->ny, g->periodic, g->cfg, steps, &t, reach_of(k->kind))) return hipErrorInvalidValue;
    StepArgs a{};
    BgkArgs b{};
    if (g->pop)
      b = bgk_args(g, src_parity);
    else
      a = step_args(g, src_parity);
    void *args[] = {g->pop ? (void *)&b : (void *)&a, &t};
    return hipLaunchKernel(k->fn, tile_grid(t), g->block, args, 0, s);
  }
  StepArgs a = step_args(g, src_parity);
  if (k->kind == KIND_GATHER) {
    void *args[] = {&a};
    const bool companion = k == g->kern1 && k != g->kern;
    return hipLaunchKernel(k->fn, companion ? g->grid1 : g->grid, companion ? g->block1 : g->block, args, 0, s);
  }
  StripMap m = g->map;
  void *args[] = {&a, &m};
  return hipLaunchKernel(k->fn, g->grid, g->block, args, 0, s);
}

// A call of n <= kBrief steps as g->brief has it.
static hipError_t launch_brief(lbt1_grid *g, int n, hipStream_t s) {
  const Brief &b = g->brief[n - 1];
  for (int k = 0; k < b.times; ++k) {
    StepArgs a{};
    BgkArgs p{};
    StripMap m = b.map;
    if (g->pop)
      p = bgk_args(g, g->parity);
    else
      a = step_args(g, g->parity);
    void *args[] = {g->pop ? (void *)&p : (void *)&a, &m};
    const hipError_t e = hipLaunchKernel(b.kern->fn, b.grid, b.block, args, 0, s);
    if (e != hipSuccess) return e;
    g->parity ^= 1;
    g->steps += n / b.times;
  }
  return hipSuccess;
}

// A graph of kBurst / K launches (K = g->kern->steps) starting from parity p:
// it advances burst_steps(g) steps and flips the parity once per launch.
static const int kBurst = 64;

static int burst_launches(const lbt1_grid *g) { return kBurst / g->launch_steps; }
static int burst_steps(const lbt1_grid *g) { return burst_launches(g) * g->launch_steps; }

static lbt1_status build_burst(lbt1_grid *g, int p) {
  hipGraph_t graph = nullptr;
  hipError_t e = hipGraphCreate(&graph, 0);
  if (e != hipSuccess) return hip_fail(e, "hipGraphCreate");
  hipGraphNode_t prev = nullptr;
  const int launches = burst_launches(g);
  std::vector<StepArgs> argv(launches);
  std::vector<BgkArgs> bargv(g->pop ? launches : 0);
  StripMap m = g->map;
  TileMap tm{};
  if (is_tile_kind(g->kern) && !tile_map(g->nx, g->ny, g->periodic, g->cfg, g->launch_steps, &tm, reach_of(g->kern->kind))) {
    hipGraphDestroy(graph);
    return fail(LBT1_EINVAL, "no tiles");
  }
  for (int s = 0; s < launches; ++s) {
    argv[s] = step_args(g, (p + s) & 1);
    if (g->pop) bargv[s] = bgk_args(g, (p + s) & 1);
    void *args_gather[] = {g->pop ? (void *)&bargv[s] : (void *)&argv[s]};
    void *args_strip[] = {&argv[s], &m};
    void *args_tile[] = {args_gather[0], &tm};
    hipKernelNodeParams kp{};
    kp.func = const_cast<void *>(g->kern->fn);
    kp.gridDim = is_tile_kind(g->kern) ? tile_grid(tm) : g->grid;
    kp.blockDim = g->block;
    kp.sharedMemBytes = 0;
    kp.kernelParams = g->kern->kind == KIND_STRIP ? args_strip : is_tile_kind(g->kern) ? args_tile : args_gather;
    kp.extra = nullptr;
    hipGraphNode_t node;
    if (g->pop && g->mp) {
      // multiphase population grids: the psi pass before each step
      hipKernelNodeParams pp = kp;
      pp.func = const_cast<void *>(bgk_psi_kernel(g->prec));
      e = hipGraphAddKernelNode(&node, graph, prev ? &prev : nullptr, prev ? 1 : 0, &pp);
      if (e != hipSuccess) {
        hipGraphDestroy(graph);
        return hip_fail(e, "hipGraphAddKernelNode");
      }
      prev = node;
    }
    e = hipGraphAddKernelNode(&node, graph, prev ? &prev : nullptr, prev ? 1 : 0, &kp);
    if (e != hipSuccess) {
      hipGraphDestroy(graph);
      return hip_fail(e, "hipGraphAddKernelNode");
    }
    prev = node;
  }
  if (g->burst[p]) hipGraphExecDestroy(g->burst[p]);
  g->burst[p] = nullptr;
  e = hipGraphInstantiate(&g->burst[p], graph, nullptr, nullptr, 0);
  hipGraphDestroy(graph);
  if (e != hipSuccess) return hip_fail(e, "hipGraphInstantiate");
  return LBT1_OK;
}

static void drop_bursts(lbt1_grid *g) {
  for (int p = 0; p < 2; ++p)
    if (g->burst[p]) {
      hipGraphExecDestroy(g->burst[p]);
      g->burst[p] = nullptr;
    }
  g->graph_valid = false;
}

lbt1_status enqueue_steps(lbt1_grid *g, int64_t n, hipStream_t s, bool use_graph) {
  hipError_t e;
  const int bs = burst_steps(g);
  // Recorded by a caller into a graph, tile launches are plain ones and even in number where
  // there are two steps or more: every replay then reads the parity that the one before it
  // wrote, as it does with single-step launches of an even number of steps.
  bool recorded = false;
  if (is_tile_kind(g->kern)) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    recorded = hipStreamIsCapturing(s, &st) == hipSuccess && st == hipStreamCaptureStatusActive;
  }
  if (use_graph && n >= kBurst && !recorded) {
    if (!g->graph_valid) {
      drop_bursts(g);
      g->graph_valid = true;
    }
    while (n >= bs) {
      const int p = g->parity;
      if (!g->burst[p]) {
        lbt1_status st = build_burst(g, p);
        if (st) return st;
      }
      if ((e = hipGraphLaunch(g->burst[p], s)) != hipSuccess) return hip_fail(e, "hipGraphLaunch");
      n -= bs;
      g->steps += bs;
      g->parity ^= burst_launches(g) & 1;
    }
  }
  const int K = g->launch_steps;
  if (n >= 1 && n <= kBrief && g->brief[n - 1].kern && !(recorded && n > 1 && g->brief[n - 1].times & 1)) {
    if ((e = launch_brief(g, (int)n, s)) != hipSuccess) return hip_fail(e, "step launch");
    return LBT1_OK;
  }
  if (is_tile_kind(g->kern)) {
    // Any number of steps up to K in a launch: as few launches as K allows, with the steps
    // spread over them.  A last launch of the few steps left over would move the state for
    // them alone (8192^2 FP32, 99 steps and a reduction: 10.99 ms, 10.63 spread).
    int64_t launches = (n + K - 1) / K;
    if (recorded && n > 1) launches += launches & 1;
    for (; n > 0; --launches) {
      const int k = (int)((n + launches - 1) / launches);
      if ((e = launch_step(g, g->kern, g->parity, s, k)) != hipSuccess) return hip_fail(e, "step launch");
      g->parity ^= 1;
      g->steps += k;
      n -= k;
    }
    return LBT1_OK;
  }
  // With a two-step companion the remainder after three-step launches is covered
  // by two-step launches: one for 2 left, two for 1 left when the single-step
  // companion is the (slower) gather kernel and at least 4 steps are asked for.
  int64_t tail2 = 0;
  if (g->kern2) {
    if (n % K == 2) tail2 = 1;
    if (n % K == 1 && n >= 4 && g->kern1->kind == KIND_GATHER) tail2 = 2;
  }
  for (; n - 2 * tail2 >= K; n -= K) {
    if ((e = launch_step(g, g->kern, g->parity, s)) != hipSuccess) return hip_fail(e, "step launch");
    g->parity ^= 1;
    g->steps += K;
  }
  for (; tail2 > 0; --tail2, n -= 2) {
    if ((e = launch_step(g, g->kern2, g->parity, s)) != hipSuccess) return hip_fail(e, "step launch");
    g->parity ^= 1;
    g->steps += 2;
  }
  for (; n > 0; --n) {
    if ((e = launch_step(g, g->kern1, g->parity, s)) != hipSuccess) return hip_fail(e, "step launch");
    g->parity ^= 1;
    g->steps += 1;
  }
  return LBT1_OK;
}

// Number of partial rows (reduction blocks) the partial pass of grid g writes.
static int reduce_blocks(const lbt1_grid *g) {
  const long n = (long)g->nx * g->ny;
  return (int)std::min<long>(g->L.nparts, std::max<long>(1, (n + 1023) / 1024));
}

// The two reduction passes of grid g on stream s: block partials into
// `partials` (reduce_blocks(g) rows of six doubles), then one wavefront combines
// them into `out`: the six raw slots, or with user_slots the slots as
// lbt1_reduce reports them (k_reduce_final_out).
static lbt1_status enqueue_reduce_into(lbt1_grid *g, uint32_t what, hipStream_t s, double *partials, double *out,
                                       bool user_slots) {
  const int blocks = reduce_blocks(g);
  hipError_t e;
  if (g->pop) {
    BgkReduceArgs a{};
    for (int q = 0; q < 9; ++q) a.cur[q] = g->plane[g->parity][q];
    for (int q = 0; q < 3; ++q) a.snap[q] = g->snap[q];
    a.flags = g->haswall ? g->flags : nullptr;
    a.nx = g->nx;
    a.ny = g->ny;
    a.pitch = g->L.pitch;
    a.rs = g->L.rs;
    a.snap_rs = g->L.snap_rs;
    a.sc = g->sc[0];
    a.sc_d = g->sc[0];
    a.sc_j = g->sc[1];
    a.is_d = 1.0 / g->sc[0];
    a.is_j = 1.0 / g->sc[1];
    a.what = what;
    a.partials = partials;
    void *args[] = {&a};
    e = hipLaunchKernel(bgk_reduce_partial_kernel(g->prec), dim3(blocks), dim3(256), args, 0, s);
  } else {
    ReduceArgs a{};
    for (int q = 0; q < 3; ++q) {
      a.cur[q] = g->plane[g->parity][q];
      a.snap[q] = g->snap[q];
    }
    a.flags = g->haswall ? g->flags : nullptr;
    a.nx = g->nx;
    a.ny = g->ny;
    a.pitch = g->L.pitch;
    a.rs = g->L.rs;
    a.sc_d = g->sc[0];
    a.sc_j = g->sc[1];
    a.what = what;
    a.partials = partials;
    void *args[] = {&a};
    e = hipLaunchKernel(reduce_partial_kernel(g->prec), dim3(blocks), dim3(256), args, 0, s);
  }
  if (e != hipSuccess) return hip_fail(e, "reduce launch");
  const double *parts = partials;
  int np = blocks;
  if (user_slots) {
    void *args2[] = {&parts, &np, &what, &out};
    e = hipLaunchKernel(reduce_final_out_kernel(), dim3(1), dim3(64), args2, 0, s);
  } else {
    void *args2[] = {&parts, &np, &out};
    e = hipLaunchKernel(reduce_final_kernel(), dim3(1), dim3(64), args2, 0, s);
  }
  if (e != hipSuccess) return hip_fail(e, "reduce launch");
  return LBT1_OK;
}

lbt1_status enqueue_reduce(lbt1_grid *g, uint32_t what, hipStream_t s) {
  return enqueue_reduce_into(g, what, s, g->partials, g->red_out, false);
}

// ----------------------------------------------------------------- allocation-free reduction
// Partial rows of lbt1_reduce_noalloc, in a file-scope device array instead of
// the grid's workspace: kReduceBlocks rows of six doubles (48 KiB on every
// device the library runs on, held until the process ends).  In host code the
// name `scratch` is only a stand-in for the symbol; its device address comes
// from hipGetSymbolAddress, once per device, and only that address is used.
constexpr int kScratchRows = kReduceBlocks;
static __device__ __align__(256) double scratch[kScratchRows * 6];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static double *g_scratch_ptr[kMaxDevices] = {};

// The address of `scratch` on device dev (which must be current).
static lbt1_status scratch_on(int dev, double **out) {
  if (dev < 0 || dev >= kMaxDevices) return fail(LBT1_EDEVICE, "device %d: at most %d devices", dev, kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!p) return fail(LBT1_EDEVICE, "hipGetSymbolAddress(scratch) returned no address");
    g_scratch_ptr[dev] = (double *)p;
  }
  *out = g_scratch_ptr[dev];
  return LBT1_OK;
}

// D2Q9 tables of section 2 for the host-side initialisation of population grids.
static const int kHostEx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
static const int kHostEy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
static const double kHostW[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};

// Populations of a stored-population grid at t = 0: the equilibrium
// (Eq. maxwellboltzmann, FP64) of each FLUID node's moments, that of the
// moments with the force shift tau F for FIXED nodes (what they send every
// step), w_q for SOLID nodes; stored as deviations f_q - w_q.
static lbt1_status set_geometry_pop(lbt1_grid *g, const uint8_t *flags, const double *rho, const double *jx,
                                    const double *jy) {
  const int nx = g->nx, ny = g->ny, pitch = g->L.pitch;
  const size_t c = value_bytes(g->prec);
  const size_t plane = (size_t)pitch * ny;
  std::vector<char> stage, sstage;
  std::vector<uint8_t> fstage;
  std::vector<double> rows;
  try {
    stage.assign(g->L.state, 0);
    fstage.assign(plane, LBT1_SOLID);
    if (g->snap[0]) sstage.assign(g->L.snap_field_off[2] + plane * c, 0);
    rows.assign((size_t)12 * nx, 0.0);
    g->given_idx.clear();
    g->given_val.clear();
  } catch (...) {
    return fail(LBT1_ENOMEM, "host staging");
  }
  double *mom = rows.data() + (size_t)9 * nx;  // rho - 1, jx, jy of one row
  for (int y = 0; y < ny; ++y) {
    for (int x = 0; x < nx; ++x) {
      const size_t i = (size_t)y * nx + x;
      const uint8_t fl = flags ? flags[i] : LBT1_FLUID;
      const double r = rho ? rho[i] : 1.0, a = jx ? jx[i] : 0.0, b = jy ? jy[i] : 0.0;
      if (fl != LBT1_FLUID) {
        g->given_idx.push_back(i);
        g->given_val.insert(g->given_val.end(), {r, a, b});
      }
      mom[x] = r - 1.0;
      mom[nx + x] = a;
      mom[2 * nx + x] = b;
      if (fl == LBT1_SOLID) {
        // zero-velocity equilibrium of the given density (never streamed; read by
        // the multiphase psi pass)
        for (int q = 0; q < 9; ++q) rows[(size_t)q * nx + x] = kHostW[q] * (r - 1.0);
        continue;
      }
      const double shift = fl == LBT1_FIXED ? g->tau : 0.0;
      const double ux = (a + shift * g->F[0]) / r, uy = (b + shift * g->F[1]) / r;
      const double usq = ux * ux + uy * uy;
      for (int q = 0; q < 9; ++q) {
        const double eu = kHostEx[q] * ux + kHostEy[q] * uy;
        rows[(size_t)q * nx + x] = kHostW[q] * r * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * usq) - kHostW[q];
      }
    }
    for (int q = 0; q < 9; ++q)
      encode_values(g->prec, rows.data() + (size_t)q * nx, nx, 1.0 / g->sc[0],
                    stage.data() + g->L.field_off[q] + (size_t)y * g->L.rs * c);
    if (g->snap[0])
      for (int q = 0; q < 3; ++q)
        encode_values(g->prec, mom + (size_t)q * nx, nx, 1.0 / g->sc[q == 0 ? 0 : 1],
                      sstage.data() + g->L.snap_field_off[q] + (size_t)y * g->L.snap_rs * c);
    for (int x = 0; x < nx; ++x) fstage[(size_t)y * pitch + x] = flags ? flags[(size_t)y * nx + x] : LBT1_FLUID;
  }
  hipError_t e;
  if ((e = hipSetDevice(g->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
  if ((e = hipStreamSynchronize(g->stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  if ((e = upload(g->base, stage.data(), g->L.state, {g->base + g->L.state}, g->stream)) != hipSuccess)
    return hip_fail(e, "hipMemcpy H2D");
  if (g->snap[0] && (e = hipMemcpy(g->base + g->L.snap_off, sstage.data(), sstage.size(), hipMemcpyHostToDevice)) != hipSuccess)
    return hip_fail(e, "hipMemcpy H2D");
  if ((e = hipMemcpy(g->flags, fstage.data(), plane, hipMemcpyHostToDevice)) != hipSuccess)
    return hip_fail(e, "hipMemcpy H2D");
  return LBT1_OK;
}

// The stored values of the fields (bits) of the current parity in rows y0 .. y0+h-1, columns
// x0 .. x0+w-1: take(q, y, row) for each field and row, once the stream is done.
template <typename F>
static lbt1_status read_fields(lbt1_grid *g, uint32_t fields, int x0, int y0, int w, int h, const F &take) {
  const size_t c = value_bytes(g->prec);
  hipError_t e;
  if ((e = hipSetDevice(g->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
  if ((e = hipStreamSynchronize(g->stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  RowSource s{};
  s.src = (const char *)g->plane[g->parity][0] + ((size_t)y0 * g->L.rs + x0) * c;
  s.c = c;
  s.stride = g->L.rs;
  s.field = (g->L.field_off[1] - g->L.field_off[0]) / c;
  s.scratch = g->partials;
  s.scratch_bytes = (size_t)g->L.nparts * 6 * sizeof(double);
  s.stream = g->stream;
  return read_rows(s, fields, w, h, take);
}

// Decode the populations of rows y0..y0+h-1, columns x0..x0+w-1 of the current
// parity into f[q][h][w] (deviations plus w_q).
static lbt1_status read_pop_window(lbt1_grid *g, int x0, int y0, int w, int h, std::vector<double> &f) {
  const size_t n = (size_t)w * h;
  try {
    f.resize(9 * n);
  } catch (...) {
    return fail(LBT1_ENOMEM, "host staging");
  }
  return read_fields(g, 0x1ffu, x0, y0, w, h, [&](int q, size_t y, const char *row) {
    double *dst = f.data() + (size_t)q * n + y * w;
    decode_values(g->prec, row, w, g->sc[0], dst);
    for (int x = 0; x < w; ++x) dst[x] += kHostW[q];
  });
}

}  // namespace lbt1

using namespace lbt1;

// =================================================================== C ABI
extern "C" {

const char *lbt1_last_error(void) { return g_err.c_str(); }

size_t lbt1_grid_bytes(int32_t nx, int32_t ny, int32_t prec, uint32_t options) {
  if (!valid_shape(nx, ny) || !valid_prec(prec)) return 0;
  return layout_of(nx, ny, prec, options).total;
}

lbt1_status lbt1_create_grid(const lbt1_grid_desc *d, lbt1_grid **out) {
  clear_error();
  if (!d || !out) return fail(LBT1_EINVAL, "null argument");
  *out = nullptr;
  if (!valid_shape(d->nx, d->ny)) return fail(LBT1_EINVAL, "grid %d x %d: each side must be 3..65536", d->nx, d->ny);
  if (!valid_prec(d->prec)) return fail(LBT1_EINVAL, "unknown precision %d", d->prec);
  if (d->wall != LBT1_WALL_PAPER && d->wall != LBT1_WALL_HALFWAY) return fail(LBT1_EINVAL, "unknown wall rule %d", d->wall);
  if (d->periodic & ~3u) return fail(LBT1_EINVAL, "periodic mask %u", d->periodic);
  if (d->options & ~(uint32_t)(LBT1_OPT_SNAPSHOT | LBT1_OPT_PLANAR | LBT1_OPT_POPULATIONS | LBT1_OPT_MULTIPHASE))
    return fail(LBT1_EINVAL, "unknown options %u", d->options);
  const bool sc = d->options & LBT1_OPT_MULTIPHASE;
  const double rho0 = d->sc_rho0 == 0.0 ? 1.0 : d->sc_rho0;
  if (sc && (!std::isfinite(d->sc_G) || !(rho0 > 0.0) || !std::isfinite(rho0)))
    return fail(LBT1_EINVAL, "multiphase: sc_G must be finite and sc_rho0 > 0");
  if (!sc && (d->sc_G != 0.0 || d->sc_rho0 != 0.0))
    return fail(LBT1_EINVAL, "sc_G / sc_rho0 given without LBT1_OPT_MULTIPHASE");
  const bool pop = d->options & LBT1_OPT_POPULATIONS;
  const double tau = d->tau == 0.0 ? 1.0 : d->tau;
  if (pop && !(tau > 0.5 && std::isfinite(tau))) return fail(LBT1_EINVAL, "tau = %g: must be finite and > 1/2", d->tau);
  if (!pop && tau != 1.0) return fail(LBT1_EINVAL, "tau = %g: LBMTau1 grids have tau = 1 (0 or 1)", d->tau);
  if (!std::isfinite(d->force[0]) || !std::isfinite(d->force[1])) return fail(LBT1_EINVAL, "force must be finite");
  if (!pow2_or_zero(d->scale[0]) || !pow2_or_zero(d->scale[1]))
    return fail(LBT1_EINVAL, "scales must be 0 or positive powers of two");
  int dev = 0, cus = 0;
  lbt1_status st = check_device(&dev, &cus);
  if (st) return st;
  lbt1_grid *g = new (std::nothrow) lbt1_grid();
  if (!g) return fail(LBT1_ENOMEM, "host allocation");
  g->device = dev;
  g->cus = cus;
  g->nx = d->nx;
  g->ny = d->ny;
  g->periodic = d->periodic;
  g->prec = d->prec;
  g->wall = d->wall;
  g->options = d->options;
  g->pop = pop;
  g->tau = tau;
  g->mp = sc;
  g->sc_G = sc ? d->sc_G : 0.0;
  g->sc_rho0 = rho0;
  g->F[0] = d->force[0];
  g->F[1] = d->force[1];
  const bool scaled = d->prec == LBT1_F16S || d->prec == LBT1_BF16S;
  g->sc[0] = (scaled && d->scale[0] != 0.0) ? d->scale[0] : 1.0;
  g->sc[1] = (scaled && d->scale[1] != 0.0) ? d->scale[1] : 1.0;
  g->L = layout_of(d->nx, d->ny, d->prec, d->options);
  hipError_t e;
  if (d->device_buffer) {
    if (d->device_bytes < g->L.total) {
      delete g;
      return fail(LBT1_ENOMEM, "device buffer has %zu bytes, grid needs %zu", d->device_bytes, g->L.total);
    }
    if (((uintptr_t)d->device_buffer) % 256) {
      delete g;
      return fail(LBT1_EINVAL, "device buffer must be 256-byte aligned");
    }
    g->base = (char *)d->device_buffer;
    g->own_mem = false;
  } else {
    void *p = nullptr;
    if ((e = hipMalloc(&p, g->L.total)) != hipSuccess) {
      delete g;
      return fail(LBT1_ENOMEM, "hipMalloc(%zu): %s", g->L.total, hipGetErrorString(e));
    }
    g->base = (char *)p;
    g->own_mem = true;
  }
  if (d->stream) {
    g->stream = (hipStream_t)d->stream;
    g->own_stream = false;
  } else {
    if ((e = hipStreamCreateWithFlags(&g->stream, hipStreamNonBlocking)) != hipSuccess) {
      if (g->own_mem) hipFree(g->base);
      delete g;
      return hip_fail(e, "hipStreamCreate");
    }
    g->own_stream = true;
  }
  for (int p = 0; p < 2; ++p)
    for (int q = 0; q < g->L.nfield; ++q) g->plane[p][q] = g->base + (size_t)p * g->L.state + g->L.field_off[q];
  g->flags = (uint8_t *)(g->base + g->L.flags_off);
  for (int q = 0; q < 3; ++q)
    g->snap[q] = (d->options & LBT1_OPT_SNAPSHOT) ? g->base + g->L.snap_off + g->L.snap_field_off[q] : nullptr;
  g->psi = g->L.psi_off ? g->base + g->L.psi_off : nullptr;
  g->partials = (double *)(g->base + g->L.part_off);
  g->red_out = (double *)(g->base + g->L.out_off);
  if ((e = hipHostMalloc((void **)&g->red_host, 8 * sizeof(double), hipHostMallocDefault)) != hipSuccess) {
    if (g->own_stream) hipStreamDestroy(g->stream);
    if (g->own_mem) hipFree(g->base);
    delete g;
    return hip_fail(e, "hipHostMalloc");
  }
  g->cfg.kernel = LBT1_KERNEL_AUTO;
  *out = g;
  return LBT1_OK;
}

lbt1_status lbt1_set_geometry(lbt1_grid *g, const uint8_t *flags, const double *rho, const double *jx,
                              const double *jy) {
  clear_error();
  if (!g) return fail(LBT1_EINVAL, "null grid");
  if (g->batch) return fail(LBT1_ESTATE, "grid is resident in a batch");
  const int nx = g->nx, ny = g->ny, pitch = g->L.pitch;
  const size_t n = (size_t)nx * ny;
  bool any_fixed = false, any_nonfluid = false;
  int64_t fluid = 0;
  if (flags) {
    for (size_t i = 0; i < n; ++i) {
      const uint8_t f = flags[i];
      if (f > LBT1_FIXED) return fail(LBT1_EINVAL, "flag %u at node %zu is not FLUID/SOLID/FIXED", f, i);
      any_fixed |= f == LBT1_FIXED;
      any_nonfluid |= f != LBT1_FLUID;
      fluid += f == LBT1_FLUID;
    }
  } else {
    fluid = (int64_t)n;
  }
  if (any_fixed && !rho && !jx && !jy) return fail(LBT1_EINVAL, "FIXED nodes need moments");
  if (any_fixed && g->mp) return fail(LBT1_EINVAL, "multiphase grids have no FIXED nodes");
  for (size_t i = 0; rho && i < n; ++i)
    if (!(rho[i] > 0.0) || !std::isfinite(rho[i])) return fail(LBT1_EINVAL, "rho[%zu] = %g must be finite and > 0", i, rho[i]);
  for (size_t i = 0; jx && i < n; ++i)
    if (!std::isfinite(jx[i])) return fail(LBT1_EINVAL, "jx[%zu] is not finite", i);
  for (size_t i = 0; jy && i < n; ++i)
    if (!std::isfinite(jy[i])) return fail(LBT1_EINVAL, "jy[%zu] is not finite", i);

  if (g->pop) {
    lbt1_status st = set_geometry_pop(g, flags, rho, jx, jy);
    if (st) return st;
    g->haswall = any_nonfluid || g->periodic != 3u;
    g->fluid = fluid;
    g->parity = 0;
    g->steps = 0;
    g->geometry = true;
    drop_bursts(g);
    return bind_config(g, lbt1_kernel_config{}, g->cus);
  }
  // Host staging in storage format with padded rows.
  const size_t c = value_bytes(g->prec);
  const size_t plane_vals = (size_t)pitch * ny;
  std::vector<char> stage;
  std::vector<uint8_t> fstage;
  try {
    stage.assign(g->L.state, 0);
    fstage.assign(plane_vals, LBT1_SOLID);
  } catch (...) {
    return fail(LBT1_ENOMEM, "host staging");
  }
  std::vector<double> row(nx);
  for (int y = 0; y < ny; ++y) {
    for (int q = 0; q < 3; ++q) {
      const double *src = q == 0 ? rho : q == 1 ? jx : jy;
      for (int x = 0; x < nx; ++x) {
        const size_t i = (size_t)y * nx + x;
        row[x] = src ? (q == 0 ? src[i] - 1.0 : src[i]) : 0.0;
      }
      encode_values(g->prec, row.data(), nx, 1.0 / g->sc[q == 0 ? 0 : 1],
                    stage.data() + g->L.field_off[q] + (size_t)y * g->L.rs * c);
    }
    for (int x = 0; x < nx; ++x) fstage[(size_t)y * pitch + x] = flags ? flags[(size_t)y * nx + x] : LBT1_FLUID;
  }
  hipError_t e;
  if ((e = hipSetDevice(g->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
  if ((e = hipStreamSynchronize(g->stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  if ((e = upload(g->base, stage.data(), g->L.state, {g->base + g->L.state, g->snap[0] ? g->base + g->L.snap_off : nullptr},
                  g->stream)) != hipSuccess)
    return hip_fail(e, "hipMemcpy H2D");
  if ((e = hipMemcpy(g->flags, fstage.data(), plane_vals, hipMemcpyHostToDevice)) != hipSuccess)
    return hip_fail(e, "hipMemcpy H2D");
  g->haswall = any_nonfluid || g->periodic != 3u;
  g->fluid = fluid;
  g->parity = 0;
  g->steps = 0;
  g->geometry = true;
  drop_bursts(g);
  lbt1_kernel_config want{};
  if (g->user_cfg) want = g->cfg;
  lbt1_status st = bind_config(g, want, g->cus);
  if (st) return st;
  return LBT1_OK;
}

lbt1_status lbt1_step(lbt1_grid *g, int64_t n) {
  clear_error();
  if (!g) return fail(LBT1_EINVAL, "null grid");
  if (n < 0) return fail(LBT1_EINVAL, "negative step count");
  if (!g->geometry) return fail(LBT1_ESTATE, "lbt1_step before lbt1_set_geometry");
  if (g->batch) return fail(LBT1_ESTATE, "grid is resident in a batch");
  hipError_t e;
  if ((e = hipSetDevice(g->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
  return enqueue_steps(g, n, g->stream, true);
}

lbt1_status lbt1_sync(lbt1_grid *g) {
  clear_error();
  if (!g) return fail(LBT1_EINVAL, "null grid");
  hipError_t e = hipStreamSynchronize(g->stream);
  if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  return LBT1_OK;
}

lbt1_status lbt1_read_window(lbt1_grid *g, int32_t x0, int32_t y0, int32_t w, int32_t h, double *rho, double *jx,
                             double *jy) {
  clear_error();
  if (!g) return fail(LBT1_EINVAL, "null grid");
  if (!g->geometry) return fail(LBT1_ESTATE, "no geometry set");
  if (w <= 0 || h <= 0 || x0 < 0 || y0 < 0 || (int64_t)x0 + w > g->nx || (int64_t)y0 + h > g->ny)
    return fail(LBT1_EINVAL, "window (%d, %d) + %d x %d is not inside the %d x %d grid", x0, y0, w, h, g->nx, g->ny);
  const size_t n = (size_t)w * h;
  if (g->pop) {
    std::vector<double> f;
    lbt1_status st = read_pop_window(g, x0, y0, w, h, f);
    if (st) return st;
    for (size_t i = 0; i < n; ++i) {
      double v[9];
      for (int q = 0; q < 9; ++q) v[q] = f[(size_t)q * n + i] - kHostW[q];
      const double d = (((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]))) + v[8];
      if (rho) rho[i] = 1.0 + d;
      if (jx) jx[i] = ((v[1] - v[3]) + (v[5] - v[6])) + (v[8] - v[7]);
      if (jy) jy[i] = ((v[2] - v[4]) + (v[5] - v[7])) + (v[6] - v[8]);
    }
    for (size_t k = 0; k < g->given_idx.size(); ++k) {
      const int gy = (int)(g->given_idx[k] / g->nx), gx = (int)(g->given_idx[k] % g->nx);
      if (gx < x0 || gx >= x0 + w || gy < y0 || gy >= y0 + h) continue;
      const size_t i = (size_t)(gy - y0) * w + (gx - x0);
      if (rho) rho[i] = g->given_val[3 * k];
      if (jx) jx[i] = g->given_val[3 * k + 1];
      if (jy) jy[i] = g->given_val[3 * k + 2];
    }
    return LBT1_OK;
  }
  double *const dsts[3] = {rho, jx, jy};
  const uint32_t fields = (rho ? 1u : 0u) | (jx ? 2u : 0u) | (jy ? 4u : 0u);
  return read_fields(g, fields, x0, y0, w, h, [&](int q, size_t y, const char *row) {
    double *dst = dsts[q] + y * w;
    decode_values(g->prec, row, w, g->sc[q == 0 ? 0 : 1], dst);
    if (q == 0)
      for (int x = 0; x < w; ++x) dst[x] += 1.0;
  });
}

lbt1_status lbt1_read_moments(lbt1_grid *g, double *rho, double *jx, double *jy) {
  if (!g) {
    clear_error();
    return fail(LBT1_EINVAL, "null grid");
  }
  return lbt1_read_window(g, 0, 0, g->nx, g->ny, rho, jx, jy);
}

lbt1_status lbt1_read_populations(lbt1_grid *g, double *f) {
  clear_error();
  if (!g || !f) return fail(LBT1_EINVAL, "null argument");
  if (!g->pop) return fail(LBT1_EINVAL, "not a population grid (LBT1_OPT_POPULATIONS)");
  if (!g->geometry) return fail(LBT1_ESTATE, "no geometry set");
  std::vector<double> v;
  lbt1_status st = read_pop_window(g, 0, 0, g->nx, g->ny, v);
  if (st) return st;
  std::memcpy(f, v.data(), v.size() * sizeof(double));
  return LBT1_OK;
}

lbt1_status lbt1_reduce(lbt1_grid *g, uint32_t what, double *out) {
  clear_error();
  if (!g || !out) return fail(LBT1_EINVAL, "null argument");
  if (what & ~15u) return fail(LBT1_EINVAL, "unknown reduce bits %u", what);
  if (!g->geometry) return fail(LBT1_ESTATE, "no geometry set");
  if ((what & LBT1_REDUCE_RESIDUAL) && !g->snap[0]) return fail(LBT1_EINVAL, "grid was created without LBT1_OPT_SNAPSHOT");
  if (g->batch) return fail(LBT1_ESTATE, "grid is resident in a batch");
  hipError_t e;
  if ((e = hipSetDevice(g->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
  lbt1_status st = enqueue_reduce(g, what, g->stream);
  if (st) return st;
  if ((e = hipMemcpyAsync(g->red_host, g->red_out, 6 * sizeof(double), hipMemcpyDeviceToHost, g->stream)) != hipSuccess)
    return hip_fail(e, "hipMemcpyAsync D2H");
  if ((e = hipStreamSynchronize(g->stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  const double *r = g->red_host;
  if (what & LBT1_REDUCE_MASS) out[0] = r[5] + r[0];
  if (what & LBT1_REDUCE_MOMENTUM) {
    out[1] = r[1];
    out[2] = r[2];
  }
  if (what & LBT1_REDUCE_RESIDUAL) out[3] = r[3];
  if (what & LBT1_REDUCE_NONFINITE) out[4] = r[4];
  out[5] = r[5];
  return LBT1_OK;
}

lbt1_status lbt1_reduce_noalloc(lbt1_grid *g, uint32_t what, double *out) {
  clear_error();
  if (!g || !out) return fail(LBT1_EINVAL, "null argument");
  if (what & ~15u) return fail(LBT1_EINVAL, "unknown reduce bits %u", what);
  if (!g->geometry) return fail(LBT1_ESTATE, "no geometry set");
  if ((what & LBT1_REDUCE_RESIDUAL) && !g->snap[0]) return fail(LBT1_EINVAL, "grid was created without LBT1_OPT_SNAPSHOT");
  if (g->batch) return fail(LBT1_ESTATE, "grid is resident in a batch");
  const int rows = reduce_blocks(g);
  if (rows > kScratchRows)
    return fail(LBT1_EINVAL, "reduction needs %d partial rows, the static scratch holds %d", rows, kScratchRows);
  hipError_t e;
  if ((e = hipSetDevice(g->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
  double *parts = nullptr;
  lbt1_status st = scratch_on(g->device, &parts);
  if (st) return st;
  return enqueue_reduce_into(g, what, g->stream, parts, out, true);
}

// Bytes of an exact checkpoint: the parity block in storage format, and the
// residual snapshot when the grid keeps one.
static size_t snapshot_bytes(const lbt1_grid *g) {
  if (!g->snap[0]) return 0;
  return g->pop ? 3 * (g->L.snap_field_off[1] - g->L.snap_field_off[0]) : g->L.state;
}

size_t lbt1_state_bytes(lbt1_grid *g) {
  if (!g) return 0;
  return g->L.state + snapshot_bytes(g);
}

lbt1_status lbt1_save_state(lbt1_grid *g, void *host, size_t bytes) {
  clear_error();
  if (!g || !host) return fail(LBT1_EINVAL, "null argument");
  if (!g->geometry) return fail(LBT1_ESTATE, "no geometry set");
  if (g->batch) return fail(LBT1_ESTATE, "grid is resident in a batch");
  if (bytes < lbt1_state_bytes(g)) return fail(LBT1_EINVAL, "buffer has %zu bytes, the state %zu", bytes, lbt1_state_bytes(g));
  hipError_t e;
  if ((e = hipSetDevice(g->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
  if ((e = hipStreamSynchronize(g->stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  char *h = (char *)host;
  if ((e = hipMemcpy(h, g->base + (size_t)g->parity * g->L.state, g->L.state, hipMemcpyDeviceToHost)) != hipSuccess)
    return hip_fail(e, "hipMemcpy D2H");
  if (snapshot_bytes(g) &&
      (e = hipMemcpy(h + g->L.state, g->base + g->L.snap_off, snapshot_bytes(g), hipMemcpyDeviceToHost)) != hipSuccess)
    return hip_fail(e, "hipMemcpy D2H");
  return LBT1_OK;
}

lbt1_status lbt1_load_state(lbt1_grid *g, const void *host, size_t bytes) {
  clear_error();
  if (!g || !host) return fail(LBT1_EINVAL, "null argument");
  if (!g->geometry) return fail(LBT1_ESTATE, "set the geometry (flags) before loading a state");
  if (g->batch) return fail(LBT1_ESTATE, "grid is resident in a batch");
  if (bytes != lbt1_state_bytes(g)) return fail(LBT1_EINVAL, "state has %zu bytes, this grid takes %zu", bytes, lbt1_state_bytes(g));
  hipError_t e;
  if ((e = hipSetDevice(g->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
  if ((e = hipStreamSynchronize(g->stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  const char *h = (const char *)host;
  // both parities: non-FLUID nodes are read from either
  if ((e = upload(g->base, h, g->L.state, {g->base + g->L.state}, g->stream)) != hipSuccess)
    return hip_fail(e, "hipMemcpy H2D");
  if (snapshot_bytes(g) &&
      (e = hipMemcpy(g->base + g->L.snap_off, h + g->L.state, snapshot_bytes(g), hipMemcpyHostToDevice)) != hipSuccess)
    return hip_fail(e, "hipMemcpy H2D");
  g->parity = 0;
  return LBT1_OK;
}

lbt1_status lbt1_destroy_grid(lbt1_grid *g) {
  clear_error();
  if (!g) return LBT1_OK;
  if (g->batch) return fail(LBT1_ESTATE, "grid is resident in a batch; evict it first");
  hipSetDevice(g->device);
  hipStreamSynchronize(g->stream);
  drop_bursts(g);
  if (g->red_host) hipHostFree(g->red_host);
  if (g->own_stream) hipStreamDestroy(g->stream);
  if (g->own_mem) hipFree(g->base);
  delete g;
  return LBT1_OK;
}

lbt1_status lbt1_set_kernel(lbt1_grid *g, const lbt1_kernel_config *cfg) {
  clear_error();
  if (!g || !cfg) return fail(LBT1_EINVAL, "null argument");
  if (g->pop) return fail(LBT1_EINVAL, "population grids have a single step kernel");
  if (!g->geometry) {
    g->cfg = *cfg;
    g->user_cfg = cfg->kernel != LBT1_KERNEL_AUTO;
    return LBT1_OK;
  }
  lbt1_kernel_config old = g->cfg;
  const StepKernel *oldk = g->kern;
  lbt1_status st = bind_config(g, *cfg, g->cus);
  if (st) {
    g->cfg = old;
    g->kern = oldk;
    const std::string said = g_err;
    bind_config(g, g->user_cfg ? old : lbt1_kernel_config{}, g->cus);
    g_err = said;
    return st;
  }
  g->user_cfg = cfg->kernel != LBT1_KERNEL_AUTO;
  drop_bursts(g);
  return LBT1_OK;
}

lbt1_status lbt1_get_kernel(lbt1_grid *g, lbt1_kernel_config *cfg, char *name, size_t cap) {
  clear_error();
  if (!g) return fail(LBT1_EINVAL, "null grid");
  if (!g->kern) return fail(LBT1_ESTATE, "no kernel bound (set the geometry first)");
  if (cfg) *cfg = g->cfg;
  if (name && cap) {
    std::strncpy(name, g->kern->name, cap - 1);
    name[cap - 1] = 0;
  }
  return LBT1_OK;
}

lbt1_status lbt1_autotune(lbt1_grid *g, int32_t steps, int32_t reps, lbt1_kernel_config *best,
                          double *ms_per_step) {
  clear_error();
  if (!g) return fail(LBT1_EINVAL, "null grid");
  if (!g->geometry) return fail(LBT1_ESTATE, "no geometry set");
  if (g->batch) return fail(LBT1_ESTATE, "grid is resident in a batch");
  if (steps < 2 || reps < 1) return fail(LBT1_EINVAL, "steps >= 2 and reps >= 1 required");
  if (g->pop) return fail(LBT1_EINVAL, "population grids have a single step kernel");
  hipError_t e;
  if ((e = hipSetDevice(g->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
  if ((e = hipStreamSynchronize(g->stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  // The candidates run on the grid's own memory (a copy elsewhere can time
  // differently: measured up to 2.5 % between two allocations of one 8192^2
  // field); both parities are saved to scratch first and restored afterwards.
  lbt1_grid t = *g;
  t.burst[0] = t.burst[1] = nullptr;
  t.graph_valid = false;
  void *p = nullptr;
  if ((e = hipMalloc(&p, 2 * g->L.state)) != hipSuccess)
    return fail(LBT1_ENOMEM, "autotune scratch: %s", hipGetErrorString(e));
  if ((e = hipMemcpyAsync(p, g->base, 2 * g->L.state, hipMemcpyDeviceToDevice, g->stream)) != hipSuccess) {
    hipFree(p);
    return hip_fail(e, "autotune save");
  }
  hipEvent_t e0, e1;
  hipEventCreate(&e0);
  hipEventCreate(&e1);
  std::vector<lbt1_kernel_config> cands;
  {
    lbt1_kernel_config c{};
    c.kernel = LBT1_KERNEL_GATHER;
    cands.push_back(c);
  }
  const int vecs[] = {1, 2, 4, 8};
  const int rows[] = {2, 6, 14, 22, 28, 30};
  const int waves[] = {0, 8, 16};
  const int fuses[] = {1, 2, 3};
  for (int v : vecs)
    for (int r : rows)
      for (int w : waves)
        for (int f : fuses) {
          if (!strip_fits(g->nx, v, g->periodic & 1u)) continue;
          if (f > 2 && (g->mp || g->haswall)) continue;
          if (g->mp && g->haswall) continue;
          if (!find_kernel(g->prec, g->haswall, g->wall, KIND_STRIP, v, r, f, g->mp)) continue;
          if (64 * v > 2 * std::max(64, g->nx)) continue;
          lbt1_kernel_config c{};
          c.kernel = LBT1_KERNEL_STRIP;
          c.vec = v;
          c.rows = r;
          c.waves = w;
          c.fuse = f;
          cands.push_back(c);
        }
  {
    // tile kernels whose modelled time is within half of the least (the model is off by up to a
    // quarter; the others would be most of the time the tuning takes, 2.1 s of it at 8192^2 FP32)
    const int kind = g->mp ? KIND_SC_TILE : KIND_TILE;
    int nk = 0;
    const StepKernel *tk = step_kernels(&nk);
    double least = 0;
    (void)tile_choice(kind, g->prec, g->haswall, g->wall, g->nx, g->ny, g->periodic, g->cus, &least);
    for (int i = 0; i < nk; ++i) {
      if (tk[i].kind != kind || tk[i].prec != g->prec || (tk[i].haswall != 0) != g->haswall ||
          (g->haswall && tk[i].wall != g->wall))
        continue;
      for (int f : kTileSteps) {
        TileMap m;
        lbt1_kernel_config c{};
        c.kernel = LBT1_KERNEL_STRIP;
        c.vec = tk[i].vec;
        c.rows = tk[i].rows;
        c.waves = tk[i].threads / 64;
        c.fuse = f;
        if (tile_map(g->nx, g->ny, g->periodic, c, f, &m, reach_of(kind)) && tile_us(tk[i], f, m.tiles, g->cus) <= 1.5 * least)
          cands.push_back(c);
      }
    }
  }
  // a whole number of fused launches for every strip candidate; the tile kernels take
  // whole launches of their own, about as many steps
  steps = (steps + 5) / 6 * 6;
  lbt1_status st = LBT1_OK;
  auto time_steps = [&](const int n, const bool use_graph) -> double {
    hipEventRecord(e0, g->stream);
    st = enqueue_steps(&t, n, g->stream, use_graph);
    hipEventRecord(e1, g->stream);
    hipEventSynchronize(e1);
    float ms = 0;
    hipEventElapsedTime(&ms, e0, e1);
    return (double)ms / n;
  };
  // screening: every candidate, best of `reps` after one warm-up run
  std::vector<std::pair<double, lbt1_kernel_config>> timed;
  for (const auto &c : cands) {
    if (bind_config(&t, c, g->cus) != LBT1_OK) continue;
    double cbest = 1e300;
    const int whole = is_tile(t.cfg) ? std::max(steps / t.launch_steps, 1) * t.launch_steps : steps;
    for (int r = 0; r < reps + 1 && st == LBT1_OK; ++r) {
      const double ms = time_steps(whole, false);
      if (r > 0) cbest = std::min(cbest, ms);
    }
    if (st) break;
    timed.push_back({cbest, t.cfg});
  }
  // final: the candidates within 5 % of the fastest, re-timed as lbt1_step runs
  // them (graph bursts) on three bursts' worth of steps, in interleaved rounds so
  // that a drift of the clock between candidates does not decide; each round
  // first runs a candidate once untimed (it builds the bursts)
  double best_ms = 1e300;
  lbt1_kernel_config bc = g->cfg;
  if (!st && !timed.empty()) {
    std::stable_sort(timed.begin(), timed.end(),
                     [](const std::pair<double, lbt1_kernel_config> &a, const std::pair<double, lbt1_kernel_config> &b) {
                       return a.first < b.first;
                     });
    size_t nf = 1;
    while (nf < timed.size() && nf < 8 && timed[nf].first <= 1.05 * timed[0].first) ++nf;
    best_ms = timed[0].first;
    bc = timed[0].second;
    if (nf > 1) {
      std::vector<double> fbest(nf, 1e300);
      for (int r = 0; r < std::max(reps, 3) && !st; ++r)
        for (size_t i = 0; i < nf && !st; ++i) {
          if (bind_config(&t, timed[i].second, g->cus) != LBT1_OK) continue;
          const int n = is_tile(t.cfg) ? 3 * burst_steps(&t) : 3 * kBurst;
          (void)time_steps(n, true);
          if (st) break;
          const double ms = time_steps(n, true);
          fbest[i] = std::min(fbest[i], ms);
        }
      if (!st) {
        size_t bi = 0;
        for (size_t i = 1; i < nf; ++i)
          if (fbest[i] < fbest[bi]) bi = i;
        best_ms = fbest[bi];
        bc = timed[bi].second;
      }
    }
  }
  hipStreamSynchronize(g->stream);
  drop_bursts(&t);  // (the clone's bursts, idle now)
  const hipError_t er = hipMemcpyAsync(g->base, p, 2 * g->L.state, hipMemcpyDeviceToDevice, g->stream);
  hipStreamSynchronize(g->stream);
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  hipFree(p);
  if (st) return st;
  if (er != hipSuccess) return hip_fail(er, "autotune restore");
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned[tune_key(g)] = bc;
  }
  st = bind_config(g, bc, g->cus);
  if (st) return st;
  g->user_cfg = true;
  drop_bursts(g);
  if (best) *best = bc;
  if (ms_per_step) *ms_per_step = best_ms;
  return LBT1_OK;
}

}  // extern "C"
