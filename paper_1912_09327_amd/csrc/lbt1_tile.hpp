// Several LBMTau1 steps per launch on a region of nodes held in registers.
//
// A step of a grid of a few hundred nodes a side is bound by the latency of a launch
// (about 4 us from one kernel's start to the next one's) and of a strip's walk down
// its rows; larger grids in FP64 or with walls are bound by HBM at the two steps per
// pass the strip kernels take.  Here a block takes a region of W * CPL columns and
// THREADS / W * RPT rows: a thread keeps RPT rows of CPL adjacent columns in registers
// and advances them K steps before the block stores.  Columns are exchanged by lane
// shifts; the rows where two threads of a column meet go through LDS, one barrier a
// step.  The region is the stored tile widened by a halo of K nodes on every side that
// is not a grid edge the region reaches (nodes outside a non-periodic axis are SOLID).
// What lies outside the region is wrong, and the wrong part moves inwards one node per
// step, so after K steps the halo is used up and the tile is exact.
//
// Same emission, wall rule and order of sums as the single-step kernels, and a node
// passes through the storage codec between steps as a store and reload would, so K
// steps give the bits of K launches of the gather kernel.  Non-FLUID nodes are held in
// both parities and not written.  A region without walls takes a body that exchanges
// reduced row sums; the choice is one vote per block and launch.
//
// Small grids are bound by the launch (256^2 FP32 cavity: 7.2 us for 8 steps, 4 us of it
// the launch; 2.87 us per step before, 0.91 now), large ones by vector-ALU issue: the
// wall-free step is 46 vector instructions a node, and a 128 x 64 region at 6 steps
// stores 73 % of what it computes (8192^2 FP32: 398 million vector instructions in the
// 669 us of 6 steps, 97 % of the issue rate, and 1.82 GB, 2.7 TB/s; 4096^2: 28.8 us per
// step, against 34.2 with three-step strips, which wait for memory at two wavefronts
// per SIMD).
#pragma once
#include "lbt1_tile_args.hpp"
#include "lbt1_device.hpp"
#include "lbt1_step.hpp"

namespace lbt1 {

// LDS of a block: what its threads send to the row group below (rows 0-2) and above
// (rows 3-5).  FP32 arithmetic keeps two copies used in turn, so one barrier a step is
// enough; FP64 keeps one, with a second barrier, so that two blocks fit a CU.
template <typename C, int NODES>
struct TileShared {
  static constexpr int kCopies = sizeof(C) == 4 ? 2 : 1;
  C v[kCopies][6][NODES];
};

// all ones where bit b of w is set, else 0, and the choice between two values by such a
// mask: two vector operations for a select, and no condition held in scalar registers
__device__ __forceinline__ uint32_t spread(const uint32_t w, const int b) {
  return (uint32_t)((int32_t)(w << (31 - b)) >> 31);
}
__device__ __forceinline__ float pick(const uint32_t m, const float yes, const float no) {
  return __uint_as_float((__float_as_uint(yes) & m) | (__float_as_uint(no) & ~m));
}
__device__ __forceinline__ double pick(const uint32_t m, const double yes, const double no) {
  const uint64_t a = (uint64_t)__double_as_longlong(yes), b = (uint64_t)__double_as_longlong(no);
  const uint32_t lo = ((uint32_t)a & m) | ((uint32_t)b & ~m), hi = ((uint32_t)(a >> 32) & m) | ((uint32_t)(b >> 32) & ~m);
  return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Lattice column and row of every node of a thread at (x, y0), -1 outside a non-periodic
// axis (one division per axis: the following ones step and wrap).
template <int CPL, int RPT>
struct TilePlace {
  int wx[CPL], wy[RPT];
  __device__ __forceinline__ TilePlace(const int x, const int y0, const int nx, const int ny, const bool px,
                                       const bool py) {
    wx[0] = wrap_axis(x, nx, px);
#pragma unroll
    for (int c = 1; c < CPL; ++c) {
      const int n = wx[c - 1] + 1;
      wx[c] = px ? (n == nx ? 0 : n) : (x + c >= 0 && x + c < nx ? x + c : -1);
    }
    wy[0] = wrap_axis(y0, ny, py);
#pragma unroll
    for (int i = 1; i < RPT; ++i) {
      const int n = wy[i - 1] + 1;
      wy[i] = py ? (n == ny ? 0 : n) : (y0 + i >= 0 && y0 + i < ny ? y0 + i : -1);
    }
  }
};

// Flags of a thread's nodes: a FLUID bit per node (node i * CPL + c), and per row of the
// thread (solid[1 + i]) a SOLID bit per column (bit c + 1).  Outside the grid SOLID.
template <int CPL, int RPT>
__device__ __forceinline__ void tile_flags(const uint8_t *flags, const int pitch, const TilePlace<CPL, RPT> &at,
                                           uint32_t (&solid)[RPT + 2], uint32_t &fluid) {
  fluid = 0;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    uint32_t sb = 0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const bool in = at.wy[i] >= 0 && at.wx[c] >= 0;
      const uint8_t f = flags[(long)max(at.wy[i], 0) * pitch + max(at.wx[c], 0)];
      sb |= (uint32_t)(!in || f == NODE_SOLID) << (c + 1);
      fluid |= (uint32_t)(in && f == NODE_FLUID) << (i * CPL + c);
    }
    solid[i + 1] = sb;
  }
}

// Eight bits per node, bit q - 1 set where its source along e_q is a wall, from the SOLID
// bits of the thread and of the threads next to it (through `bits`, 2 * THREADS words of
// LDS); outside the region SOLID (a grid edge, or the halo).
template <int W, int CPL, int RPT, int THREADS>
__device__ __forceinline__ void tile_walls(uint32_t (&solid)[RPT + 2], uint32_t *bits,
                                           uint32_t (&from_wall)[(RPT * CPL + 3) / 4]) {
  const int lane = threadIdx.x & (W - 1), grp = threadIdx.x / W;
#pragma unroll
  for (int i = 1; i <= RPT; ++i) {
    const uint32_t lw = (uint32_t)dpp_shift<kDppWaveShr1>((int)(solid[i] >> CPL & 1u));
    const uint32_t rw = (uint32_t)dpp_shift<kDppWaveShl1>((int)(solid[i] >> 1 & 1u));
    solid[i] |= (lane == 0 ? 1u : lw) | (lane == W - 1 ? 1u : rw) << (CPL + 1);
  }
  bits[threadIdx.x] = solid[1];
  bits[THREADS + threadIdx.x] = solid[RPT];
  __syncthreads();
  solid[0] = grp > 0 ? bits[THREADS + threadIdx.x - W] : 0xffffffffu;
  solid[RPT + 1] = grp < THREADS / W - 1 ? bits[threadIdx.x + W] : 0xffffffffu;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < (RPT * CPL + 3) / 4; ++k) from_wall[k] = 0;
#pragma unroll
  for (int i = 0; i < RPT; ++i)
#pragma unroll
    for (int c = 0; c < CPL; ++c)
#pragma unroll
      for (int q = 1; q < 9; ++q) {
        const int node = i * CPL + c;
        from_wall[node / 4] |= (solid[i + 1 - kEy[q]] >> (c + 1 - kEx[q]) & 1u) << (node % 4 * 8 + q - 1);
      }
}

// The tile of a block: block b runs on XCD b % 8, and each XCD takes a contiguous range of
// tiles along the rows, so the halos that neighbouring tiles share meet in one L2.
__device__ __forceinline__ int tile_of(const TileMap &m) {
  return (int)(blockIdx.x & 7) * m.per_xcd + (int)(blockIdx.x >> 3);
}

template <int P, int WALL, int W, int CPL, int RPT, int THREADS, bool UNIT, bool CONDS>
struct TileRegion {
  using T = Traits<P>;
  using C = typename T::C;
  using S = typename T::S;
  using SP = Pack<S, CPL>;
  using CP = Pack<C, CPL>;
  static constexpr int GROUPS = THREADS / W;
  static constexpr int NODES = GROUPS * W * CPL;
  using Shared = TileShared<C, NODES>;

  C d[RPT][CPL], jx[RPT][CPL], jy[RPT][CPL];
  C Fx, Fy, sd, sj, ed, ej;
  int at, above, below;  // LDS index of this thread's columns in its own group and the groups next to it

  __device__ __forceinline__ void codec(C &v0, C &v1, C &v2) const {
    if constexpr (T::kScaled) {
      v0 = UNIT ? T::dec(T::enc(v0)) : T::dec(T::enc(v0 * ed)) * sd;
      v1 = UNIT ? T::dec(T::enc(v1)) : T::dec(T::enc(v1 * ej)) * sj;
      v2 = UNIT ? T::dec(T::enc(v2)) : T::dec(T::enc(v2 * ej)) * sj;
    }
  }
  static __device__ __forceinline__ void put(C *p, const C (&v)[CPL]) {
    CP o;
#pragma unroll
    for (int c = 0; c < CPL; ++c) o.v[c] = v[c];
    *reinterpret_cast<CP *>(p) = o;
  }
  static __device__ __forceinline__ void get(const C *p, C (&v)[CPL]) {
    const CP o = *reinterpret_cast<const CP *>(p);
#pragma unroll
    for (int c = 0; c < CPL; ++c) v[c] = o.v[c];
  }

  // What the nodes of source row i send, in the columns it arrives in: g[q] of column c
  // travelled along e_q (into the row below for q = 5, 2, 6, above for 8, 4, 7); f: as sent.
  __device__ __forceinline__ void arrivals(const int i, C (&f)[CPL][9], C (&g)[CPL][9]) const {
#pragma unroll
    for (int c = 0; c < CPL; ++c) emit<C>(d[i][c], jx[i][c], jy[i][c], Fx, Fy, f[c]);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      if (kEx[q] == 0) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) g[c][q] = f[c][q];
      } else if (kEx[q] == 1) {
        g[0][q] = dpp_shift<kDppWaveShr1>(f[CPL - 1][q]);
#pragma unroll
        for (int c = 1; c < CPL; ++c) g[c][q] = f[c - 1][q];
      } else {
        g[CPL - 1][q] = dpp_shift<kDppWaveShl1>(f[0][q]);
#pragma unroll
        for (int c = 0; c < CPL - 1; ++c) g[c][q] = f[c + 1][q];
      }
    }
  }

  // One walk down the thread's rows per step.  A target row is complete when the row
  // after it has been walked; the first and the last wait for the neighbouring groups,
  // whose sums (without walls) or arrivals (with walls) come through LDS.
  __device__ __forceinline__ void march(Shared &sh, const int steps) {
    for (int s = 0; s < steps; ++s) {
      C(*const e)[NODES] = sh.v[s % Shared::kCopies];
      C l0[CPL], x0[CPL], w0[CPL], v0[CPL];      // target row 0: level sums, sums of row 1
      C ps[CPL], px[CPL], pu[CPL];               // pending target: up + level sums, up sum alone
      C us[CPL], ux[CPL];                        // up sums of the newest row
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        if (T::kScaled && s > 0) {
#pragma unroll
          for (int c = 0; c < CPL; ++c) codec(d[i][c], jx[i][c], jy[i][c]);
        }
        C f[CPL][9], g[CPL][9], ws[CPL], wx[CPL];
        arrivals(i, f, g);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          ws[c] = row_sum(g[c][8], g[c][4], g[c][7]);
          wx[c] = row_dif(g[c][8], g[c][7]);
          if (i == 1) {
            w0[c] = ws[c];
            v0[c] = wx[c];
          }
          if (i > 1) {
            d[i - 1][c] = ps[c] + ws[c];
            jx[i - 1][c] = px[c] + wx[c];
            jy[i - 1][c] = pu[c] - ws[c];
          }
          const C ls = row_sum(g[c][1], g[c][0], g[c][3]), lx = row_dif(g[c][1], g[c][3]);
          if (i == 0) {
            l0[c] = ls;
            x0[c] = lx;
          } else {
            ps[c] = us[c] + ls;
            px[c] = ux[c] + lx;
            pu[c] = us[c];
          }
          us[c] = row_sum(g[c][5], g[c][2], g[c][6]);
          ux[c] = row_dif(g[c][5], g[c][6]);
        }
        if (i == 0) {
          put(&e[3][at], ws);
          put(&e[4][at], wx);
        }
      }
      put(&e[0][at], us);
      put(&e[1][at], ux);
      __syncthreads();
      C as[CPL], ax[CPL], bs[CPL], bx[CPL];
      get(&e[0][above], as);
      get(&e[1][above], ax);
      get(&e[3][below], bs);
      get(&e[4][below], bx);
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        if (RPT > 1) {
          finish<C>(as[c], ax[c], l0[c], x0[c], w0[c], v0[c], d[0][c], jx[0][c], jy[0][c]);
          d[RPT - 1][c] = ps[c] + bs[c];
          jx[RPT - 1][c] = px[c] + bx[c];
          jy[RPT - 1][c] = pu[c] - bs[c];
        } else {
          finish<C>(as[c], ax[c], l0[c], x0[c], bs[c], bx[c], d[0][c], jx[0][c], jy[0][c]);
        }
      }
      if (Shared::kCopies == 1) __syncthreads();
    }
  }

  // The same walk with walls.  from_wall: eight bits per node, bit q - 1 set where its
  // source along e_q is a wall; fluid: a bit per node (node i * CPL + c).  An arrival from
  // a wall is replaced by the target's own value before it is summed.
  static constexpr int kWords = (RPT * CPL + 3) / 4;
  // with one or two nodes a thread their 18 conditions stay in scalar registers over the
  // loop: one vector operation a select instead of two
  static constexpr bool kConditions = CONDS && RPT * CPL <= 2;
  __device__ __forceinline__ void march_walls(Shared &sh, const int steps, uint32_t (&from_wall)[kWords], uint32_t fluid) {
    constexpr bool HALF = WALL == WALL_HALFWAY;
    for (int s = 0; s < steps; ++s) {
      C(*const e)[NODES] = sh.v[s % Shared::kCopies];
      if (!kConditions) {
        // the masks are formed anew in every step: kept over the loop they would take a
        // register each
#pragma unroll
        for (int k = 0; k < kWords; ++k) asm volatile("" : "+v"(from_wall[k]));
        asm volatile("" : "+v"(fluid));
      }
      C l0[CPL], x0[CPL], w0[CPL], v0[CPL];
      C ps[CPL], px[CPL], pu[CPL];
      C u[CPL][3];                                        // arrivals of the newest row in the row below
      C own0[HALF ? CPL : 1][3], own[HALF ? CPL : 1][3];  // half-way rule: what row 0 sends up, the newest row down
      (void)own0;
      (void)own;
      // arrival of target (i, c) along e_q, or what stands for it when its source is a wall
      auto sel = [&](const int i, const int c, const int q, const C arrived, const C sent_back)
          __attribute__((always_inline)) -> C {
        const C v = HALF ? sent_back : q <= 4 ? wall_axis<C>(d[i][c]) : wall_diag<C>(d[i][c]);
        const int node = i * CPL + c, bit = node % 4 * 8 + q - 1;
        if (kConditions) return (from_wall[node / 4] >> bit & 1u) ? v : arrived;
        return pick(spread(from_wall[node / 4], bit), v, arrived);
      };
      auto store = [&](const int i, const int c, const C dn, const C xn, const C yn) __attribute__((always_inline)) {
        if (kConditions) {
          const bool on = fluid >> (i * CPL + c) & 1u;
          d[i][c] = on ? dn : d[i][c];
          jx[i][c] = on ? xn : jx[i][c];
          jy[i][c] = on ? yn : jy[i][c];
          return;
        }
        const uint32_t live = spread(fluid, i * CPL + c);
        d[i][c] = pick(live, dn, d[i][c]);
        jx[i][c] = pick(live, xn, jx[i][c]);
        jy[i][c] = pick(live, yn, jy[i][c]);
      };
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        // one row at a time, so the rows' temporaries are not live together
        if (RPT * CPL > 2) __builtin_amdgcn_sched_barrier(0);
        if (T::kScaled && s > 0) {
#pragma unroll
          for (int c = 0; c < CPL; ++c) {
            C t0 = d[i][c], t1 = jx[i][c], t2 = jy[i][c];
            codec(t0, t1, t2);
            store(i, c, t0, t1, t2);
          }
        }
        C f[CPL][9], g[CPL][9];
        arrivals(i, f, g);
        if (i == 0) {
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            C o[CPL];
#pragma unroll
            for (int c = 0; c < CPL; ++c) o[c] = g[c][k == 0 ? 8 : k == 1 ? 4 : 7];
            put(&e[3 + k][at], o);
          }
        }
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const int h = HALF ? c : 0;
          if (i > 0) {  // target row i - 1 from this row
            const C a8 = sel(i - 1, c, 8, g[c][8], own[h][0]), a4 = sel(i - 1, c, 4, g[c][4], own[h][1]),
                    a7 = sel(i - 1, c, 7, g[c][7], own[h][2]);
            const C ws = row_sum(a8, a4, a7), wx = row_dif(a8, a7);
            if (i == 1) {
              w0[c] = ws;
              v0[c] = wx;
            } else {
              store(i - 1, c, ps[c] + ws, px[c] + wx, pu[c] - ws);
            }
          }
          const C a1 = sel(i, c, 1, g[c][1], f[c][3]), a3 = sel(i, c, 3, g[c][3], f[c][1]);
          const C ls = row_sum(a1, g[c][0], a3), lx = row_dif(a1, a3);
          if (i == 0) {
            l0[c] = ls;
            x0[c] = lx;
          } else {
            const C a5 = sel(i, c, 5, u[c][0], f[c][7]), a2 = sel(i, c, 2, u[c][1], f[c][4]),
                    a6 = sel(i, c, 6, u[c][2], f[c][8]);
            pu[c] = row_sum(a5, a2, a6);
            ps[c] = pu[c] + ls;
            px[c] = row_dif(a5, a6) + lx;
          }
          u[c][0] = g[c][5];
          u[c][1] = g[c][2];
          u[c][2] = g[c][6];
          if (HALF) {
            own[h][0] = f[c][6];
            own[h][1] = f[c][2];
            own[h][2] = f[c][5];
            if (i == 0) {
              own0[h][0] = f[c][7];
              own0[h][1] = f[c][4];
              own0[h][2] = f[c][8];
            }
          }
        }
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        C o[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) o[c] = u[c][k];
        put(&e[k][at], o);
      }
      __syncthreads();
      C a[3][CPL], b[3][CPL];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        get(&e[k][above], a[k]);
        get(&e[3 + k][below], b[k]);
      }
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int h = HALF ? c : 0;
        const C a5 = sel(0, c, 5, a[0][c], own0[h][0]), a2 = sel(0, c, 2, a[1][c], own0[h][1]),
                a6 = sel(0, c, 6, a[2][c], own0[h][2]);
        const C b8 = sel(RPT - 1, c, 8, b[0][c], own[h][0]), b4 = sel(RPT - 1, c, 4, b[1][c], own[h][1]),
                b7 = sel(RPT - 1, c, 7, b[2][c], own[h][2]);
        const C bs = row_sum(b8, b4, b7), bx = row_dif(b8, b7);
        C dn, xn, yn;
        if (RPT > 1) {
          store(RPT - 1, c, ps[c] + bs, px[c] + bx, pu[c] - bs);
          finish<C>(row_sum(a5, a2, a6), row_dif(a5, a6), l0[c], x0[c], w0[c], v0[c], dn, xn, yn);
        } else {
          finish<C>(row_sum(a5, a2, a6), row_dif(a5, a6), l0[c], x0[c], bs, bx, dn, xn, yn);
        }
        store(0, c, dn, xn, yn);
      }
      if (Shared::kCopies == 1) __syncthreads();
    }
  }
};

template <int P, bool HASWALL, int WALL, int W, int CPL, int RPT, int THREADS, bool UNIT, bool CONDS = true>
__device__ __forceinline__ void tile_body(
    const StepArgs &a, const TileMap &m, const int tile, typename TileRegion<P, WALL, W, CPL, RPT, THREADS, UNIT, CONDS>::Shared &sh) {
  using R = TileRegion<P, WALL, W, CPL, RPT, THREADS, UNIT, CONDS>;
  using T = Traits<P>;
  using C = typename T::C;
  using S = typename T::S;
  using SP = Pack<S, CPL>;
  static_assert(W == 32 || W == 64, "a row is half a wavefront or one");
  static_assert(RPT * CPL <= 32, "one FLUID bit per node of a thread");
  R r;
  r.Fx = C(a.fx);
  r.Fy = C(a.fy);
  r.sd = C(a.sc_d);
  r.sj = C(a.sc_j);
  r.ed = C(a.is_d);
  r.ej = C(a.is_j);
  const int lane = threadIdx.x & (W - 1), grp = threadIdx.x / W;
  const int col = lane * CPL;
  r.at = grp * W * CPL + col;
  // the outermost groups read their own rows instead of a neighbour's: halo or grid edge
  r.above = grp > 0 ? r.at - W * CPL : r.at;
  r.below = grp < R::GROUPS - 1 ? r.at + W * CPL : r.at;
  const int ty = tile / m.tiles_x, tx = tile - ty * m.tiles_x;
  const int x = tx * m.ox - m.hx + col;
  const int y0 = ty * m.oy - m.hy + grp * RPT;
  const bool px = !HASWALL || (a.periodic & 1u), py = !HASWALL || (a.periodic & 2u);
  const S *const s0 = static_cast<const S *>(a.src[0]), *const s1 = static_cast<const S *>(a.src[1]),
                *const s2 = static_cast<const S *>(a.src[2]);

  const TilePlace<CPL, RPT> at(x, y0, a.nx, a.ny, px, py);
  // x is a multiple of CPL, so where CPL divides nx or x is not periodic (the rest of a
  // row's last chunk is padding) a chunk is one aligned vector
  SP v0[RPT], v1[RPT], v2[RPT];
  if (CPL > 1 && !(px && a.nx % CPL != 0)) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const long k = (long)max(at.wy[i], 0) * a.rs + max(at.wx[0], 0);
      v0[i] = *reinterpret_cast<const SP *>(s0 + k);
      v1[i] = *reinterpret_cast<const SP *>(s1 + k);
      v2[i] = *reinterpret_cast<const SP *>(s2 + k);
    }
  } else {
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const long k = (long)max(at.wy[i], 0) * a.rs + max(at.wx[c], 0);
        v0[i].v[c] = s0[k];
        v1[i].v[c] = s1[k];
        v2[i].v[c] = s2[k];
      }
  }
  uint32_t solid[RPT + 2], fluid = 0;
  (void)solid;
  bool walls = false;
  if constexpr (HASWALL) tile_flags<CPL, RPT>(a.flags, a.pitch, at, solid, fluid);
#pragma unroll
  for (int i = 0; i < RPT; ++i)
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      r.d[i][c] = T::dec(v0[i].v[c]);
      r.jx[i][c] = T::dec(v1[i].v[c]);
      r.jy[i][c] = T::dec(v2[i].v[c]);
      if (T::kScaled && !UNIT) {
        r.d[i][c] *= r.sd;
        r.jx[i][c] *= r.sj;
        r.jy[i][c] *= r.sj;
      }
    }
  if constexpr (HASWALL) {
    constexpr uint32_t kAll = RPT * CPL == 32 ? 0xffffffffu : (1u << (RPT * CPL % 32)) - 1u;
    // (without a halo the region's edge is the grid's)
    walls = __syncthreads_or(fluid != kAll) || m.hx == 0 || m.hy == 0;
  }
  if constexpr (HASWALL) {
    if (walls) {
      uint32_t from_wall[R::kWords];
      tile_walls<W, CPL, RPT, THREADS>(solid, reinterpret_cast<uint32_t *>(&sh), from_wall);
      r.march_walls(sh, m.steps, from_wall, fluid);
    } else {
      r.march(sh, m.steps);
    }
  } else {
    r.march(sh, m.steps);
  }

  const int r0 = grp * RPT;
  S *const d0 = static_cast<S *>(a.dst[0]), *const d1 = static_cast<S *>(a.dst[1]), *const d2 = static_cast<S *>(a.dst[2]);
  const bool col_in = col >= m.hx && col < m.hx + m.ox && x < a.nx;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int y = y0 + i;
    if (!col_in || r0 + i < m.hy || r0 + i >= m.hy + m.oy || y >= a.ny) continue;
    SP o0, o1, o2;
    bool whole = true;
    bool own[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      o0.v[c] = T::enc(T::kScaled && !UNIT ? r.d[i][c] * r.ed : r.d[i][c]);
      o1.v[c] = T::enc(T::kScaled && !UNIT ? r.jx[i][c] * r.ej : r.jx[i][c]);
      o2.v[c] = T::enc(T::kScaled && !UNIT ? r.jy[i][c] * r.ej : r.jy[i][c]);
      own[c] = x + c < a.nx && (!HASWALL || (fluid >> (i * CPL + c) & 1u));
      whole &= own[c];
    }
    const long k = (long)y * a.rs + x;
    if (whole) {
      *reinterpret_cast<SP *>(d0 + k) = o0;
      *reinterpret_cast<SP *>(d1 + k) = o1;
      *reinterpret_cast<SP *>(d2 + k) = o2;
    } else {
#pragma unroll
      for (int c = 0; c < CPL; ++c)
        if (own[c]) {
          d0[k + c] = o0.v[c];
          d1[k + c] = o1.v[c];
          d2[k + c] = o2.v[c];
        }
    }
  }
}

template <int P, bool HASWALL, int WALL, int W, int CPL, int RPT, int THREADS>
__global__ void __launch_bounds__(THREADS) k_step_tile(StepArgs a, TileMap m) {
  __shared__ __align__(16) TileShared<typename Traits<P>::C, THREADS * CPL> sh;
  const int tile = tile_of(m);
  if (tile >= m.tiles) return;  // uniform across the block
  if constexpr (Traits<P>::kScaled) {
    // unit storage scales (the default): the codec without its multiplications
    if (a.sc_d == 1.0 && a.sc_j == 1.0 && a.is_d == 1.0 && a.is_j == 1.0)
      tile_body<P, HASWALL, WALL, W, CPL, RPT, THREADS, true>(a, m, tile, sh);
    else
      tile_body<P, HASWALL, WALL, W, CPL, RPT, THREADS, false>(a, m, tile, sh);
  } else {
    tile_body<P, HASWALL, WALL, W, CPL, RPT, THREADS, true>(a, m, tile, sh);
  }
}

}  // namespace lbt1
