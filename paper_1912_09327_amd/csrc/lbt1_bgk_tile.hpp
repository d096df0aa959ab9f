// Several steps per launch of the stored-population BGK method on regions of nodes held
// in registers (the regions, halos and exchange of lbt1_tile.hpp; the method and its
// arithmetic of lbt1_bgk.hpp).
//
// One step at a time the method reads and writes nine values a node: 72 bytes in FP32,
// 5.0 TB/s and 57 us a step at 2048^2, with nothing left to gain but fewer passes.  Here
// a thread keeps the nine populations of RPT nodes of one column; a step relaxes them row
// by row and takes each new population from the node it comes from: its own row by lane
// shifts, the rows next to it from registers or, between threads, through LDS.  What
// enters a wall comes back to its sender, so a node whose source along e_q is a wall
// takes w_q rho of its own or, half-way, its own relaxed population along -e_q.  A halo
// of a node per step, as in lbt1_tile.hpp; the same bits as single steps.  Regions of
// 64 x 64 nodes at 4 to 6 steps (64 x 32 with walls, whose masks take registers) read
// 1.3 to 1.5 of the state and write it once: 18.7 us a step at 2048^2 FP32, 35.9 in
// FP64 (114 before), 19.8 in FP16S (50 before).
#pragma once
#include "lbt1_args.hpp"
#include "lbt1_bgk.hpp"
#include "lbt1_tile.hpp"

namespace lbt1 {

template <int P, bool HASWALL, int WALL, int W, int RPT, int THREADS>
struct BgkRegion {
  using T = Traits<P>;
  using C = typename T::C;
  static constexpr int NODES = THREADS;
  using Shared = TileShared<C, NODES>;
  static constexpr int kWords = (RPT + 3) / 4;

  C g[RPT][9];
  C Fx, Fy, om, sc, is;
  int at, above, below;

  // BOUNDED: the region holds walls or fixed nodes
  template <bool BOUNDED>
  __device__ __forceinline__ void march(Shared &sh, const int steps, uint32_t (&from_wall)[kWords], uint32_t fluid) {
    constexpr bool HALF = WALL == WALL_HALFWAY;
    for (int s = 0; s < steps; ++s) {
      C(*const e)[NODES] = sh.v[s % Shared::kCopies];
      if constexpr (BOUNDED) {
#pragma unroll
        for (int k = 0; k < kWords; ++k) asm volatile("" : "+v"(from_wall[k]));
        asm volatile("" : "+v"(fluid));
      }
      // new value of population q of node i, unless the node is held
      auto store = [&](const int i, const int q, const C v) __attribute__((always_inline)) {
        g[i][q] = BOUNDED ? pick(spread(fluid, i), v, g[i][q]) : v;
      };
      // what arrives at node i along e_q, or comes back from a wall: d its rho - 1, back
      // its relaxed population along -e_q
      auto sel = [&](const int i, const int q, const C arrived, const C d, const C back)
          __attribute__((always_inline)) -> C {
        if (!BOUNDED) return arrived;
        const C v = HALF ? back : q <= 4 ? wall_axis<C>(d) : wall_diag<C>(d);
        return pick(spread(from_wall[i / 4], i % 4 * 8 + q - 1), v, arrived);
      };
      C up[3];                          // what the newest row sends into the row below it
      C dn = C(0), d0 = C(0);           // rho - 1 of the newest row, of row 0
      C back[3] = {}, back0[3] = {};    // half-way: what they send up (newest) and up into row -1 (row 0)
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        __builtin_amdgcn_sched_barrier(0);  // one row's temporaries at a time
        if (T::kScaled && s > 0) {
#pragma unroll
          for (int q = 0; q < 9; ++q) store(i, q, T::dec(T::enc(g[i][q] * is)) * sc);
        }
        const C d = pop_density<C>(g[i]);
        const C jx = ((g[i][1] - g[i][3]) + (g[i][5] - g[i][6])) + (g[i][8] - g[i][7]);
        const C jy = ((g[i][2] - g[i][4]) + (g[i][5] - g[i][7])) + (g[i][6] - g[i][8]);
        C post[9];
        emit<C>(d, jx, jy, Fx, Fy, post);
#pragma unroll
        for (int q = 0; q < 9; ++q) {
          post[q] = fmaC<C>(om, post[q] - g[i][q], g[i][q]);
          if (BOUNDED) post[q] = pick(spread(fluid, i), post[q], g[i][q]);  // FIXED nodes send what they hold
        }
        C a[9];
#pragma unroll
        for (int q = 0; q < 9; ++q)
          a[q] = kEx[q] == 1 ? dpp_shift<kDppWaveShr1>(post[q]) : kEx[q] == -1 ? dpp_shift<kDppWaveShl1>(post[q]) : post[q];
        if (i == 0) {
          e[3][at] = a[8];
          e[4][at] = a[4];
          e[5][at] = a[7];
        } else {
          store(i - 1, 8, sel(i - 1, 8, a[8], dn, back[0]));
          store(i - 1, 4, sel(i - 1, 4, a[4], dn, back[1]));
          store(i - 1, 7, sel(i - 1, 7, a[7], dn, back[2]));
        }
        store(i, 0, a[0]);
        store(i, 1, sel(i, 1, a[1], d, post[3]));
        store(i, 3, sel(i, 3, a[3], d, post[1]));
        if (i == 0) {
          d0 = d;
          back0[0] = post[7];
          back0[1] = post[4];
          back0[2] = post[8];
        } else {
          store(i, 5, sel(i, 5, up[0], d, post[7]));
          store(i, 2, sel(i, 2, up[1], d, post[4]));
          store(i, 6, sel(i, 6, up[2], d, post[8]));
        }
        up[0] = a[5];
        up[1] = a[2];
        up[2] = a[6];
        dn = d;
        back[0] = post[6];
        back[1] = post[2];
        back[2] = post[5];
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) e[k][at] = up[k];
      __syncthreads();
      store(0, 5, sel(0, 5, e[0][above], d0, back0[0]));
      store(0, 2, sel(0, 2, e[1][above], d0, back0[1]));
      store(0, 6, sel(0, 6, e[2][above], d0, back0[2]));
      store(RPT - 1, 8, sel(RPT - 1, 8, e[3][below], dn, back[0]));
      store(RPT - 1, 4, sel(RPT - 1, 4, e[4][below], dn, back[1]));
      store(RPT - 1, 7, sel(RPT - 1, 7, e[5][below], dn, back[2]));
      if (Shared::kCopies == 1) __syncthreads();
    }
  }
};

template <int P, bool HASWALL, int WALL, int W, int RPT, int THREADS>
__global__ void __launch_bounds__(THREADS) k_bgk_tile(BgkArgs a, TileMap m) {
  using R = BgkRegion<P, HASWALL, WALL, W, RPT, THREADS>;
  using T = Traits<P>;
  using C = typename T::C;
  using S = typename T::S;
  __shared__ __align__(16) typename R::Shared sh;
  R r;
  r.Fx = C(a.fx);
  r.Fy = C(a.fy);
  r.om = C(a.omega);
  r.sc = C(a.sc);
  r.is = C(a.is);
  const int lane = threadIdx.x & (W - 1), grp = threadIdx.x / W;
  r.at = threadIdx.x;
  r.above = grp > 0 ? r.at - W : r.at;
  r.below = grp < THREADS / W - 1 ? r.at + W : r.at;
  const int tile = tile_of(m);
  if (tile >= m.tiles) return;  // uniform across the block
  const int ty = tile / m.tiles_x, tx = tile - ty * m.tiles_x;
  const int x = tx * m.ox - m.hx + lane;
  const int y0 = ty * m.oy - m.hy + grp * RPT;
  const bool px = !HASWALL || (a.periodic & 1u), py = !HASWALL || (a.periodic & 2u);
  const TilePlace<1, RPT> at(x, y0, a.nx, a.ny, px, py);
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const long k = (long)max(at.wy[i], 0) * a.rs + max(at.wx[0], 0);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      r.g[i][q] = T::dec(static_cast<const S *>(a.src[q])[k]);
      if (T::kScaled) r.g[i][q] *= r.sc;
    }
  }
  uint32_t solid[RPT + 2], fluid = (1u << RPT) - 1u, from_wall[R::kWords] = {};
  (void)solid;
  bool bounded = false;
  if constexpr (HASWALL) {
    tile_flags<1, RPT>(a.flags, a.pitch, at, solid, fluid);
    bounded = __syncthreads_or(fluid != (1u << RPT) - 1u) || m.hx == 0 || m.hy == 0;
    if (bounded) {
      tile_walls<W, 1, RPT, THREADS>(solid, reinterpret_cast<uint32_t *>(&sh), from_wall);
      r.template march<true>(sh, m.steps, from_wall, fluid);
    }
  }
  if (!bounded) r.template march<false>(sh, m.steps, from_wall, fluid);

  const int r0 = grp * RPT;
  if (lane < m.hx || lane >= m.hx + m.ox || x >= a.nx) return;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int y = y0 + i;
    if (r0 + i < m.hy || r0 + i >= m.hy + m.oy || y >= a.ny || !(fluid >> i & 1u)) continue;
    const long k = (long)y * a.rs + x;
#pragma unroll
    for (int q = 0; q < 9; ++q) static_cast<S *>(a.dst[q])[k] = T::enc(T::kScaled ? r.g[i][q] * r.is : r.g[i][q]);
  }
}

}  // namespace lbt1
