// Several multiphase steps per launch on regions of nodes held in registers (the regions and
// exchange of lbt1_tile.hpp; the force of lbt1_multiphase.hpp).
//
// The force of a node needs the pseudopotential of its neighbours and its update the
// emissions of its neighbours, so a step exchanges rows twice (psi, then arrivals) and uses up
// two nodes of the region's halo.  Any geometry: a SOLID neighbour contributes the psi of its
// stored density, a neighbour outside a non-periodic axis that of the node itself.  A node
// costs one exponential a step where the gather kernel evaluates 81.  Arithmetic and order of
// the gather and strip kernels: the same bits.
//
// One or two steps at a time, drops up to 1024^2 were bound by launches and a strip's walk
// (FP32 1024^2: 9.8 us a step; 5.7 now), grids with walls or of odd width by the gather
// kernel's repeated work (109 us; 7.2 now).  Here vector-ALU issue is: about 90 operations a
// node, of which a 64 x 64 region at 4 steps stores 56 %.
#pragma once
#include "lbt1_tile.hpp"

namespace lbt1 {

template <typename C, int THREADS>
struct ScShared {
  C v[8][THREADS];  // psi of a group's last row and first row, then as TileShared
};

template <int P, int WALL, int W, int RPT, int THREADS>
struct ScRegion {
  using T = Traits<P>;
  using C = typename T::C;
  static constexpr int kWords = (RPT + 3) / 4;

  C d[RPT], jx[RPT], jy[RPT];
  C Fx, Fy, G, rho0, irho0, sd, sj, ed, ej;
  int at, above, below;

  struct Row {  // psi of a row: in this column, to the left and to the right
    C c, l, r;
  };
  static __device__ __forceinline__ Row row_of(const C p) {
    return {p, dpp_shift<kDppWaveShr1>(p), dpp_shift<kDppWaveShl1>(p)};
  }

  // BOUNDED: the region holds walls or reaches a grid edge.  edge: bit 0 / 1: the column left /
  // right of this thread's is outside the grid, bit 2 + i / 2 + RPT + i: the row before /
  // after row i is.
  template <bool BOUNDED>
  __device__ __forceinline__ void march(ScShared<C, THREADS> &sh, const int steps, uint32_t (&from_wall)[kWords],
                                        uint32_t fluid, uint32_t edge) {
    constexpr bool HALF = WALL == WALL_HALFWAY;
    C(*const e)[THREADS] = sh.v;
    for (int s = 0; s < steps; ++s) {
      if constexpr (BOUNDED) {
#pragma unroll
        for (int k = 0; k < kWords; ++k) asm volatile("" : "+v"(from_wall[k]));
        asm volatile("" : "+v"(fluid), "+v"(edge));
      }
      auto store = [&](const int i, const C dn, const C xn, const C yn) __attribute__((always_inline)) {
        const uint32_t live = BOUNDED ? spread(fluid, i) : 0u;
        d[i] = BOUNDED ? pick(live, dn, d[i]) : dn;
        jx[i] = BOUNDED ? pick(live, xn, jx[i]) : xn;
        jy[i] = BOUNDED ? pick(live, yn, jy[i]) : yn;
      };
      auto sel = [&](const int i, const int q, const C arrived, const C back) __attribute__((always_inline)) -> C {
        if (!BOUNDED) return arrived;
        const C v = HALF ? back : q <= 4 ? wall_axis<C>(d[i]) : wall_diag<C>(d[i]);
        return pick(spread(from_wall[i / 4], i % 4 * 8 + q - 1), v, arrived);
      };
      C psi[RPT];
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        if (T::kScaled && s > 0)
          store(i, T::dec(T::enc(d[i] * ed)) * sd, T::dec(T::enc(jx[i] * ej)) * sj, T::dec(T::enc(jy[i] * ej)) * sj);
        psi[i] = sc_psi<C>(C(1) + d[i], rho0, irho0);
      }
      e[0][at] = psi[RPT - 1];
      e[1][at] = psi[0];
      __syncthreads();
      const C below_psi = e[1][below];
      Row lo = row_of(e[0][above]), mid = row_of(psi[0]);
      C l0 = C(0), x0 = C(0), w0 = C(0), v0 = C(0), ps = C(0), px = C(0), pu = C(0), us = C(0), ux = C(0);
      C u[3] = {}, own[3] = {}, own0[3] = {};
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        __builtin_amdgcn_sched_barrier(0);  // one row's temporaries at a time
        const Row hi = row_of(i + 1 < RPT ? psi[i + 1 < RPT ? i + 1 : 0] : below_psi);
        C p9[9] = {mid.c, mid.r, hi.c, mid.l, lo.c, hi.r, hi.l, lo.l, lo.r};
        if (BOUNDED) {
          const uint32_t ml = spread(edge, 0), mr = spread(edge, 1), mu = spread(edge, 2 + i), md = spread(edge, 2 + RPT + i);
#pragma unroll
          for (int q = 1; q < 9; ++q) {
            uint32_t m = 0;
            if (kEx[q] < 0) m |= ml;
            if (kEx[q] > 0) m |= mr;
            if (kEy[q] < 0) m |= mu;
            if (kEy[q] > 0) m |= md;
            p9[q] = pick(m, p9[0], p9[q]);
          }
        }
        C gx, gy;
        sc_force<C>(p9, G, gx, gy);
        C f[9], a[9];
        emit<C>(d[i], jx[i], jy[i], Fx + gx, Fy + gy, f);
#pragma unroll
        for (int q = 0; q < 9; ++q)
          a[q] = kEx[q] == 1 ? dpp_shift<kDppWaveShr1>(f[q]) : kEx[q] == -1 ? dpp_shift<kDppWaveShl1>(f[q]) : f[q];
        if (i == 0) {
          if (BOUNDED) {
            e[5][at] = a[8];
            e[6][at] = a[4];
            e[7][at] = a[7];
          } else {
            e[5][at] = row_sum(a[8], a[4], a[7]);
            e[6][at] = row_dif(a[8], a[7]);
          }
        } else {
          const C a8 = sel(i - 1, 8, a[8], own[0]), a4 = sel(i - 1, 4, a[4], own[1]), a7 = sel(i - 1, 7, a[7], own[2]);
          const C ws = row_sum(a8, a4, a7), wx = row_dif(a8, a7);
          if (i == 1) {
            w0 = ws;
            v0 = wx;
          } else {
            store(i - 1, ps + ws, px + wx, pu - ws);
          }
        }
        const C a1 = sel(i, 1, a[1], f[3]), a3 = sel(i, 3, a[3], f[1]);
        const C ls = row_sum(a1, a[0], a3), lx = row_dif(a1, a3);
        if (i == 0) {
          l0 = ls;
          x0 = lx;
        } else {
          if (BOUNDED) {
            const C a5 = sel(i, 5, u[0], f[7]), a2 = sel(i, 2, u[1], f[4]), a6 = sel(i, 6, u[2], f[8]);
            us = row_sum(a5, a2, a6);
            ux = row_dif(a5, a6);
          }
          ps = us + ls;
          px = ux + lx;
          pu = us;
        }
        if (BOUNDED) {
          u[0] = a[5];
          u[1] = a[2];
          u[2] = a[6];
          own[0] = f[6];
          own[1] = f[2];
          own[2] = f[5];
          if (i == 0) {
            own0[0] = f[7];
            own0[1] = f[4];
            own0[2] = f[8];
          }
        } else {
          us = row_sum(a[5], a[2], a[6]);
          ux = row_dif(a[5], a[6]);
        }
        lo = mid;
        mid = hi;
      }
      e[2][at] = BOUNDED ? u[0] : us;
      e[3][at] = BOUNDED ? u[1] : ux;
      if (BOUNDED) e[4][at] = u[2];
      __syncthreads();
      C as, ax, bs, bx;
      if (BOUNDED) {
        const C a5 = sel(0, 5, e[2][above], own0[0]), a2 = sel(0, 2, e[3][above], own0[1]), a6 = sel(0, 6, e[4][above], own0[2]);
        const C b8 = sel(RPT - 1, 8, e[5][below], own[0]), b4 = sel(RPT - 1, 4, e[6][below], own[1]),
                b7 = sel(RPT - 1, 7, e[7][below], own[2]);
        as = row_sum(a5, a2, a6);
        ax = row_dif(a5, a6);
        bs = row_sum(b8, b4, b7);
        bx = row_dif(b8, b7);
      } else {
        as = e[2][above];
        ax = e[3][above];
        bs = e[5][below];
        bx = e[6][below];
      }
      C dn, xn, yn;
      static_assert(RPT > 1, "the first and the last row of a thread are different rows");
      store(RPT - 1, ps + bs, px + bx, pu - bs);
      finish<C>(as, ax, l0, x0, w0, v0, dn, xn, yn);
      store(0, dn, xn, yn);
    }
  }
};

template <int P, bool HASWALL, int WALL, int W, int RPT, int THREADS>
__global__ void __launch_bounds__(THREADS) k_sc_tile(StepArgs a, TileMap m) {
  using R = ScRegion<P, WALL, W, RPT, THREADS>;
  using T = Traits<P>;
  using C = typename T::C;
  using S = typename T::S;
  __shared__ __align__(16) ScShared<C, THREADS> sh;
  const int tile = tile_of(m);
  if (tile >= m.tiles) return;  // uniform across the block
  R r;
  r.Fx = C(a.fx);
  r.Fy = C(a.fy);
  r.G = C(a.sc_G);
  r.rho0 = C(a.sc_rho0);
  r.irho0 = C(1.0 / a.sc_rho0);
  r.sd = C(a.sc_d);
  r.sj = C(a.sc_j);
  r.ed = C(a.is_d);
  r.ej = C(a.is_j);
  const int lane = threadIdx.x & (W - 1), grp = threadIdx.x / W;
  r.at = threadIdx.x;
  r.above = grp > 0 ? r.at - W : r.at;
  r.below = grp < THREADS / W - 1 ? r.at + W : r.at;
  const int ty = tile / m.tiles_x, tx = tile - ty * m.tiles_x;
  const int x = tx * m.ox - m.hx + lane;
  const int y0 = ty * m.oy - m.hy + grp * RPT;
  const bool px = !HASWALL || (a.periodic & 1u), py = !HASWALL || (a.periodic & 2u);
  const TilePlace<1, RPT> at(x, y0, a.nx, a.ny, px, py);
#pragma unroll
  for (int i = 0; i < RPT; ++i)
    load_node<P>(a, (long)max(at.wy[i], 0) * a.rs + max(at.wx[0], 0), r.d[i], r.jx[i], r.jy[i]);
  uint32_t solid[RPT + 2], fluid = (1u << RPT) - 1u, from_wall[R::kWords] = {}, edge = 0;
  (void)solid;
  bool bounded = false;
  if constexpr (HASWALL) {
    tile_flags<1, RPT>(a.flags, a.pitch, at, solid, fluid);
    bounded = __syncthreads_or(fluid != (1u << RPT) - 1u) || m.hx == 0 || m.hy == 0;
    if (bounded) {
      tile_walls<W, 1, RPT, THREADS>(solid, reinterpret_cast<uint32_t *>(&sh), from_wall);
      edge = (uint32_t)(!px && x == 0) | (uint32_t)(!px && x == a.nx - 1) << 1;
#pragma unroll
      for (int i = 0; i < RPT; ++i)
        edge |= (uint32_t)(!py && y0 + i == 0) << (2 + i) | (uint32_t)(!py && y0 + i == a.ny - 1) << (2 + RPT + i);
      r.template march<true>(sh, m.steps, from_wall, fluid, edge);
    }
  }
  if (!bounded) r.template march<false>(sh, m.steps, from_wall, fluid, edge);

  const int r0 = grp * RPT;
  if (lane < m.hx || lane >= m.hx + m.ox || x >= a.nx) return;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int y = y0 + i;
    if (r0 + i < m.hy || r0 + i >= m.hy + m.oy || y >= a.ny || !(fluid >> i & 1u)) continue;
    const long k = (long)y * a.rs + x;
    static_cast<S *>(a.dst[0])[k] = T::enc(T::kScaled ? r.d[i] * r.ed : r.d[i]);
    static_cast<S *>(a.dst[1])[k] = T::enc(T::kScaled ? r.jx[i] * r.ej : r.jx[i]);
    static_cast<S *>(a.dst[2])[k] = T::enc(T::kScaled ? r.jy[i] * r.ej : r.jy[i]);
  }
}

}  // namespace lbt1
