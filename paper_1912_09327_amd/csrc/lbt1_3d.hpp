// Three-dimensional LBMTau1 step (D3Q19, D3Q27) for gfx950.
//
// The method of section 2 / Algorithm 1 on the 3-D lattices of the memory
// analysis of section 4: a node keeps its density and momentum (four values,
// 2 * 4 * c bytes per node over both parities against (2 Q + 4) c for the
// standard method), and its new moments are the sums over the Q directions of
// the equilibrium that the upwind node x - e_q sends along e_q.  Walls, lid
// (FIXED) nodes and the body force as in 2-D.
//
// Arithmetic as the 2-D kernels: density as d = rho - 1, equilibrium
// deviations w_q [d + 3 e.J + 4.5 (e.J)^2 / rho - 1.5 |J|^2 / rho] with the
// forced momentum J = j + F.  Direction order here: rest, the six faces, the
// twelve edges, the eight corners (D3Q19 = the first 19).
#pragma once
#include <type_traits>

#include "lbt1_device.hpp"

namespace lbt1 {

__device__ constexpr int k3x[27] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0,
                                    1, -1, 1, -1, 1, -1, 1, -1};
__device__ constexpr int k3y[27] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1,
                                    1, -1, 1, -1, -1, 1, -1, 1};
__device__ constexpr int k3z[27] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1,
                                    1, -1, -1, 1, 1, -1, -1, 1};

struct Step3Args {
  const void *src[4];  // d, jx, jy, jz of the current parity
  void *dst[4];
  const uint8_t *flags;  // NULL: every node FLUID and all three axes periodic
  int nx, ny, nz;
  int pitch;             // values per row of one field (nx rounded up to 64)
  long rs, zs;           // row and plane strides of the moment fields, in values
  long fzs;              // plane stride of the flags
  uint32_t periodic;     // bit 0 x, bit 1 y, bit 2 z
  double fx, fy, fz;
  double sc_d, sc_j, is_d, is_j;
};

// Tiles of k_step3_march: rows of a tile, planes of a chunk, tiles per row, per plane and in
// all, and per XCD (8 * per_xcd blocks).
struct March3Map {
  int oy, zc;
  int tiles_x, tiles_y, tiles, per_xcd;
  int past;  // stores past the caches
};

// The Q equilibrium deviations of a source node with deviation d and forced momentum J:
// w_q [base + 4.5 (e.J)^2 / rho + 3 e.J] with base = d - 1.5 tr P, P = J J / rho, built from
// shared terms (59 operations for D3Q19, 83 for D3Q27, where a direction at a time takes
// five or six each).
template <typename C, int Q>
__device__ __forceinline__ void emit3(const C d, const C Jx, const C Jy, const C Jz, C (&f)[Q]) {
  const C inv = recip<C>(C(1) + d);
  const C ux = Jx * inv, uy = Jy * inv, uz = Jz * inv;
  const C pxx = Jx * ux, pyy = Jy * uy, pzz = Jz * uz;
  const C pxy = Jx * uy, pxz = Jx * uz, pyz = Jy * uz;
  const C sxy = pxx + pyy, sxz = pxx + pzz, syz = pyy + pzz;
  const C t = sxy + pzz;
  const C base = fmaC<C>(C(-1.5), t, d);
  // weights of the faces wf and edges we: coefficients 4.5 w, 9 w and 3 w
  constexpr double wf = Q == 19 ? 1.0 / 18.0 : 2.0 / 27.0, we = Q == 19 ? 1.0 / 36.0 : 1.0 / 54.0;
  // 3 wf; for D3Q19 in 32 bits the neighbour of 1/6 with which the momentum's coefficients,
  // two of faces and eight of 1/12, add up to one exactly (1/6 and 1/12 are both rounded up,
  // and 3e-8 of the momentum a step would be gained)
  constexpr C w3f = sizeof(C) == 4 && Q == 19 ? C(0.1666666567325592) : C(3 * wf);
  f[0] = C(Q == 19 ? 1.0 / 3.0 : 8.0 / 27.0) * base;
  const C bf = C(wf) * base, be = C(we) * base;
  const C ax = fmaC<C>(C(4.5 * wf), pxx, bf), ay = fmaC<C>(C(4.5 * wf), pyy, bf), az = fmaC<C>(C(4.5 * wf), pzz, bf);
  f[1] = fmaC<C>(w3f, Jx, ax);
  f[2] = fmaC<C>(-w3f, Jx, ax);
  f[3] = fmaC<C>(w3f, Jy, ay);
  f[4] = fmaC<C>(-w3f, Jy, ay);
  f[5] = fmaC<C>(w3f, Jz, az);
  f[6] = fmaC<C>(-w3f, Jz, az);
  // edges of a plane (a, b): e = (1, 1), (-1, -1), (1, -1), (-1, 1)
  auto edges = [&](const int q, const C s, const C x, const C Ja, const C Jb) __attribute__((always_inline)) {
    const C b = fmaC<C>(C(4.5 * we), s, be);
    const C p = fmaC<C>(C(9 * we), x, b), m = fmaC<C>(C(-9 * we), x, b);
    const C sp = Ja + Jb, sm = Ja - Jb;
    f[q] = fmaC<C>(C(3 * we), sp, p);
    f[q + 1] = fmaC<C>(C(-3 * we), sp, p);
    f[q + 2] = fmaC<C>(C(3 * we), sm, m);
    f[q + 3] = fmaC<C>(C(-3 * we), sm, m);
  };
  edges(7, sxy, pxy, Jx, Jy);
  edges(11, sxz, pxz, Jx, Jz);
  edges(15, syz, pyz, Jy, Jz);
  if constexpr (Q == 27) {
    constexpr double wc = 1.0 / 216.0;
    const C b = fmaC<C>(C(4.5 * wc), t, C(wc) * base);
    const C a = pxz + pyz, c = pxz - pyz, sp = Jx + Jy, sm = Jx - Jy;
    auto corner = [&](const int q, const C x, const C dot) __attribute__((always_inline)) {
      const C m = fmaC<C>(C(9 * wc), x, b);
      f[q] = fmaC<C>(C(3 * wc), dot, m);
      f[q + 1] = fmaC<C>(C(-3 * wc), dot, m);
    };
    corner(19, pxy + a, sp + Jz);
    corner(21, pxy - a, sp - Jz);
    corner(23, c - pxy, sm + Jz);
    corner(25, -c - pxy, sm - Jz);
  }
}

// Direction with velocity (EX, EY, EZ), or -1 where the lattice has none.
template <int Q, int EX, int EY, int EZ>
constexpr int dir3() {
  constexpr int x[27] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1};
  constexpr int y[27] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, -1, 1, -1, 1};
  constexpr int z[27] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1, 1, -1, -1, 1, 1, -1, -1, 1};
  for (int q = 0; q < Q; ++q)
    if (x[q] == EX && y[q] == EY && z[q] == EZ) return q;
  return -1;
}

// Arrivals at a target are summed in groups of one (e_y, e_z), then over e_y, then over e_z.
// This order is part of the contract between the kernels.  FP32 against FP64 after 20 steps at
// 256^3: 1.2e-7 of the largest value (2.9e-7 when the arrivals were added one by one).
// A group's sum and x difference: the source on the left, the one in the target's column,
// the one on the right (D3Q19 has the middle one alone where e_y and e_z are both set).
template <typename C>
struct Group3 {
  C s, x;
};
template <typename C, int Q, int EY, int EZ>
__device__ __forceinline__ Group3<C> group3(const C (&a)[Q]) {
  constexpr int l = dir3<Q, 1, EY, EZ>(), c = dir3<Q, 0, EY, EZ>(), r = dir3<Q, -1, EY, EZ>();
  if constexpr (l < 0)
    return {a[c], C(0)};
  else
    return {(a[l] + a[c]) + a[r], a[l] - a[r]};
}
// The sums over e_y of one e_z: density, x and y.  WIDE: the outer groups have an x difference.
template <typename C>
struct Plane3 {
  C s, x, y;
};
template <bool WIDE, typename C>
__device__ __forceinline__ Plane3<C> plane3(const Group3<C> &u, const Group3<C> &l, const Group3<C> &w) {
  return {(u.s + l.s) + w.s, WIDE ? (u.x + l.x) + w.x : l.x, u.s - w.s};
}

// Walls: a SOLID source sends nothing, and what stands for it is added to the target's sums
// after the plane below, before the planes level with it and above.  m: bit
// (ez + 1) * 9 + (ey + 1) * 3 + ex + 1 set where the source x - e is a wall.
// Eq. feqnoslip: w_q d of its own for each, formed from integer counts of the weights (36ths
// or 216ths).  Half-way: its own emission f along -e_q for each, summed as arrivals are.
template <int Q>
__device__ __forceinline__ constexpr uint32_t wall_bit3(const int q) {
  return 1u << ((k3z[q] + 1) * 9 + (k3y[q] + 1) * 3 + k3x[q] + 1);
}
template <int Q>
__device__ __forceinline__ constexpr uint32_t wall_bits3() {
  uint32_t m = 0;
  for (int q = 1; q < Q; ++q) m |= wall_bit3<Q>(q);
  return m;
}
template <int Q>
__device__ __forceinline__ constexpr uint32_t wall_group3(const int ex, const int ey, const int ez, const int e2) {
  uint32_t m = 0;  // directions with these components (2: any) and this many nonzero ones
  for (int q = 1; q < Q; ++q)
    if ((ex == 2 || k3x[q] == ex) && (ey == 2 || k3y[q] == ey) && (ez == 2 || k3z[q] == ez) &&
        k3x[q] * k3x[q] + k3y[q] * k3y[q] + k3z[q] * k3z[q] == e2)
      m |= wall_bit3<Q>(q);
  return m;
}
// The weights' sum over the wall sources with these components, in 36ths (216ths).
template <int Q, int EX, int EY, int EZ>
__device__ __forceinline__ int wall_weight3(const uint32_t m) {
  constexpr uint32_t f = wall_group3<Q>(EX, EY, EZ, 1), e = wall_group3<Q>(EX, EY, EZ, 2), c = wall_group3<Q>(EX, EY, EZ, 3);
  if constexpr (Q == 19) return 2 * __builtin_popcount(m & f) + __builtin_popcount(m & e);
  return 16 * __builtin_popcount(m & f) + 4 * __builtin_popcount(m & e) + __builtin_popcount(m & c);
}
template <typename C>
struct Moments3 {
  C d, x, y, z;
};
// Half-way, where every node's wall sources are all on its left or all on its right (beside a wall
// or grid edge across x, the most frequent wall there is: every row has it): the same sums with the
// absent terms, which are zeros, left out.
template <int Q>
__device__ __forceinline__ constexpr uint32_t wall_column3(const int ex) {
  uint32_t m = 0;
  for (int q = 1; q < Q; ++q)
    if (k3x[q] == ex) m |= wall_bit3<Q>(q);
  return m;
}
template <typename C, int Q>
__device__ __forceinline__ Moments3<C> wall_side3(const uint32_t m, const C (&f)[Q]) {
  auto take = [&](const int l, const int r) __attribute__((always_inline)) {  // directions with e_x = 1 and -1
    const C v = (m & wall_bit3<Q>(r)) ? f[((r - 1) ^ 1) + 1] : C(0);
    return (m & wall_bit3<Q>(l)) ? f[((l - 1) ^ 1) + 1] : v;
  };
  C s[3], y[3];  // by e_z + 1
  const C u = take(dir3<Q, 1, 1, 0>(), dir3<Q, -1, 1, 0>()), l = take(dir3<Q, 1, 0, 0>(), dir3<Q, -1, 0, 0>()),
          w = take(dir3<Q, 1, -1, 0>(), dir3<Q, -1, -1, 0>());
  s[1] = (u + l) + w;
  y[1] = u - w;
  s[2] = take(dir3<Q, 1, 0, 1>(), dir3<Q, -1, 0, 1>());
  s[0] = take(dir3<Q, 1, 0, -1>(), dir3<Q, -1, 0, -1>());
  y[2] = y[0] = C(0);
  if constexpr (Q == 27) {
    const C bu = take(dir3<Q, 1, 1, 1>(), dir3<Q, -1, 1, 1>()), bw = take(dir3<Q, 1, -1, 1>(), dir3<Q, -1, -1, 1>());
    const C tu = take(dir3<Q, 1, 1, -1>(), dir3<Q, -1, 1, -1>()), tw = take(dir3<Q, 1, -1, -1>(), dir3<Q, -1, -1, -1>());
    s[2] = (bu + s[2]) + bw;
    y[2] = bu - bw;
    s[0] = (tu + s[0]) + tw;
    y[0] = tu - tw;
  }
  const C d = (s[2] + s[1]) + s[0];
  return {d, (m & wall_column3<Q>(1)) ? d : -d, (y[2] + y[1]) + y[0], s[2] - s[0]};
}
template <typename C, int Q, int WALL>
__device__ __forceinline__ Moments3<C> wall3(const uint32_t m, const C d, const C (&f)[Q]) {
  if constexpr (WALL == WALL_PAPER) {
    const C u = C(Q == 19 ? 1.0 / 36.0 : 1.0 / 216.0) * d;
    return {C(wall_weight3<Q, 2, 2, 2>(m)) * u,
            C(wall_weight3<Q, 1, 2, 2>(m) - wall_weight3<Q, -1, 2, 2>(m)) * u,
            C(wall_weight3<Q, 2, 1, 2>(m) - wall_weight3<Q, 2, -1, 2>(m)) * u,
            C(wall_weight3<Q, 2, 2, 1>(m) - wall_weight3<Q, 2, 2, -1>(m)) * u};
  } else {
    constexpr uint32_t L = wall_column3<Q>(1), R = wall_column3<Q>(-1);
    if (!__any((m & wall_bits3<Q>() & ~(L | R)) || ((m & L) && (m & R)))) return wall_side3<C, Q>(m, f);
    C v[Q];
    auto take = [&](const int ez) __attribute__((always_inline)) {  // one e_z at a time, for the registers' sake
      if (sizeof(C) == 8) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (k3z[q] == ez) v[q] = (m & wall_bit3<Q>(q)) ? f[q ? ((q - 1) ^ 1) + 1 : 0] : C(0);  // the order pairs e and -e
    };
    constexpr bool WIDE = Q == 27;
    take(1);
    const Plane3<C> b = plane3<WIDE>(group3<C, Q, 1, 1>(v), group3<C, Q, 0, 1>(v), group3<C, Q, -1, 1>(v));
    take(0);
    v[0] = C(0);
    const Plane3<C> c = plane3<true>(group3<C, Q, 1, 0>(v), group3<C, Q, 0, 0>(v), group3<C, Q, -1, 0>(v));
    take(-1);
    const Plane3<C> t = plane3<WIDE>(group3<C, Q, 1, -1>(v), group3<C, Q, 0, -1>(v), group3<C, Q, -1, -1>(v));
    return {(b.s + c.s) + t.s, (b.x + c.x) + t.x, (b.y + c.y) + t.y, b.s - t.s};
  }
}

template <int P>
__device__ __forceinline__ void load3(const Step3Args &a, long i, typename Traits<P>::C &d, typename Traits<P>::C &jx,
                                      typename Traits<P>::C &jy, typename Traits<P>::C &jz) {
  using T = Traits<P>;
  using S = typename T::S;
  using C = typename T::C;
  d = T::dec(static_cast<const S *>(a.src[0])[i]);
  jx = T::dec(static_cast<const S *>(a.src[1])[i]);
  jy = T::dec(static_cast<const S *>(a.src[2])[i]);
  jz = T::dec(static_cast<const S *>(a.src[3])[i]);
  if (T::kScaled) {
    d *= C(a.sc_d);
    jx *= C(a.sc_j);
    jy *= C(a.sc_j);
    jz *= C(a.sc_j);
  }
}

// load3 in two halves: the stored values of node i, and their decoding (the same
// operations in the same order).  k_step3_march keeps a plane's stored values in
// registers while its loads are in flight and decodes them one plane later, so no
// wait for the loads is forced before the current plane is formed.
template <int P>
__device__ __forceinline__ void load3_raw(const Step3Args &a, long i, typename Traits<P>::S &d, typename Traits<P>::S &jx,
                                          typename Traits<P>::S &jy, typename Traits<P>::S &jz) {
  using S = typename Traits<P>::S;
  d = static_cast<const S *>(a.src[0])[i];
  jx = static_cast<const S *>(a.src[1])[i];
  jy = static_cast<const S *>(a.src[2])[i];
  jz = static_cast<const S *>(a.src[3])[i];
}
template <int P>
__device__ __forceinline__ typename Traits<P>::C dec3_d(const Step3Args &a, typename Traits<P>::S v) {
  using C = typename Traits<P>::C;
  C d = Traits<P>::dec(v);
  if (Traits<P>::kScaled) d *= C(a.sc_d);
  return d;
}
template <int P>
__device__ __forceinline__ typename Traits<P>::C dec3_j(const Step3Args &a, typename Traits<P>::S v) {
  using C = typename Traits<P>::C;
  C j = Traits<P>::dec(v);
  if (Traits<P>::kScaled) j *= C(a.sc_j);
  return j;
}

// One thread per node; blocks of 64 x 4 nodes in (x, y), grid (x tiles, y tiles, nz).
template <int P, int Q, bool HASWALL, int WALL>
__global__ void __launch_bounds__(256) k_step3_gather(Step3Args a) {
  using T = Traits<P>;
  using C = typename T::C;
  using S = typename T::S;
  const int x = blockIdx.x * 64 + threadIdx.x;
  const int y = blockIdx.y * 4 + threadIdx.y;
  const int z = blockIdx.z;
  if (x >= a.nx || y >= a.ny) return;
  const long i = (long)z * a.zs + (long)y * a.rs + x;
  if (HASWALL && a.flags[(long)z * a.fzs + (long)y * a.pitch + x] != NODE_FLUID) return;  // held
  const C Fx = C(a.fx), Fy = C(a.fy), Fz = C(a.fz);
  C d0 = C(0), jx0 = C(0), jy0 = C(0), jz0 = C(0);
  if (HASWALL) load3<P>(a, i, d0, jx0, jy0, jz0);
  C arr[Q];
  uint32_t walls = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int sx = wrap_axis(x - k3x[q], a.nx, a.periodic & 1u);
    const int sy = wrap_axis(y - k3y[q], a.ny, a.periodic & 2u);
    const int sz = wrap_axis(z - k3z[q], a.nz, a.periodic & 4u);
    bool solid = sx < 0 || sy < 0 || sz < 0;
    if (HASWALL && !solid) solid = a.flags[(long)sz * a.fzs + (long)sy * a.pitch + sx] == NODE_SOLID;
    arr[q] = C(0);
    if (solid) {
      walls |= wall_bit3<Q>(q);
      continue;
    }
    C d, jx, jy, jz, f[Q];
    load3<P>(a, (long)sz * a.zs + (long)sy * a.rs + sx, d, jx, jy, jz);
    emit3<C, Q>(d, jx + Fx, jy + Fy, jz + Fz, f);
    arr[q] = f[q];
  }
  constexpr bool WIDE = Q == 27;
  const Plane3<C> m = plane3<WIDE>(group3<C, Q, 1, 1>(arr), group3<C, Q, 0, 1>(arr), group3<C, Q, -1, 1>(arr));
  const Plane3<C> c = plane3<true>(group3<C, Q, 1, 0>(arr), group3<C, Q, 0, 0>(arr), group3<C, Q, -1, 0>(arr));
  const Plane3<C> p = plane3<WIDE>(group3<C, Q, 1, -1>(arr), group3<C, Q, 0, -1>(arr), group3<C, Q, -1, -1>(arr));
  C dn = m.s, xn = m.x, yn = m.y, zn = m.s;
  if (HASWALL && walls) {
    C f[Q];
    emit3<C, Q>(d0, jx0 + Fx, jy0 + Fy, jz0 + Fz, f);
    const Moments3<C> w = wall3<C, Q, WALL>(walls, d0, f);
    dn += w.d;
    xn += w.x;
    yn += w.y;
    zn += w.z;
  }
  dn = (dn + c.s) + p.s;
  xn = (xn + c.x) + p.x;
  yn = (yn + c.y) + p.y;
  zn -= p.s;
  if (T::kScaled) {
    dn *= C(a.is_d);
    xn *= C(a.is_j);
    yn *= C(a.is_j);
    zn *= C(a.is_j);
  }
  static_cast<S *>(a.dst[0])[i] = T::enc(dn);
  static_cast<S *>(a.dst[1])[i] = T::enc(xn);
  static_cast<S *>(a.dst[2])[i] = T::enc(yn);
  static_cast<S *>(a.dst[3])[i] = T::enc(zn);
}

// A lane shift whose outermost lane takes `in`.
template <int CTRL> __device__ __forceinline__ int dpp_shift_in(int in, int x) {
  return __builtin_amdgcn_update_dpp(in, x, CTRL, 0xf, 0xf, false);
}
template <int CTRL> __device__ __forceinline__ float dpp_shift_in(float in, float x) {
  return __int_as_float(dpp_shift_in<CTRL>(__float_as_int(in), __float_as_int(x)));
}
template <int CTRL> __device__ __forceinline__ double dpp_shift_in(double in, double x) {
  const long long n = __double_as_longlong(in), b = __double_as_longlong(x);
  const int lo = dpp_shift_in<CTRL>((int)(n & 0xffffffffLL), (int)(b & 0xffffffffLL));
  const int hi = dpp_shift_in<CTRL>((int)(n >> 32), (int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// A block marches along z through a chunk of planes of a tile of 64 columns by GROUPS * RPT
// rows; a wavefront holds RPT rows of 64 columns.  A plane's moments are read once; every
// node's Q emissions are formed once, moved to their target's column by lane shifts and
// summed per (e_y, e_z); the sums over e_y take the rows next to them from registers or,
// between wavefronts, through LDS (one barrier a plane); the three planes that reach a target
// are added as they pass, in seven registers a node.  The moments of the next plane are
// loaded while a plane is worked on.  The outermost row on each side is halo: its sums are
// wrong and not stored.  The column on each side belongs to one more wavefront, which forms
// what these nodes send into the tile one plane ahead of the others and hands it to their
// outermost lanes through LDS.
//
// Grids with walls: a SOLID source sends zeros.  The SOLID bits run two planes ahead of the
// moments, so that a node knows the 26 nodes around it when its emissions are formed, and
// what the wall rule puts in the place of its SOLID sources comes from these emissions.
//
// Why this shape.  It replaces kernels in which every target formed its Q arrivals from
// three planes in LDS: 210 vector operations and 44 LDS instructions a node for D3Q19, now
// 118 and 6 a node formed, halo wavefront included (146 and 7 a node stored at 256^3).  What
// bounds it then is the memory system, not the arithmetic (50 % of the issue rate at 256^3):
// rows that are read by two tiles cost, so tiles are tall (28 rows: 114 us a step at 256^3
// FP32, 26 rows 123, 19 rows 131, 12 rows 155), and loads and stores that start between
// cache lines cost, so tiles are 64 aligned columns and the columns next to them have a
// wavefront of their own (62 columns of 64 lanes, without it: 139-158). The same loads and
// stores with no arithmetic take 110-126 us, a linear copy 88. D3Q19, 256^3, FP32: 128 ->
// 111 us a step (4.8 TB/s); D3Q27 171 -> 122; FP16S D3Q19 102 -> 82; lid-driven box 200 x
// 180 x 150 FP32: 73 -> 50; 64^3 box 51 -> 10; 512^3 1002 -> 913.
constexpr int kMarch3X = 64;  // columns of a tile

// Emissions with e_x = 1 and -1 of one (e_y, e_z) share a slot.
__device__ constexpr int k3slot[27] = {-1, 0, 0, -1, -1, -1, -1, 1, 2, 2, 1, 3, 4, 4, 3, -1, -1, -1, -1,
                                       5, 8, 6, 7, 7, 6, 8, 5};
// How a block goes through the planes.  CHUNK: some of them, and one more on each side.  FLAT: a
// grid of one plane, which is its own neighbour on both sides where the axis is periodic, formed
// once.  RING: all planes of a periodic axis, each formed once; what the first two planes send to
// the targets that the last one completes waits in LDS (9 values a node, 13 with walls).  On thin
// grids the two planes more that a chunk forms are much of its work: 2048 x 2048 x 2 FP32 82 us a
// step in chunks, 65 as a ring, 512 x 512 x 2 9.8 and 8.5 (the rule is in lbt1_3d.hip).
enum March3Form { MARCH3_CHUNK, MARCH3_FLAT, MARCH3_RING };
template <typename C, int Q, int GROUPS, int SIDES, int KEEP>
struct March3Shared {
  static constexpr int kCopies = sizeof(C) == 4 && KEEP == 0 ? 2 : 1;
  static constexpr int kVals = Q == 27 ? 6 : 4;   // of a row for the row below it, and for the row above
  C v[kCopies][2 * kVals][GROUPS * 64];
  alignas(16) C side[2][64 * SIDES][Q == 27 ? 12 : 8];  // left column, then right
  uint8_t solid[4][2][GROUPS * 64];               // by plane: SOLID bits of a wavefront's first and last row
  uint8_t edge[4][64 * SIDES];                    // by plane: SOLID bits of the halo columns
  C keep[KEEP ? KEEP : 1][KEEP ? GROUPS * 64 : 1];  // RING: a column per thread
};

// Wavefronts for the halo columns: 32 rows each.
constexpr int march3_sides(const int rpt, const int groups) { return (rpt * groups + 31) / 32; }

template <int P, int Q, bool HASWALL, int WALL, int RPT, int GROUPS, int WAVES, int FORM>
__global__ void __launch_bounds__(64 * (GROUPS + march3_sides(RPT, GROUPS)), WAVES) k_step3_march(Step3Args a, March3Map m) {
  using T = Traits<P>;
  using C = typename T::C;
  using S = typename T::S;
  constexpr bool WIDE = Q == 27;
  constexpr bool FLAT = FORM == MARCH3_FLAT, RING = FORM == MARCH3_RING;
  constexpr int SIDES = march3_sides(RPT, GROUPS);
  constexpr int KEPT = HASWALL ? 13 : 9;  // values a node keeps (RING)
  using Shared = March3Shared<C, Q, GROUPS, SIDES, RING ? RPT * KEPT : 0>;
  __shared__ Shared sh;
  const int tile = (int)(blockIdx.x & 7) * m.per_xcd + (int)(blockIdx.x >> 3);  // XCD x: a range of tiles
  if (tile >= m.tiles) return;  // uniform across the block
  const int tz = tile / (m.tiles_x * m.tiles_y), rest = tile - tz * m.tiles_x * m.tiles_y;
  const int ty = rest / m.tiles_x, tx = rest - ty * m.tiles_x;
  const int lane = threadIdx.x & 63, grp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int z0 = tz * m.zc, z1 = min(a.nz, z0 + m.zc);
  const bool px = !HASWALL || (a.periodic & 1u), py = !HASWALL || (a.periodic & 2u), pz = !HASWALL || (a.periodic & 4u);
  const C Fx = C(a.fx), Fy = C(a.fy), Fz = C(a.fz);
  auto plane_of = [&](const int z) __attribute__((always_inline)) {  // -1: outside a non-periodic axis
    return z < 0 ? (pz ? a.nz - 1 : -1) : z < a.nz ? z : pz ? 0 : -1;
  };

  // The planes that are formed, from zb to ze: one more than the chunk on each side, but none
  // outside a non-periodic axis (they send nothing).
  const bool shut = HASWALL && !pz;
  const int zb = FLAT || RING ? 0 : shut ? max(z0 - 1, 0) : z0 - 1;
  const int ze = FLAT ? 0 : RING ? a.nz - 1 : shut ? min(z1, a.nz - 1) : z1;

  // The emissions of a node; a SOLID node (NODE_SOLID is the one odd flag) sends zeros, which
  // is what a node with no deviation and no momentum sends.
  static_assert(NODE_SOLID == 1 && NODE_FLUID == 0 && NODE_FIXED == 2, "bit 0: SOLID");
  auto source = [&](const S (&raw)[4], const uint32_t solid, C (&f)[Q]) __attribute__((always_inline)) {
    C d = dec3_d<P>(a, raw[0]), Jx = dec3_j<P>(a, raw[1]) + Fx, Jy = dec3_j<P>(a, raw[2]) + Fy, Jz = dec3_j<P>(a, raw[3]) + Fz;
    if (HASWALL) {
      d = solid ? C(0) : d;
      Jx = solid ? C(0) : Jx;
      Jy = solid ? C(0) : Jy;
      Jz = solid ? C(0) : Jz;
    }
    emit3<C, Q>(d, Jx, Jy, Jz, f);
  };

  if (grp >= GROUPS) {
    const int right = lane >> 5, row = (grp - GROUPS) * 32 + (lane & 31);
    const int wx = wrap_axis(right ? tx * kMarch3X + kMarch3X : tx * kMarch3X - 1, a.nx, px);
    const int wy = wrap_axis(ty * m.oy - 1 + row, a.ny, py);
    const long at = (long)max(wy, 0) * a.rs + max(wx, 0), fat = (long)max(wy, 0) * a.pitch + max(wx, 0);
    S raw[4];
    auto fetch = [&](const int z) __attribute__((always_inline)) {
      load3_raw<P>(a, (long)max(plane_of(z), 0) * a.zs + at, raw[0], raw[1], raw[2], raw[3]);
    };
    auto flag = [&](const int z) __attribute__((always_inline)) {
      const int wz = plane_of(min(z, z1));
      return a.flags[(long)max(wz, 0) * a.fzs + fat] | (uint32_t)(wz < 0 || wy < 0 || wx < 0);
    };
    auto edge = [&](const int z, const uint32_t f) __attribute__((always_inline)) {
      sh.edge[z & 3][right * 32 * SIDES + row] = f & 1u;
    };
    uint32_t ahead = 0;
    (void)flag;
    (void)ahead;
    (void)edge;
    auto send = [&](const int z) __attribute__((always_inline)) {
      C(*const o)[Q == 27 ? 12 : 8] = sh.side[(z - z0 + 1) & 1];
      C f[Q];
      source(raw, HASWALL && sh.edge[z & 3][right * 32 * SIDES + row], f);
      auto put = [&](const int slot, const C l, const C r) __attribute__((always_inline)) {
        o[right * 32 * SIDES + row][slot] = right ? r : l;
      };
      put(0, f[1], f[2]);
      put(1, f[7], f[10]);
      put(2, f[9], f[8]);
      put(3, f[11], f[14]);
      put(4, f[13], f[12]);
      if constexpr (Q == 27) {
        put(5, f[19], f[26]);
        put(6, f[21], f[24]);
        put(7, f[23], f[22]);
        put(8, f[25], f[20]);
      }
    };
    fetch(zb);
    if constexpr (HASWALL) {
      // (all loads before the first wait)
      const uint32_t f3 = RING ? flag(zb - 1) : 0u, f0 = flag(zb), f1 = FLAT ? 0u : flag(zb + 1), f2 = FLAT ? 0u : flag(zb + 2);
      if (!FLAT) ahead = flag(zb + 3);
      if (RING) edge(zb - 1, f3);
      edge(zb, f0);
      if (!FLAT) {
        edge(zb + 1, f1);
        edge(zb + 2, f2);
      }
    }
    send(zb);
    fetch(min(zb + 1, ze));
    __syncthreads();
    if (HASWALL) __syncthreads();
    for (int z = zb; z <= ze; ++z) {
      if (z < ze) send(z + 1);
      fetch(min(z + 2, ze));
      if constexpr (HASWALL && !FLAT) {
        edge(z + 3, ahead);
        ahead = flag(z + 4);
      }
      __syncthreads();
      if (Shared::kCopies == 1) __syncthreads();
    }
    return;
  }

  const int x = tx * kMarch3X + lane, y0 = ty * m.oy - 1 + grp * RPT;
  const int at = threadIdx.x;
  const int above = grp > 0 ? at - 64 : at, below = grp < GROUPS - 1 ? at + 64 : at;
  // Each row's offset in a plane, in bytes (FP64, whose planes can pass 4 GB: in values), and
  // the rows outside a non-periodic axis.
  constexpr uint32_t kUnit = sizeof(S) == 8 ? 1 : sizeof(S);
  const int wx = wrap_axis(x, a.nx, px);
  uint32_t off[RPT];
  constexpr uint32_t kNowhere = 0x40000000u;
  uint32_t foff[HASWALL ? RPT : 1], to[RPT], out[HASWALL ? RPT : 1];  // to: in the rows of the tile, in bytes
  (void)foff;
  (void)out;
  int wy = wrap_axis(y0, a.ny, py);
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int r = grp * RPT + i;
    if (i) wy = py ? (wy + 1 == a.ny ? 0 : wy + 1) : (y0 + i >= 0 && y0 + i < a.ny ? y0 + i : -1);
    off[i] = ((uint32_t)max(wy, 0) * (uint32_t)a.rs + (uint32_t)max(wx, 0)) * kUnit;
    if (HASWALL) {
      foff[i] = (uint32_t)max(wy, 0) * (uint32_t)a.pitch + (uint32_t)max(wx, 0);
      out[i] = wy < 0 || wx < 0;
    }
    to[i] = x < a.nx && r >= 1 && r <= m.oy && y0 + i < a.ny ? ((uint32_t)(r - 1) * (uint32_t)a.rs + (uint32_t)x) * sizeof(S) : kNowhere;
  }
  S raw[RPT][4];
  uint32_t fl[RPT];
  auto fetch = [&](const int i, const int z) __attribute__((always_inline)) {
    const int wz = plane_of(z);
    const long zo = (long)max(wz, 0) * a.zs * (long)sizeof(S);
#pragma unroll
    for (int v = 0; v < 4; ++v)
      raw[i][v] = *reinterpret_cast<const S *>(static_cast<const char *>(a.src[v]) + zo +
                                               (size_t)off[i] * (sizeof(S) / kUnit));
  };
  auto fetch_flag = [&](const int i, const int z) __attribute__((always_inline)) {
    const int wz = plane_of(min(z, z1));
    const uint32_t f = (a.flags + (long)max(wz, 0) * a.fzs)[foff[i]];
    return f | out[i] | (uint32_t)(wz < 0);
  };
  (void)fetch_flag;

  // per row: sums of the planes below and at the target (density, x, y; density of the plane
  // below alone), and of the newest plane for the next target
  C cs[RPT] = {}, cx[RPT] = {}, cy[RPT] = {}, cm[RPT] = {}, ns[RPT] = {}, nx[RPT] = {}, ny[RPT] = {};
  C nz[HASWALL ? RPT : 1] = {};          // as ns, for z: a wall adds to it by itself
  uint32_t near[HASWALL ? RPT : 1];      // SOLID bits around the newest plane's nodes
  uint32_t held[HASWALL ? RPT : 1] = {}; // bits of nodes that are not FLUID, by plane
  (void)nz;
  (void)near;
  (void)held;

  // Every store is issued: rows and planes that are not this block's go past the end of the
  // buffer, where the hardware drops them.  The number of stores after the loads of a plane
  // is then known and the wait for a load is not one for the stores issued after it; nor do
  // branches part the rows (95 registers instead of 113 with three rows a thread).
  auto put = [&](const auto past, const bool live, const int z, const uint32_t o, const C (&value)[4])
      __attribute__((always_inline)) {
    constexpr int kHint = decltype(past)::value ? 2 : 0;  // 2: non-temporal
    const long row0 = ((long)z * a.zs + (long)(ty * m.oy) * a.rs) * (long)sizeof(S);
    const int bytes = live ? (int)((uint32_t)(RPT * GROUPS) * (uint32_t)a.rs * sizeof(S)) : 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const __amdgpu_buffer_rsrc_t b =
          __builtin_amdgcn_make_buffer_rsrc(static_cast<char *>(a.dst[v]) + row0, 0, bytes, 0x00027000);
      const S e = T::enc(value[v]);
      if constexpr (sizeof(S) == 8) {
        typedef int pair __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(pair, e), b, o, 0, kHint);
      } else if constexpr (sizeof(S) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, e), b, o, 0, kHint);
      } else {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, e), b, o, 0, kHint);
      }
    }
  };

  // the sums of one row of plane z: lo e_z = -1 (completes the target below), mid 0, hi 1
  auto finish = [&](const int i, const int zn, const Plane3<C> &lo, const Plane3<C> &mid, const Plane3<C> &hi)
      __attribute__((always_inline)) {
    const int z = FLAT ? 1 : zn;
    if constexpr (FLAT) {
      const C h = HASWALL ? hi.s + ns[i] : hi.s, hx = HASWALL ? hi.x + nx[i] : hi.x, hy = HASWALL ? hi.y + ny[i] : hi.y;
      cs[i] = h + mid.s;
      cx[i] = hx + mid.x;
      cy[i] = hy + mid.y;
      cm[i] = HASWALL ? hi.s + nz[i] : hi.s;
    }
    if constexpr (RING) {
      // plane 0 completes the last target and begins target 0 (nothing was sent up to it yet:
      // ns ... nz hold what its walls stand for), plane 1 completes target 0
      auto keep = [&](const int k, const C v) __attribute__((always_inline)) { sh.keep[i * KEPT + k][at] = v; };
      if (z == 0) {
        keep(0, lo.s);
        keep(1, lo.x);
        keep(2, lo.y);
        keep(3, mid.s);
        keep(4, mid.x);
        keep(5, mid.y);
        if (HASWALL) {
          keep(9, ns[i]);
          keep(10, nx[i]);
          keep(11, ny[i]);
          keep(12, nz[i]);
        }
      } else if (z == 1) {
        keep(6, lo.s);
        keep(7, lo.x);
        keep(8, lo.y);
      }
    }
    C o[4] = {cs[i] + lo.s, cx[i] + lo.x, cy[i] + lo.y, cm[i] - lo.s};
    cs[i] = ns[i] + mid.s;
    cx[i] = nx[i] + mid.x;
    cy[i] = ny[i] + mid.y;
    cm[i] = HASWALL ? nz[i] : ns[i];
    ns[i] = hi.s;
    nx[i] = hi.x;
    ny[i] = hi.y;
    // SOLID and FIXED nodes are not stored
    const uint32_t o_at = HASWALL ? (FLAT ? held[i] : held[i] >> 3 & 1u) << 30 | to[i] : to[i];
    if (T::kScaled) {
      o[0] *= C(a.is_d);
      o[1] *= C(a.is_j);
      o[2] *= C(a.is_j);
      o[3] *= C(a.is_j);
    }
    const bool live = RING ? z > 1 : z > z0;
    const int target = RING && z > a.nz ? 0 : z - 1;
    if (sizeof(S) < 8 && m.past)
      put(std::true_type{}, live, target, o_at, o);
    else
      put(std::false_type{}, live, target, o_at, o);
  };

#pragma unroll
  for (int i = 0; i < RPT; ++i) fetch(i, zb);
  // SOLID bits of plane z (its flags are in fl): a row's right, own and left column, then the
  // nine around each node
  uint32_t row[RPT + 2];
  (void)row;
  auto row_bits = [&](const int i, const int z) __attribute__((always_inline)) {
    const int b = fl[i] & 1u, h = sh.edge[z & 3][(lane & 32) * SIDES + grp * RPT + i];
    row[i + 1] = (uint32_t)b << 1 | (uint32_t)dpp_shift_in<kDppWaveShl1>(h, b) |
                 (uint32_t)dpp_shift_in<kDppWaveShr1>(h, b) << 2;
    held[i] = held[i] << 1 | (uint32_t)(fl[i] != NODE_FLUID);
    if (i == 0) sh.solid[z & 3][0][at] = (uint8_t)row[1];
    if (i == RPT - 1) sh.solid[z & 3][1][at] = (uint8_t)row[RPT];
  };
  auto nine_bits = [&](const int z) __attribute__((always_inline)) {  // after a barrier
    row[0] = sh.solid[z & 3][1][above];
    row[RPT + 1] = sh.solid[z & 3][0][below];
    // sources of e_y = -1 in the row after, of e_y = 1 in the row before; older planes are
    // shifted out of the bits that are looked at
#pragma unroll
    for (int i = 0; i < RPT; ++i) near[i] = near[i] << 9 | (row[i + 2] | row[i + 1] << 3 | row[i] << 6);
  };
  (void)row_bits;
  (void)nine_bits;
  if constexpr (HASWALL) {
    // RING: the plane before the first is the last one
    const int zf = RING ? zb - 1 : zb;
    uint32_t next[RPT], third[RPT], fourth[RPT], first[RPT + 2];  // (all loads before the first wait)
    (void)third;
    (void)fourth;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      near[i] = 0x1ffu;  // outside; a periodic axis has no target here
      fl[i] = fetch_flag(i, zf);
      next[i] = fetch_flag(i, zf + 1);
      if (!FLAT) third[i] = fetch_flag(i, zf + 2);
      if (RING) fourth[i] = fetch_flag(i, zf + 3);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPT; ++i) row_bits(i, zf);
#pragma unroll
    for (int i = 0; i < RPT + 2; ++i) first[i] = row[i];
    if constexpr (!FLAT) {
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        fl[i] = next[i];
        row_bits(i, zf + 1);
        next[i] = row[i + 1];
      }
      if constexpr (RING) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
          fl[i] = third[i];
          row_bits(i, zf + 2);
          third[i] = row[i + 1];
        }
      }
#pragma unroll
      for (int i = 0; i < RPT; ++i) row[i + 1] = first[i + 1];
    }
    __syncthreads();
    nine_bits(zf);
    if constexpr (FLAT) {
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const uint32_t nine = near[i] & 0x1ffu;
        near[i] = shut ? 0x1ffu << 18 | nine << 9 | 0x1ffu : nine << 18 | nine << 9 | nine;
      }
    } else {
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        row[i + 1] = next[i];
        if (!RING) fl[i] = third[i];
      }
      nine_bits(zf + 1);
      if constexpr (RING) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
          row[i + 1] = third[i];
          fl[i] = fourth[i];
        }
        nine_bits(zf + 2);
      }
    }
  } else {
    __syncthreads();
  }
  for (int z = zb; z <= ze; ++z) {
    const int par = (z - z0 + 1) & 1;
    C(*const e)[GROUPS * 64] = sh.v[Shared::kCopies == 2 ? par : 0];
    // three e_z (index e_z + 1) of e_y = 1 (up), 0 (l) and -1 (w)
    Group3<C> up[3], l0[3], w1[3], ps[3];
    C pu[3];
    static_assert(RPT > 1, "the first and the last row of a thread are different rows");
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      __builtin_amdgcn_sched_barrier(0);  // one row's temporaries at a time
      const C *const side = sh.side[par][(lane & 32) * SIDES + grp * RPT + i];
      C f[Q];
      source(raw[i], HASWALL ? near[i] >> 13 & 1u : 0u, f);
      if constexpr (HASWALL) {
        nz[i] = ns[i];
        // (half-way: a SOLID node takes nothing in, and its neighbours would send the lanes beside it
        // the long way)
        const uint32_t walls =
            WALL == WALL_HALFWAY && (near[i] >> 13 & 1u) ? 0u : near[i] & wall_bits3<Q>();
        if (walls) {
          const Moments3<C> w = wall3<C, Q, WALL>(walls, dec3_d<P>(a, raw[i][0]), f);
          ns[i] += w.d;
          nx[i] += w.x;
          ny[i] += w.y;
          nz[i] += w.z;
        }
        if constexpr (!FLAT) {
          row_bits(i, z + 2);
          fl[i] = fetch_flag(i, z + 3);
        }
      }
      fetch(i, min(z + 1, ze));
#pragma unroll
      for (int q = 0; q < Q; ++q)
        f[q] = k3x[q] == 1    ? dpp_shift_in<kDppWaveShr1>(side[k3slot[q]], f[q])
               : k3x[q] == -1 ? dpp_shift_in<kDppWaveShl1>(side[k3slot[q]], f[q])
                              : f[q];
      if (FLAT && shut) {  // the planes on both sides are outside
#pragma unroll
        for (int q = 0; q < Q; ++q)
          if (k3z[q]) f[q] = C(0);
      }
      const Group3<C> w[3] = {group3<C, Q, -1, -1>(f), group3<C, Q, -1, 0>(f), group3<C, Q, -1, 1>(f)};
      const Group3<C> l[3] = {group3<C, Q, 0, -1>(f), group3<C, Q, 0, 0>(f), group3<C, Q, 0, 1>(f)};
      if (i == 0) {
        e[0][at] = w[0].s;
        e[1][at] = w[1].s;
        e[2][at] = w[2].s;
        e[3][at] = w[1].x;
        if (WIDE) {
          e[4][at] = w[0].x;
          e[5][at] = w[2].x;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) l0[k] = l[k];
      } else {
        if (i == 1) {
#pragma unroll
          for (int k = 0; k < 3; ++k) w1[k] = w[k];
        } else {
          Plane3<C> t[3];
#pragma unroll
          for (int k = 0; k < 3; ++k) t[k] = {ps[k].s + w[k].s, WIDE || k == 1 ? ps[k].x + w[k].x : ps[k].x, pu[k] - w[k].s};
          finish(i - 1, z, t[0], t[1], t[2]);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          ps[k].s = up[k].s + l[k].s;
          ps[k].x = WIDE || k == 1 ? up[k].x + l[k].x : l[k].x;
          pu[k] = up[k].s;
        }
      }
      up[0] = group3<C, Q, 1, -1>(f);
      up[1] = group3<C, Q, 1, 0>(f);
      up[2] = group3<C, Q, 1, 1>(f);
    }
    constexpr int V = Shared::kVals;
    e[V][at] = up[0].s;
    e[V + 1][at] = up[1].s;
    e[V + 2][at] = up[2].s;
    e[V + 3][at] = up[1].x;
    if (WIDE) {
      e[V + 4][at] = up[0].x;
      e[V + 5][at] = up[2].x;
    }
    __syncthreads();
    if constexpr (HASWALL && !FLAT) nine_bits(z + 2);
    {
      const Group3<C> ua[3] = {{e[V][above], WIDE ? e[V + (WIDE ? 4 : 0)][above] : C(0)},
                               {e[V + 1][above], e[V + 3][above]},
                               {e[V + 2][above], WIDE ? e[V + (WIDE ? 5 : 0)][above] : C(0)}};
      finish(0, z, plane3<WIDE>(ua[0], l0[0], w1[0]), plane3<true>(ua[1], l0[1], w1[1]), plane3<WIDE>(ua[2], l0[2], w1[2]));
    }
    {
      const Group3<C> wb[3] = {{e[0][below], WIDE ? e[WIDE ? 4 : 0][below] : C(0)},
                               {e[1][below], e[3][below]},
                               {e[2][below], WIDE ? e[WIDE ? 5 : 0][below] : C(0)}};
      Plane3<C> t[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) t[k] = {ps[k].s + wb[k].s, WIDE || k == 1 ? ps[k].x + wb[k].x : ps[k].x, pu[k] - wb[k].s};
      finish(RPT - 1, z, t[0], t[1], t[2]);
    }
    if (Shared::kCopies == 1) __syncthreads();
  }
  if constexpr (RING) {
    const Plane3<C> none = {C(0), C(0), C(0)};
    auto kept = [&](const int i, const int k) __attribute__((always_inline)) { return sh.keep[i * KEPT + k][at]; };
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      if (HASWALL) {
        held[i] <<= 1;
        nz[i] = ns[i] + kept(i, 12);
        ns[i] += kept(i, 9);
        nx[i] += kept(i, 10);
        ny[i] += kept(i, 11);
      }
      finish(i, a.nz, {kept(i, 0), kept(i, 1), kept(i, 2)}, {kept(i, 3), kept(i, 4), kept(i, 5)}, none);
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      if (HASWALL) held[i] <<= 1;
      finish(i, a.nz + 1, {kept(i, 6), kept(i, 7), kept(i, 8)}, none, none);
    }
    return;
  }
  if (!FLAT && shut && z1 == a.nz) {
    const Plane3<C> none = {C(0), C(0), C(0)};
#pragma unroll
    for (int i = 0; i < RPT; ++i) held[i] <<= 1;
#pragma unroll
    for (int i = 0; i < RPT; ++i) finish(i, a.nz, none, none, none);
  }
}

struct Reduce3Args {
  const void *cur[4];
  void *snap[4];
  const uint8_t *flags;
  int nx, ny, nz, pitch;
  long rs, zs, fzs;
  double sc_d, sc_j;
  uint32_t what;
  double *partials;  // 8 per block
};

template <typename S, int V>
struct alignas(V * sizeof(S)) Run3 {
  S v[V];
};

// out slots: 0 sum d, 1..3 sum j, 4 max residual, 5 non-finite, 6 FLUID count
// Bound by HBM: with the residual the state and the snapshot are read and the snapshot is
// written.  A thread takes 16 bytes of each field at a time and steps to its next run by adding
// the grid's stride in rows and runs.  256^3 FP32 (805 MB): 143 us, 5.6 TB/s; a value at a
// time, with two 64-bit divisions each, 205.  The box of 200 x 180 x 150: 67 -> 48.
template <int P>
__global__ void __launch_bounds__(256) k_reduce3_partial(Reduce3Args a) {
  using T = Traits<P>;
  using S = typename T::S;
  constexpr int V = 16 / sizeof(S);
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const bool want_res = a.what & 4u;
  // rows are pitch values (a multiple of 64) apart in every field, so a row's last run
  // stays inside it
  const int runs = (a.nx + V - 1) / V;
  const long rows = (long)a.ny * a.nz;
  const int stride = gridDim.x * blockDim.x, first = blockIdx.x * blockDim.x + threadIdx.x;
  int run = first % runs;
  long row = first / runs;
  while (row < rows) {
    const int x = run * V;
    const long i = row * a.rs + x;
    Run3<S, V> r[4], s[4];
    Run3<uint8_t, V> fl;
#pragma unroll
    for (int m = 0; m < 4; ++m) r[m] = *reinterpret_cast<const Run3<S, V> *>(static_cast<const S *>(a.cur[m]) + i);
    if (a.flags) fl = *reinterpret_cast<const Run3<uint8_t, V> *>(a.flags + row * a.pitch + x);
    if (want_res) {
#pragma unroll
      for (int m = 0; m < 4; ++m) s[m] = *reinterpret_cast<const Run3<S, V> *>(static_cast<const S *>(a.snap[m]) + i);
    }
#pragma unroll
    for (int k = 0; k < V; ++k) {
      if (x + k >= a.nx || (a.flags && fl.v[k] != NODE_FLUID)) continue;
      double v[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) v[m] = (double)T::dec(r[m].v[k]) * (m == 0 ? a.sc_d : a.sc_j);
#pragma unroll
      for (int m = 0; m < 4; ++m) acc[m] += v[m];
      const bool fin = __builtin_isfinite(v[0]) && __builtin_isfinite(v[1]) && __builtin_isfinite(v[2]) &&
                       __builtin_isfinite(v[3]);
      acc[5] += fin ? 0.0 : 1.0;
      acc[6] += 1.0;
      if (want_res) {
        const double rho = 1.0 + v[0];
        const double sr = 1.0 + (double)T::dec(s[0].v[k]) * a.sc_d;
        double res = 0.0;
#pragma unroll
        for (int m = 1; m < 4; ++m) {
          const double su = (double)T::dec(s[m].v[k]) * a.sc_j / sr;
          res = __builtin_fmax(res, __builtin_fabs(v[m] / rho - su));
        }
        acc[4] = __builtin_fmax(acc[4], res);
#pragma unroll
        for (int m = 0; m < 4; ++m) s[m].v[k] = r[m].v[k];
      }
    }
    if (want_res) {
#pragma unroll
      for (int m = 0; m < 4; ++m) *reinterpret_cast<Run3<S, V> *>(static_cast<S *>(a.snap[m]) + i) = s[m];
    }
    run += stride % runs;
    row += stride / runs;
    if (run >= runs) {
      run -= runs;
      ++row;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const double o = __shfl_xor(acc[m], off);
      acc[m] = m == 4 ? __builtin_fmax(acc[m], o) : acc[m] + o;
    }
  }
  __shared__ double part[4][8];
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
    for (int m = 0; m < 8; ++m) part[wave][m] = acc[m];
  __syncthreads();
  if (threadIdx.x < 8) {
    const int m = threadIdx.x;
    double v = part[0][m];
    for (int w = 1; w < 4; ++w) v = m == 4 ? __builtin_fmax(v, part[w][m]) : v + part[w][m];
    a.partials[blockIdx.x * 8 + m] = v;
  }
}

// one wavefront: lane l combines partial rows l, l + 64, ... in index order, then a
// fixed butterfly over the lanes (slot 4 is a maximum, the others sums)
__global__ void __launch_bounds__(64) k_reduce3_final(const double *partials, int nparts, double *out) {
  const int l = threadIdx.x;
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int b = l; b < nparts; b += 64) {
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const double x = partials[b * 8 + m];
      acc[m] = m == 4 ? __builtin_fmax(acc[m], x) : acc[m] + x;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const double o = __shfl_xor(acc[m], off);
      acc[m] = m == 4 ? __builtin_fmax(acc[m], o) : acc[m] + o;
    }
  }
  if (l == 0) {
#pragma unroll
    for (int m = 0; m < 8; ++m) out[m] = acc[m];
  }
}

}  // namespace lbt1
