// Launch arguments of the tile kernels.
#pragma once
#include "lbt1_args.hpp"

namespace lbt1 {

// Tiles of k_step_tile, k_bgk_tile and k_sc_tile: steps this launch takes, halo and stored
// nodes of a tile on each axis, tiles per row of tiles, in all and per XCD (8 * per_xcd blocks).
struct TileMap {
  int steps;
  int hx, hy, ox, oy;
  int tiles_x, tiles, per_xcd;
};

}  // namespace lbt1
