// Host-side interface of the resident-tile kernels (tile2d.h) for small 2D
// grids.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "s5d_internal.h"

namespace s5d {

// One tile shape of one stencil.  The depth of a launch is an argument.
struct TileKernel2D {
  hipError_t (*launch)(const Round2D&, int bt);
  int (*fill_item)(void* item, const Round2D&, int bt);  // returns the grid's workgroups
  LaunchBatchFn launch_batch;                            // null (and fill_item): not batched
  int item_bytes;
  int rows, cols;   // tile, overlap included
  int step_clocks;  // clocks of vector issue one workgroup's step takes of a CU (an estimate)
};

constexpr int kTileShapes2D = 2;

// The kernel of a tile shape (0 .. kTileShapes2D - 1), or null if the stencil
// has none: stars of radius 1..4 and boxes of radius 1 and 2 of every kernel
// kind, the quotient stencils and gradient2d in float32 and float64.
const TileKernel2D* tile_kernel2d(int kind, int expr, int r, bool box, int shape);

}  // namespace s5d
