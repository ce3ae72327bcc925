// Instantiations of the resident-tile kernels (tile2d.h): two tile shapes for
// every 2D stencil they cover.
#include "tile2d.h"

namespace s5d {
namespace {

// Tile shapes.  0: 64 rows x 64 columns, one column per lane, for grids that
// would not fill the machine with wider tiles; 1: 64 rows x 128 columns, less
// overlap.  Radius 3 and 4 hold 8 rows a wave in both (the exchanged rows of
// 16 waves would take most of the LDS).  Measured (T = 100; shape 0 / shape 1,
// best depth each): float64 5-point star 512^2 80 / 97 us, 1024^2 147 / 116,
// 4096^2 1279 / 897; float32 25-point box 512^2 167 / 198, 2048^2 883 / 629.
// 32 x 64 and 64 x 256 tiles gain at most 6 % on some sizes and are not built.
template <typename T, int ACC, int EXPR, int R, bool BOX, int CPL, int M, int NW>
TileKernel2D make() {
  // instructions of a wave's step: the terms, the lane shifts (two moves per
  // double) and about 20 for the exchange and the loop
  constexpr int words = sizeof(T) / 4;
  constexpr int term = ACC ? 10 : 1;
  constexpr int cell = EXPR == EXPR_GRADIENT ? 45 : term * npts(2, R, BOX) + (EXPR == EXPR_DIV ? 8 : 0);
  constexpr int instr = M * CPL * cell + (BOX ? M + 2 * R : M) * 2 * R * words + 20;
  // the wide float64 tiles of radius >= 2 take so many registers that a CU
  // holds one workgroup: nothing overlaps its exchange (measured a quarter)
  constexpr int clocks = instr * NW * (words == 2 && R >= 2 && CPL == 2 ? 5 : 4) / 4;
  // gradient2d is not batched: its streaming kernels have no batched entry point
  if constexpr (EXPR == EXPR_GRADIENT)
    return TileKernel2D{&launch_tile2d<T, ACC, EXPR, R, BOX, CPL, M, NW>, nullptr, nullptr, 0, NW * M, 64 * CPL, clocks};
  else
    return TileKernel2D{&launch_tile2d<T, ACC, EXPR, R, BOX, CPL, M, NW>,
                        &fill_tile2d<T, EXPR, R, BOX, CPL, M, NW>,
                        &launch_tile2d_batch<T, ACC, EXPR, R, BOX, CPL, M, NW>,
                        static_cast<int>(sizeof(TileItem2D<T, ncoef(2, R, BOX, EXPR)>)),
                        NW * M,
                        64 * CPL,
                        clocks};
}

template <typename T, int ACC, int EXPR, int R, bool BOX>
const TileKernel2D* shapes(int shape) {
  static const TileKernel2D k[2] = {make<T, ACC, EXPR, R, BOX, 1, R <= 2 ? 4 : 8, R <= 2 ? 16 : 8>(),
                                    make<T, ACC, EXPR, R, BOX, 2, 8, 8>()};
  return &k[shape];
}

template <typename T, int ACC>
const TileKernel2D* linear(int r, bool box, int shape) {
  switch (r * 2 + box) {
    case 2: return shapes<T, ACC, EXPR_LINEAR, 1, false>(shape);
    case 3: return shapes<T, ACC, EXPR_LINEAR, 1, true>(shape);
    case 4: return shapes<T, ACC, EXPR_LINEAR, 2, false>(shape);
    case 5: return shapes<T, ACC, EXPR_LINEAR, 2, true>(shape);
    case 6: return shapes<T, ACC, EXPR_LINEAR, 3, false>(shape);
    case 8: return shapes<T, ACC, EXPR_LINEAR, 4, false>(shape);
    default: return nullptr;
  }
}

template <typename T>
const TileKernel2D* expression(int expr, int r, bool box, int shape) {
  if (expr == EXPR_GRADIENT) return r == 1 && !box ? shapes<T, 0, EXPR_GRADIENT, 1, false>(shape) : nullptr;
  if (expr != EXPR_DIV) return nullptr;
  switch (r * 2 + box) {
    case 2: return shapes<T, 0, EXPR_DIV, 1, false>(shape);
    case 3: return shapes<T, 0, EXPR_DIV, 1, true>(shape);
    case 4: return shapes<T, 0, EXPR_DIV, 2, false>(shape);
    default: return nullptr;
  }
}

}  // namespace

const TileKernel2D* tile_kernel2d(int kind, int expr, int r, bool box, int shape) {
  if (shape < 0 || shape >= kTileShapes2D) return nullptr;
  if (expr != EXPR_LINEAR) {
    if (kind == KIND_F32) return expression<float>(expr, r, box, shape);
    if (kind == KIND_F64) return expression<double>(expr, r, box, shape);
    return nullptr;
  }
  if (kind == KIND_F32) return linear<float, 0>(r, box, shape);
  if (kind == KIND_F64) return linear<double, 0>(r, box, shape);
  if (kind == KIND_F32_COMP) return linear<float, 1>(r, box, shape);
  return nullptr;
}

}  // namespace s5d
