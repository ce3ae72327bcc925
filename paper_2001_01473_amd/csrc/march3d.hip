// Instantiations of the marching kernel (march3d.h) for 3D stars.
#include "march.h"
#include "march3d.h"

namespace s5d {
namespace {

template <typename T, int R, int CPL, int M, int NW>
Kernel3D make() {
  return Kernel3D{&launch_march3d<T, 0, R, CPL, M, NW>,
                  &occupancy_march3d<T, 0, R, CPL, M, NW>,
                  CPL,
                  NW * M,
                  1,
                  1,
                  &fill_march3d<T, 0, R, CPL, M, NW>,
                  &launch_march3d_batch<T, 0, R, CPL, M, NW>,
                  static_cast<int>(sizeof(MarchItem3D<T, npts(3, R, false)>))};
}

}  // namespace

// Tiles: 32 rows of 8 waves by 128 columns, but 64 columns at radius 4 (and 16
// waves in float32), whose pending planes then leave room for more waves.
// Measured at 420 x 512 x 483 (us a step, row streaming -> this): float32
// radius 2 358 -> 184, 3 607 -> 253, 4 1095 -> 247; float64 651 -> 330, 912 ->
// 358, 1730 -> 441.  At 512^3, where row streaming has no ragged rows: float32
// 315 -> 335, 411 -> 323, 510 -> 325; float64 596 -> 560, 756 -> 547, 906 -> 524.
Kernel3D march_kernel3d(int kind, int r) {
  if (kind == KIND_F32) {
    if (r == 2) return make<float, 2, 2, 4, 8>();
    if (r == 3) return make<float, 3, 2, 4, 8>();
    if (r == 4) return make<float, 4, 1, 4, 16>();
  } else if (kind == KIND_F64) {
    if (r == 2) return make<double, 2, 2, 4, 8>();
    if (r == 3) return make<double, 3, 2, 4, 8>();
    if (r == 4) return make<double, 4, 1, 4, 8>();
  }
  return Kernel3D{};
}

}  // namespace s5d
