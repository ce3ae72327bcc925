// Host-side interface of the marching one-step kernels (march3d.h).
#pragma once

#include "s5d_internal.h"

namespace s5d {

// The marching kernel of a plain 3D star of radius 2..4 (launch null for other
// kinds and radii): tiles of m * nw rows by 64 * cpl columns; a round's chunk is
// the planes of a block.
Kernel3D march_kernel3d(int kind, int r);

}  // namespace s5d
