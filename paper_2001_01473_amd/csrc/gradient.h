// gradient2d's update of one cell (device code).
#pragma once

#include "kcommon.h"

namespace s5d {

// cc*f + 1/sqrt(c0 + sum_n (f - f_n)^2) over the four axis neighbours in
// canonical order (AN5D Table 3), every operation rounded on its own.
template <typename T>
__device__ __forceinline__ T gradient_cell(T cc, T c0, T f, T up, T left, T right, T down) {
#pragma clang fp contract(off)
  T s2 = c0;
  T d = f - up;
  s2 = s2 + d * d;
  d = f - left;
  s2 = s2 + d * d;
  d = f - right;
  s2 = s2 + d * d;
  d = f - down;
  s2 = s2 + d * d;
  const T root = ieee_sqrt(s2);
  const T q = T(1) / root;
  return cc * f + q;
}

}  // namespace s5d
