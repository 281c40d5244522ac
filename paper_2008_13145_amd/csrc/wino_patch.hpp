// Input patch of one Winograd tile, as host and device code.
#pragma once
#include <hip/hip_runtime.h>

namespace kt {

// v = the 4x4 patch of an H x W image whose upper left corner is (y0, x0), zero
// where it lies in the padding.  `at(y, x)` loads a position; it is asked for
// positions inside the image only.  Every position is clamped into the image
// and what lies in the padding is cleared after it, so no branch stands
// between the 16 loads.  An image without rows or columns (its outputs lie in
// the padding alone) has no inside, hence no loads.
template <typename V, typename I, typename Load>
__host__ __device__ __forceinline__ void wino_patch(I H, I W, I y0, I x0, V zero, Load at, V (&v)[4][4]) {
  if (H > 0 && W > 0) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const I y = y0 + u, x = x0 + w;
        const I yc = y < 0 ? 0 : y, xc = x < 0 ? 0 : x;
        v[u][w] = at(yc < H - 1 ? yc : H - 1, xc < W - 1 ? xc : W - 1);
      }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (y0 + u < 0 || y0 + u >= H || x0 + w < 0 || x0 + w >= W) v[u][w] = zero;
}

}  // namespace kt
