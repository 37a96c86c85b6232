// Device code shared by the kernels that rasterize tetrahedra.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace morea {

// Exact x-interval update for one face: the j with A j + b > 0.  The FP64
// quotient estimate is corrected by one exact evaluation on each side; T is
// double (exact for extents <= 2^16) or int64.
template <typename T>
__device__ __forceinline__ void clip_face(int kind, T A, double invA, T b, int W, int& js, int& je) {
  if (kind > 0) {
    const double t = fmin(fmax(-static_cast<double>(b) * invA, -2.0), W + 1.0);
    int j = static_cast<int>(floor(t)) + 1;
    if (A * static_cast<T>(j) + b <= 0) j += 1;
    else if (A * static_cast<T>(j - 1) + b > 0) j -= 1;
    js = max(js, j);
  } else if (kind < 0) {
    const double t = fmin(fmax(-static_cast<double>(b) * invA, -2.0), W + 1.0);
    int j = static_cast<int>(ceil(t)) - 1;
    if (A * static_cast<T>(j) + b <= 0) j -= 1;
    else if (A * static_cast<T>(j + 1) + b > 0) j += 1;
    je = min(je, j);
  } else if (!(b > 0)) {
    je = -1;
  }
}

}  // namespace morea
