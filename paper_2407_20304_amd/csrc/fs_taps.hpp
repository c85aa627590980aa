// Tap positions of the Fourier-slice gridding, shared by the forward and the
// transpose (and by host checks).
#pragma once
#include <hip/hip_runtime.h>
#include <cmath>

namespace holo {

constexpr int kFsWidth = 8;        // gridding kernel taps per axis

// Position of a polar sample along one axis (grid units, frequency zero at
// M/2): first of its taps and the distance of the sample from it, in double
// precision.  Taps start at floor(pos) - kFsWidth/2 + 1, so every distance lies
// in (-kFsWidth/2, kFsWidth/2].
struct FsTap {
  int i0;
  double r;
};
__host__ __device__ inline FsTap fs_tap(int m, double step, int M) {
  const double gx = (double)m * step, fl = floor(gx);
  FsTap t;
  t.i0 = (int)fl - kFsWidth / 2 + 1 + M / 2;
  t.r = (gx - fl) + (double)(kFsWidth / 2 - 1);
  return t;
}
// Distance of the sample from its tap b, rounded once.
__host__ __device__ inline float fs_dist(double r, int b) { return (float)(r - (double)b); }

}  // namespace holo
