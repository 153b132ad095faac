// Internal: the grid of distances of the radial MLP's reverse pass (radial_grid.hip).
#pragma once
#include <hip/hip_runtime.h>

#define RG_BINS 2048
#define RG_PTS 6
#define RG_NODES (RG_BINS + RG_PTS - 1)

// Lagrange weights of the six grid points -2 .. 3 around an interval, at position t in [0, 1) inside it
__device__ __forceinline__ void rg_weights(float t, float (&phi)[RG_PTS]) {
  const float a = t + 2.0f, b = t + 1.0f, c = t, d = t - 1.0f, e = t - 2.0f, f = t - 3.0f;
  phi[0] = b * c * d * e * f * (-1.0f / 120.0f);
  phi[1] = a * c * d * e * f * (1.0f / 24.0f);
  phi[2] = a * b * d * e * f * (-1.0f / 12.0f);
  phi[3] = a * b * c * e * f * (1.0f / 12.0f);
  phi[4] = a * b * c * d * f * (-1.0f / 24.0f);
  phi[5] = a * b * c * d * e * (1.0f / 120.0f);
}
