// Internal: the vector of an edge, from its destination to its source.
#pragma once
#include "egnn_internal.h"

// In double precision from the fp32 positions and the periodic shift.  Two kernels write it down (edge_radial.hip, edge_fused.hip),
// and the reverse pass takes it from either: the fused operations are spelled out, so that both have the same bits.
struct EdgeVector { double x, y, z, rho2, d; };   // rho2 = x^2 + y^2, d = length
__device__ __forceinline__ EdgeVector egnn_edge_vector(const float* __restrict__ pos, const int8_t* __restrict__ shift, long k,
                                                       int i, int j, double bx, double by, double bz) {
  EdgeVector v;
  v.x = (double)pos[3 * i + 0] - (double)pos[3 * j + 0];
  v.y = (double)pos[3 * i + 1] - (double)pos[3 * j + 1];
  v.z = (double)pos[3 * i + 2] - (double)pos[3 * j + 2];
  if (shift) {
    v.x = fma((double)shift[3 * k + 0], bx, v.x);
    v.y = fma((double)shift[3 * k + 1], by, v.y);
    v.z = fma((double)shift[3 * k + 2], bz, v.z);
  }
  v.rho2 = fma(v.y, v.y, v.x * v.x);
  v.d = sqrt(fma(v.z, v.z, v.rho2));
  return v;
}
// unit vector and length, as the kernels read them
__device__ __forceinline__ float4 egnn_edge_record(const EdgeVector& v, double inv) {
  return make_float4((float)(v.x * inv), (float)(v.y * inv), (float)(v.z * inv), (float)v.d);
}
