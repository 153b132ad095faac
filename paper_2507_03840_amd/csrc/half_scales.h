// The power-of-two scalings of the half-precision pieces of a radial contraction's operands, in parts (see
// half_scales_part_kernel).
#pragma once
#include "egnn_internal.h"
// (The parts end at word 32: the reverse pass keeps another word behind its first 128 bytes of scales.)
#define HS_BLOCKS 24
#define HS_PART 8
static_assert(HS_PART + HS_BLOCKS <= 32, "see above");

// x -> (hi, lo) half-precision pieces, as raw bits
__device__ __forceinline__ void rw_split(float x, uint32_t& hi, uint32_t& lo) {
  const _Float16 h = (_Float16)x;
  const _Float16 l = (_Float16)(x - (float)h);
  hi = __builtin_bit_cast(unsigned short, h);
  lo = __builtin_bit_cast(unsigned short, l);
}

// element i of W_r2 (x), times alpha and s_w, as S3 reads it: out[i / 64][piece][i % 64]
__device__ __forceinline__ void half_piece_of_w2(float x, int i, float s_w, uint16_t* __restrict__ out, int log2E,
                                                 const PathAlpha& alpha) {
  const int n = i >> 6, j = i & 63;
  uint32_t hi, lo;
  rw_split(x * alpha.a[n >> log2E] * s_w, hi, lo);
  uint16_t* o = out + (size_t)n * 2 * EGNN_HIDDEN + j;
  o[0] = (uint16_t)hi;
  o[EGNN_HIDDEN] = (uint16_t)lo;
}

// part `block` of HS_BLOCKS, by a workgroup of 256 threads
__device__ __forceinline__ void half_scales_part(int block, const float* __restrict__ W_r1, const float* __restrict__ W_r2,
                                                 int n_rbf, int PE, int log2E, const PathAlpha& alpha,
                                                 float* __restrict__ scales) {
  __shared__ float red[4];
  float mw = 0.0f;
  const float4* W4 = reinterpret_cast<const float4*>(W_r2);
#pragma unroll 4
  for (int i = block * 256 + threadIdx.x; i < PE * (EGNN_HIDDEN / 4); i += HS_BLOCKS * 256) {
    const float4 v = W4[i];
    const float al = fabsf(alpha.a[(i / (EGNN_HIDDEN / 4)) >> log2E]);
    mw = fmaxf(mw, al * fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mw = fmaxf(mw, __shfl_xor(mw, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mw;
  __syncthreads();
  if (threadIdx.x == 0) scales[HS_PART + block] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  if (block == 0 && threadIdx.x < EGNN_HIDDEN) {
    float mg = 0.0f;
    for (int b = 0; b < n_rbf; ++b) mg += fabsf(W_r1[threadIdx.x * n_rbf + b]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mg = fmaxf(mg, __shfl_xor(mg, off));
    if (threadIdx.x == 0) scales[3] = mg;
  }
}

// s_w, s_g and 1 / (s_w s_g) from the parts; by a whole wavefront
__device__ __forceinline__ void half_scales_of(const float* __restrict__ scales, float& s_w, float& s_g, float& inv) {
  const int lane = threadIdx.x & 63;
  float mw = lane < HS_BLOCKS ? scales[HS_PART + lane] : 0.0f;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mw = fmaxf(mw, __shfl_xor(mw, off));
  const float mg = scales[3];
  // (zero, infinite or NaN weights: no scaling; the result then shows them as it would without)
  auto exp_of = [](float m) { return (m > 0.0f && m < 3.0e38f) ? ilogbf(m) : 13; };
  int ew = 13 - exp_of(mw), eg = 13 - exp_of(mg);
  ew = ew < -60 ? -60 : (ew > 60 ? 60 : ew);
  eg = eg < -60 ? -60 : (eg > 60 ? 60 : eg);
  s_w = ldexpf(1.0f, ew);
  s_g = ldexpf(1.0f, eg);
  inv = ldexpf(1.0f, -ew - eg);
}

