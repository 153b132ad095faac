// The gradient of the radial weights of a layer, summed per length interval as it is made: no dw in memory.
//
// On the grid route (radial_grid.hip) dw[k][n] enters through  Zp[m][i][n] = sum_{k in interval m} phi_i(d_k) dw[k][n]  alone.
// A wavefront takes edges of one interval, forms dw of each from the two rows it comes from (features of the source, gradient of
// the destination's sum; both rotated into the edge's frame) and adds it to the six sums in registers.
//
// Work: a workgroup takes an interval and up to 32 channels, its four wavefronts every fourth group of 64 / channels edges;
// lane = (edge, channel).  Six sums of 42 paths are 252 registers a lane, so the halves of a wavefront, which hold the same
// channels of different edges, share the paths out: after one exchange the lower half has the first 21 gradients of both halves' edges,
// the upper half the other 21 (126 sums).
// The rows (2 x 3.2 KB an edge at lmax 4, 32 channels) go from memory to LDS one group ahead, as the rows of a gathered edge come
// from an L2 at best and nothing else hides that; indices two groups ahead, edge numbers three.
//
// 627,000 edges, lmax 4, 32 channels: 560 us (605 where an edge number was touched in the turn that loads it), in place of 640 for reading dw (3.4 GB) and 760 of the adjoint kernel's 1,350 for writing it.
// What bounds it: issue of vector instructions (945 a group and wavefront, at 3.6 cycles of a SIMD each with two wavefronts on it; by the
// counters waits take 11 % of their time, 17 with the touch, 2.8 GB of the 4 GB of rows miss the L2s and come from the last-level cache).
#include "egnn_internal.h"
#include "bond_frame.h"
#include "edge_fused.h"
#include "radial_grid.h"

struct TpBins {
  const int* src;
  const int* dst;
  const float4* rhat_d;
  const float* h;
  const float* da;
  const int* bin_ptr;
  const int* perm;
  float* Zp;
  const int* route;
  int log2E, PE, n_edges;
  float inv_h, scale;
};

// a = {lower half: its x, upper half: the lower half's y}, b = {lower half: the upper half's x, upper half: its y}
__device__ __forceinline__ void tpb_exchange(float x, float y, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

template <int LMAX, int L1>
struct TpBinsDegree {
  using Mid = typename LayerMid<LMAX>::T;
  __device__ __forceinline__ static void run(const float* v, const float* go, float* gw) {
    constexpr int first = Mid::CHUNK_FIRST[L1], count = Mid::CHUNK_COUNT[L1];
    float none[count], gv[2 * L1 + 1];       // (the gradient of the feature is not asked for here)
#pragma unroll
    for (int p = 0; p < count; ++p) none[p] = 0.0f;
    Mid::template run_bwd_l1<L1>(v + L1 * L1, none, go, gv, gw + first);
    if constexpr (L1 < LMAX) TpBinsDegree<LMAX, L1 + 1>::run(v, go, gw);
  }
};

template <int LMAX, int LC>      // 2^LC channels: all of them, or 32
__global__ __launch_bounds__(256, 2) void tp_bins_kernel(TpBins g) {
  if (!g.route[0]) return;
  using Mid = typename LayerMid<LMAX>::T;
  constexpr int D = (LMAX + 1) * (LMAX + 1), P = Mid::P, HP = (P + 1) / 2;
  constexpr int C = 1 << LC, EPW = 64 >> LC;                       // channels, edges of a wavefront
  constexpr int CHUNKS = D * C / 4;                                // 16-byte pieces of an edge's row
  constexpr int ES = ((D * C - C + 63) / 64) * 64 + C;             // an edge's room: banks differ from edge to edge by C
  constexpr int ROWS = EPW * ES;
  static_assert(ROWS * 2 >= HP * 64, "the sums go through the same LDS");
  __shared__ __align__(16) float sX[4][2][ROWS];

  const int m = RG_BINS - 1 - (int)blockIdx.x;                     // longest (fullest) intervals first
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & (C - 1), e = lane >> LC, cg0 = (int)blockIdx.y << LC;
  const int c0 = g.bin_ptr[m], c1 = g.bin_ptr[m + 1];
  float acc[HP][RG_PTS];
#pragma unroll
  for (int i = 0; i < HP; ++i)
#pragma unroll
    for (int k = 0; k < RG_PTS; ++k) acc[i][k] = 0.0f;

  const int begin = c0 + wave * EPW;
  if (begin < c1) {
    const int row = D << g.log2E;
    float* const myX = sX[wave][0];
    float* const myG = sX[wave][1];
    // (a number is put in range only where it becomes an index, a turn after its load: loads return in order, so a touch in the turn of
    // the load would wait for the rows asked for before it)
    auto edge_at = [&](int at) { return g.perm[min(at + e, c1 - 1)]; };
    auto in_range = [&](int k) { return min(max(k, 0), g.n_edges - 1); };
    // rows of the group's edges (j: the lane's own edge's node) to LDS
    auto load_rows = [&](const float* x, int j, float* to) {
#pragma unroll
      for (int ee = 0; ee < EPW; ++ee) {
        const int node = __builtin_amdgcn_readlane(j, ee << LC);
        const float* r = x + (size_t)node * row + cg0;
#pragma unroll
        for (int i = 0; i < (CHUNKS + 63) / 64; ++i) {
          const int q = 64 * i + lane;
          if (64 * i + 64 <= CHUNKS || q < CHUNKS)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(r + (((size_t)(q >> (LC - 2))) << g.log2E) + 4 * (q & (C / 4 - 1))),
                (__attribute__((address_space(3))) void*)(to + ee * ES + 256 * i), 16, 0, 0);
        }
      }
    };
    constexpr int STEP = 4 * EPW;
    const int k1 = in_range(edge_at(begin)), k2 = in_range(edge_at(begin + STEP));
    int k3 = edge_at(begin + 2 * STEP);
    int s1 = g.src[k1], j1 = g.dst[k1], s2 = g.src[k2], j2 = g.dst[k2];
    float4 r1 = g.rhat_d[k1], r2 = g.rhat_d[k2];
    load_rows(g.h, s1, myX);
    load_rows(g.da, j1, myG);
    for (int at = begin; at < c1; at += STEP) {
      ef_wait_arrived();
      float v[D], go[D], gw[2 * HP];
#pragma unroll
      for (int q = 0; q < D; ++q) {
        v[q] = myX[e * ES + q * C + c];
        go[q] = myG[e * ES + q * C + c];
      }
      const float4 r = r1;
      const bool valid = at + e < c1;
      ef_wait_read();
      // (the last group's are loaded once more by the ones after it)
      load_rows(g.h, s2, myX);
      load_rows(g.da, j2, myG);
      r1 = r2;
      const int k = in_range(k3);
      s2 = g.src[k];
      j2 = g.dst[k];
      r2 = g.rhat_d[k];
      k3 = edge_at(at + 3 * STEP);
      __builtin_amdgcn_sched_barrier(0);
      BondTrig t;
      egnn_bond_trig<LMAX>(r.x, r.y, r.z, t);
      egnn_to_bond_frame<LMAX>(v, t);
      egnn_to_bond_frame<LMAX>(go, t);
      if constexpr (2 * HP > P) gw[2 * HP - 1] = 0.0f;
      TpBinsDegree<LMAX, 0>::run(v, go, gw);
      float phi[RG_PTS], pa[RG_PTS], pb[RG_PTS];
      rg_weights(r.w * g.inv_h - (float)m, phi);
#pragma unroll
      for (int k = 0; k < RG_PTS; ++k) {
        const float x = valid ? phi[k] : 0.0f;
        tpb_exchange(x, x, pa[k], pb[k]);
      }
#pragma unroll
      for (int i = 0; i < HP; ++i) {
        float a, b;
        tpb_exchange(gw[i], gw[i + HP], a, b);
#pragma unroll
        for (int k = 0; k < RG_PTS; ++k) {
          acc[i][k] += pa[k] * a;
          acc[i][k] += pb[k] * b;
        }
      }
    }
    ef_wait_arrived();               // (nothing is on its way to LDS when it is used for the sums)
  }

  // edges of a half, then the wavefronts, in a fixed order
  float* const red = &sX[0][0][0];   // [wave][value][lane]
#pragma unroll
  for (int k = 0; k < RG_PTS; ++k) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < HP; ++i) {
      float x = acc[i][k];
#pragma unroll
      for (int off = C; off < 32; off <<= 1) x += __shfl_xor(x, off);
      red[(wave * HP + i) * 64 + lane] = x;
    }
    __syncthreads();
    float* out = g.Zp + ((size_t)m * RG_PTS + k) * g.PE + cg0;
    for (int idx = tid; idx < P * C; idx += 256) {
      const int p = idx >> LC, cc = idx & (C - 1), at = p < HP ? p * 64 + cc : (p - HP) * 64 + 32 + cc;
      const float x = (red[at] + red[at + HP * 64]) + (red[at + 2 * HP * 64] + red[at + 3 * HP * 64]);
      out[((size_t)p << g.log2E) + cc] = g.scale * x;
    }
  }
}

// Where making the gradients twice over (here for the sums, in the adjoint kernel for the features) is faster than writing and reading
// them, whole adjoint calls on 60 .. 2,500 atoms of 19 .. 107 edges: every interval costs a workgroup, so it takes edges enough.
// From 12,000 edges on (5,700 / 13,500 / 31,500 / 260,000 edges) lmax 1 1.01 / 1.05 / 1.08 / 1.33, lmax 2 1.0 / 1.03 / 1.06 / 1.3,
// lmax 3 0.99 / 1.03 / 1.08 / 1.41, lmax 4 0.96 / 1.01 / 1.11 / 1.5 times as fast at 32 and 64 channels.  With few channels a wavefront
// takes 4 or 8 edges and its rows come in more, smaller pieces: 16 channels at lmax 3 and 4 0.95 / 0.96 / 1.03 / 1.35, 8 channels there
// 0.89 / 0.92 / 0.97 / 1.35 (47,000: 1.03, 111,000: 1.2).  lmax 0, one path: not taken.
// (One wavefront an interval instead of four: lmax 4 1.02 to 1.1 times as fast up to 10,000 edges, slower from 30,000 on, lmax 2 slower.)
bool egnn_tp_bins_fits(const egnn_ctx* ctx, int64_t n_edges) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  return lmax >= 1 && n_edges >= (lmax < 3 || E >= 32 ? 12000 : E == 16 ? 30000 : 60000);
}

int egnn_launch_tp_bins(egnn_ctx* ctx, const TpBinsArgs& a, const float* rhat_d, int64_t n_edges, const int* bin_ptr, const int* perm,
                        float* Zp, const int* route, hipStream_t stream) {
  const int E = ctx->desc.channels, le = ctx->log2_channels;
  const TpBins x = {a.src, a.dst, reinterpret_cast<const float4*>(rhat_d), a.h, a.da, bin_ptr, perm, Zp, route, le,
                    ctx->n_paths[0] * E, (int)n_edges, (float)RG_BINS / ctx->desc.r_cut, 1.0f / sqrtf(ctx->desc.agg_norm)};
  const dim3 grid(RG_BINS, le > 5 ? E / 32 : 1);
#define LAUNCH(L, LC) \
  hipLaunchKernelGGL((tp_bins_kernel<L, LC>), grid, dim3(256), 0, stream, x)
#define CASES(L)                                                                 \
  case L:                                                                        \
    if (le == 3) LAUNCH(L, 3);                                                   \
    else if (le == 4) LAUNCH(L, 4);                                              \
    else if (le <= 7 && le > 4) LAUNCH(L, 5);                                    \
    else return egnn_fail(ctx, EGNN_EINVAL, "tp_bins: channels out of range");   \
    break;
  switch (ctx->desc.lmax) {
    CASES(1) CASES(2) CASES(3) CASES(4)
    default: return egnn_fail(ctx, EGNN_EINVAL, "tp_bins: lmax out of range");
  }
#undef CASES
#undef LAUNCH
  EGNN_LAUNCH_CHECK(ctx, "tp_bins_kernel");
  return EGNN_OK;
}
