// The edge block's message transform without operands in memory: rotate, mix, rotate back and update per tile of 32 edges.
//
// T_out[k] = T_in[k] + f_c D^T W (D x_src, D x_dst, D T_in[k]): what the separate kernels move through memory per edge (the
// rotated rows, 9.6 KB at lmax 4 and 32 channels, written and read, and the products) stays in LDS and registers here, and
// HBM sees T_in twice and T_out once.
//
// A workgroup takes 32 edges through stages of 16 channels of one group (edge, source, destination): threads (edge, channel)
// rotate a row, scale it by a power of two of the edge's own and cut it into half-precision pieces in LDS; the 4 waves
// contract it with the weights, which come from L2 (1 MB for 32 edges), into accumulators of [output channel][edge], 25 x 32 x 32
// floats at lmax 4 = 100 registers a thread.  Two workgroups share a compute unit, one rotating while the other contracts, whose
// wavefronts go first where both could issue (s_setprio).
// 628,000 edges, lmax 4, 32 channels: 3.11 ms.  Parts, by leaving the others out: rotations and pieces 1.05 ms, contraction 1.55 (matrix
// cores 0.75, 20 GB of weights from L2, 20 GB of operands from LDS), rotating back and updating 0.65 (4 GB, 6 TB/s): they hardly
// overlap.  Tiles of 64 edges and 8 waves, half the weights' traffic but one workgroup per compute unit: 3.45; without the priority 3.24;
// weights two steps ahead 3.30, operands read one step ahead 3.34, rows to update asked for ahead 3.25: nothing waits for those.
// Separate kernels: 5.0 (gather 1.5, products 2.4, update 1.1).  16 waves of 128 registers: 8.4 (47 spilled).
#include "bond_frame.h"
#include "egnn_internal.h"
#include "so2_edge.h"
#include "stream_gemm.h"

#define SO2E_EDGES 32
#define SO2E_WAVES 4
#define SO2E_THREADS (64 * SO2E_WAVES)
#define SO2E_CE 16           // channels of one group per stage: the contraction length of one matrix instruction
// bytes of one component (l, m) of a stage's operand: two pieces of two half-waves of 32 x 16 bytes, each half-wave padded by 64
// bytes, so that the pieces and halves that a wave writes together fall into different banks
#define SO2E_HALF (16 * SO2E_EDGES + 64)
#define SO2E_PIECE (2 * SO2E_HALF)
#define SO2E_COMP (2 * SO2E_PIECE)
#define SO2E_LDY 36          // row pitch (floats) of the products on their way back: 16 channels x 32 edges per component
#define SO2E_INLINE __attribute__((always_inline))

// Work units: outputs (lo, +m) and (lo, -m) of a pair share their weights Wr, Wi; of order 0, two degrees lo share their
// operand.  Both are two 32 x 32 accumulators (two outputs x 32 edges) and four operand registers of weights
// per input degree.  Units are dealt to the 4 waves largest first, at most four each.
template <int LMAX>
struct So2eUnits {
  static constexpr int MAX = 16;
  int n, total_l;              // units; sum of their input degrees
  int m[MAX], lo[MAX], l0[MAX];
  int slot[SO2E_WAVES][4], most;    // units of a wave; largest number of them
  constexpr So2eUnits() : n(0), total_l(0), m{}, lo{}, l0{}, slot{}, most(0) {
    for (int q = 0; q <= LMAX; ++q)
      for (int d = q; d <= LMAX; d += (q == 0 ? 2 : 1)) {
        m[n] = q;
        lo[n] = d;
        l0[n] = total_l;
        total_l += LMAX + 1 - q;
        ++n;
      }
    int load[SO2E_WAVES] = {}, used[SO2E_WAVES] = {};
    bool done[MAX] = {};
    for (int w = 0; w < SO2E_WAVES; ++w)
      for (int q = 0; q < 4; ++q) slot[w][q] = -1;
    for (int t = 0; t < n; ++t) {
      int bu = -1, bc = -1;
      for (int u = 0; u < n; ++u) {
        const int cost = (LMAX + 1 - m[u]) * (m[u] ? 4 : lo[u] < LMAX ? 2 : 1);
        if (!done[u] && cost > bc) { bu = u; bc = cost; }
      }
      int bw = -1;
      for (int w = 0; w < SO2E_WAVES; ++w)
        if (used[w] < 4 && (bw < 0 || load[w] < load[bw])) bw = w;
      slot[bw][used[bw]++] = bu;
      if (used[bw] > most) most = used[bw];
      load[bw] += bc;
      done[bu] = true;
    }
  }
};

// ---------------------------------------------------------------------------------------------- weights
// out[block of 32 output channels][stage][unit, input degree][weight 0 / 1][piece][lane]; a lane holds eight input channels of
// one output channel
template <int LMAX>
__global__ __launch_bounds__(256) void so2e_pack_kernel(const float* __restrict__ W, int E, int n_stages, long n_lanes,
                                                        const unsigned* __restrict__ w_max, uint4* __restrict__ out) {
  static constexpr So2eUnits<LMAX> units{};
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_lanes) return;
  const int lane = (int)(i & 63), f = (int)(i >> 6) & 1;
  const long blk = i >> 7;
  const int ul = (int)(blk % units.total_l);
  const int st = (int)((blk / units.total_l) % n_stages), cb = (int)(blk / units.total_l / n_stages);
  int u = 0;
  while (u + 1 < units.n && units.l0[u + 1] <= ul) ++u;
  const int m = units.m[u], li = m + ul - units.l0[u], lo = units.lo[u] + (m ? 0 : f), nl = LMAX + 1 - m;
  const int per_group = E / SO2E_CE, g = (st / per_group + 2) % 3, c0 = (st % per_group) * SO2E_CE + 8 * (lane >> 5);
  const int co = cb * 32 + (lane & 31);
  size_t off = 0;
  for (int q = 0; q < m; ++q) off += (size_t)(q ? 2 : 1) * (LMAX + 1 - q) * (LMAX + 1 - q) * 3 * E * E;
  if (m && f) off += (size_t)nl * nl * 3 * E * E;
  float v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q)
    v[q] = co < E && lo <= LMAX ? W[off + (size_t)((lo - m) * E + co) * (nl * 3 * E) + (li - m) * 3 * E + g * E + c0 + q] : 0.0f;
  uint4 hi, lw;
  sgh_split8(v, ldexpf(1.0f, sgh_scale_exp(*w_max)), hi, lw);
  out[(blk * 4 + 2 * f) * 64 + lane] = hi;
  out[(blk * 4 + 2 * f + 1) * 64 + lane] = lw;
}

// ---------------------------------------------------------------------------------------------- the block
struct So2eArgs {
  const int* src;
  const int* dst;
  const float4* rhat_d;
  const float* x;
  unsigned x_bytes;
  const float* T_in;
  float* T_out;
  const uint4* w;
  const unsigned* w_max;
  long n_edges;
  int n_tiles, per_xcd, n_cb, log2E;
  float r_cut;
};

// high piece in the low half, rest in the high half
__device__ __forceinline__ uint32_t so2e_split(float x, float scale) {
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  const _Float16 h = (_Float16)__builtin_fmaf(x, scale, 0.0f);
  return __builtin_bit_cast(uint32_t, h2{h, (_Float16)__builtin_fmaf(x, scale, -(float)h)});
}
__device__ __forceinline__ uint4 so2e_neg(uint4 a) {
  return make_uint4(a.x ^ 0x80008000u, a.y ^ 0x80008000u, a.z ^ 0x80008000u, a.w ^ 0x80008000u);
}

template <int LMAX>
__global__ __launch_bounds__(SO2E_THREADS, 2) void so2e_block_kernel(So2eArgs p) {
  constexpr int D = (LMAX + 1) * (LMAX + 1), NS = So2eUnits<LMAX>().most;
  static constexpr So2eUnits<LMAX> units{};
  typedef __amdgpu_buffer_rsrc_t rsrc;
  extern __shared__ uint4 so2e_smem[];
  __shared__ float s_ratio[SO2E_EDGES];
  __shared__ sg_f4 s_trig[SO2E_EDGES][4];      // per edge: the angles' multiples, envelope and rows (kept out of the registers)
  __shared__ float s_fc[SO2E_EDGES];
  __shared__ int s_row[3][SO2E_EDGES];
  char* s_a = reinterpret_cast<char*>(so2e_smem);
  float* s_y = reinterpret_cast<float*>(so2e_smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  const int idx = (int)(blockIdx.x >> 3), cb = idx % p.n_cb;
  const int tile = (int)(blockIdx.x & 7) * p.per_xcd + idx / p.n_cb;
  if (idx / p.n_cb >= p.per_xcd || tile >= p.n_tiles) return;
  const int log2E = p.log2E, E = 1 << log2E, per_group = E / SO2E_CE, n_stages = 3 * per_group;
  const long e0 = (long)tile * SO2E_EDGES;
  const int ne = p.n_edges - e0 < SO2E_EDGES ? (int)(p.n_edges - e0) : SO2E_EDGES;
  // (buffers: the offsets of a row's components are scalars, and stores past the last edge's row are dropped)
  const rsrc xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.x), 0, (int)p.x_bytes, 0x00020000);
  const rsrc tr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.T_in + (((size_t)e0 * D) << log2E)), 0,
                                                    (ne * D) << (log2E + 2), 0x00020000);
  const rsrc to = __builtin_amdgcn_make_buffer_rsrc(p.T_out + (((size_t)e0 * D) << log2E), 0, (ne * D) << (log2E + 2), 0x00020000);

  if (tid < SO2E_EDGES) {
    const int e = tid < ne ? tid : ne - 1;     // (edges past the last repeat it)
    const float4 g = p.rhat_d[e0 + e];
    BondTrig t;
    egnn_bond_trig<4>(g.x, g.y, g.z, t);
#pragma unroll
    for (int m = 1; m <= 4; ++m) s_trig[tid][m - 1] = sg_f4{t.cp[m], t.sp[m], t.ct[m], t.st[m]};
    s_fc[tid] = egnn_envelope(g.w, p.r_cut);
    s_row[0][tid] = (e * D) << (log2E + 2);
    s_row[1][tid] = (int)(((unsigned)p.src[e0 + e] * D) << (log2E + 2));
    s_row[2][tid] = (int)(((unsigned)p.dst[e0 + e] * D) << (log2E + 2));
  }
  auto trig = [&](int e, BondTrig& t) SO2E_INLINE {
#pragma unroll
    for (int m = 1; m <= LMAX; ++m) {
      const sg_f4 q = s_trig[e][m - 1];
      t.cp[m] = q[0]; t.sp[m] = q[1]; t.ct[m] = q[2]; t.st[m] = q[3];
    }
  };
  __syncthreads();

  // thread -> (edge, channel of the stage), two edges
  const int c = lane & 15, edge0 = wave * 4 + (lane >> 4);
  int e_cur[2] = {60, 60};
  auto fetch = [&](int st, int e, float* v) SO2E_INLINE {
    const int g = st / per_group, ch = (st - g * per_group) * SO2E_CE * 4;      // edge, source, destination
    const int o = s_row[g][e] + 4 * c;
    const rsrc r = g == 0 ? tr : xr;
#pragma unroll
    for (int i = 0; i < D; ++i) v[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, o, (i << (log2E + 2)) + ch, 0));
  };
  float16v acc[NS][2];
#pragma unroll
  for (int u = 0; u < NS; ++u)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[u][t][i] = 0.0f;
  const char* frag = s_a + hh * SO2E_HALF + l32 * 16;
  // weights of the next input degree, unit or stage, requested one step ahead, so the first of a stage arrive while the rows are
  // rotated (requested within the unit only: 3.65 instead of 3.45 ms with tiles of 64 edges)
  auto weights = [&](int st, int u) SO2E_INLINE {
    return p.w + (((size_t)cb * n_stages + st) * units.total_l + units.l0[units.slot[wave][u]]) * 256 + lane;
  };
  uint4 wn[4];
  if (units.slot[wave][0] >= 0) {
    const uint4* w = weights(0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) wn[q] = w[q * 64];
  }

  for (int st = 0; st < n_stages; ++st) {
    // rotated, scaled by the edge's own power of two (that of the largest value met so far) and cut into pieces
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      float v[D];
      const int e = edge0 + it * (SO2E_EDGES / 2);
      fetch(st, e, v);
      BondTrig t;
      trig(e, t);
      egnn_to_bond_frame<LMAX>(v, t);
      float mx = 0.0f;
#pragma unroll
      for (int i = 0; i < D; ++i) mx = fmaxf(mx, fabsf(v[i]));
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
      const int e_row = mx == 0.0f ? 60 : sgh_scale_exp(__float_as_uint(mx));
      const int e_new = e_row < e_cur[it] ? e_row : e_cur[it];
      if (c == 0) s_ratio[e] = ldexpf(1.0f, e_new - e_cur[it]);
      e_cur[it] = e_new;
      const float sc = ldexpf(1.0f, e_new);
      // pairs of channels share a word: the even one writes the high pieces of both, the odd one the low pieces
      char* base = s_a + (c & 1) * SO2E_PIECE + (c >> 3) * SO2E_HALF + e * 16 + ((c & 7) >> 1) * 4;
      const uint32_t sel = (c & 1) ? 0x03020706u : 0x05040100u;
#pragma unroll
      for (int i = 0; i < D; ++i) {
        const uint32_t own = so2e_split(v[i], sc);
        const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);   // lane ^ 1
        *reinterpret_cast<uint32_t*>(base + i * SO2E_COMP) = __builtin_amdgcn_perm(other, own, sel);
      }
    }
    __syncthreads();
    __builtin_amdgcn_s_setprio(2);
    const float ratio = s_ratio[l32];
    const bool rescale = __any(ratio != 1.0f);
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int unit = units.slot[wave][u];
      if (unit < 0) continue;
      if (rescale) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[u][t][i] *= ratio;
      }
      const int m = units.m[unit];
      const uint4* w = weights(st, u);
      const uint4* after = u + 1 < NS && units.slot[wave][u + 1 < NS ? u + 1 : u] >= 0 ? weights(st, u + 1) : weights(st + 1 < n_stages ? st + 1 : st, 0);
#define SO2E_F(comp, piece) (*reinterpret_cast<const uint4*>(frag + (comp) * SO2E_COMP + (piece) * SO2E_PIECE))
#define SO2E_MMA(W, A, C) C = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(W), sgh_as_h8(A), C, 0, 0, 0)
      for (int l = m; l <= LMAX; ++l) {
        uint4 wc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) wc[q] = wn[q];
        w = l < LMAX ? w + 256 : after;
#pragma unroll
        for (int q = 0; q < 4; ++q) wn[q] = w[q * 64];
        const int cp = l * l + l + m, cm = l * l + l - m;
        const uint4 ph = SO2E_F(cp, 0), pl = SO2E_F(cp, 1);
        float16v &a0 = acc[u][0], &a1 = acc[u][1];
        SO2E_MMA(wc[1], ph, a0); SO2E_MMA(wc[3], ph, a1);
        SO2E_MMA(wc[0], pl, a0); SO2E_MMA(wc[2], pl, a1);
        if (m == 0) {
          SO2E_MMA(wc[0], ph, a0); SO2E_MMA(wc[2], ph, a1);
        } else {
          // y_+ = Wr x_+ - Wi x_-, y_- = Wi x_+ + Wr x_-
          const uint4 mh = SO2E_F(cm, 0), ml = SO2E_F(cm, 1), nh = so2e_neg(mh), nl = so2e_neg(ml);
          SO2E_MMA(wc[3], nh, a0); SO2E_MMA(wc[1], mh, a1);
          SO2E_MMA(wc[2], nl, a0); SO2E_MMA(wc[0], ml, a1);
          SO2E_MMA(wc[0], ph, a0); SO2E_MMA(wc[2], ph, a1);
          SO2E_MMA(wc[2], nh, a0); SO2E_MMA(wc[0], mh, a1);
        }
      }
#undef SO2E_MMA
#undef SO2E_F
    }
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
  }

  // back through LDS, 16 output channels at a time: threads (edge, channel) rotate the products back and update the row
  const int eb = sgh_scale_exp(*p.w_max);
#pragma unroll
  for (int it = 0; it < 2; ++it)
    if (c == 0) s_ratio[edge0 + it * (SO2E_EDGES / 2)] = ldexpf(1.0f, -e_cur[it]) * ldexpf(1.0f, -eb);
  __syncthreads();
  const float unscale = s_ratio[l32];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (half * 16 >= E) break;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int unit = units.slot[wave][u];
      if (unit < 0) continue;
      const int m = units.m[unit], lo = units.lo[unit];
      const int c0 = lo * lo + lo + m, c1 = m ? lo * lo + lo - m : (lo + 1) * (lo + 2);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if (t && m == 0 && lo == LMAX) break;      // (no second degree)
        float* y = s_y + ((t ? c1 : c0) * 16 + 4 * hh) * SO2E_LDY + l32;
#pragma unroll
        for (int i = 0; i < 8; ++i) y[(8 * (i >> 2) + (i & 3)) * SO2E_LDY] = acc[u][t][half * 8 + i] * unscale;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const int e = edge0 + it * (SO2E_EDGES / 2);
      if (e < ne) {
        float o[D], ti[D];
        const int row = s_row[0][e] + 4 * c, ch = (cb * 32 + half * 16) * 4;
#pragma unroll
        for (int i = 0; i < D; ++i) ti[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(tr, row, (i << (log2E + 2)) + ch, 0));
#pragma unroll
        for (int i = 0; i < D; ++i) o[i] = s_y[(i * 16 + c) * SO2E_LDY + e];
        BondTrig t;
        trig(e, t);
        egnn_from_bond_frame<LMAX>(o, t);
        const float fc = s_fc[e];
#pragma unroll
        for (int i = 0; i < D; ++i)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ti[i] + fc * o[i]), to, row, (i << (log2E + 2)) + ch, 0);
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------- host side
static long so2e_blocks(const egnn_ctx* ctx) {
  const int E = ctx->desc.channels;
  static const int total_l[5] = {So2eUnits<0>().total_l, So2eUnits<1>().total_l, So2eUnits<2>().total_l, So2eUnits<3>().total_l,
                                 So2eUnits<4>().total_l};
  return (long)((E + 31) / 32) * 3 * (E / SO2E_CE) * total_l[ctx->desc.lmax];
}
size_t so2e_weight_bytes(const egnn_ctx* ctx) { return (size_t)so2e_blocks(ctx) * 256 * 16; }

template <int LMAX>
static int so2e_launch(egnn_ctx* ctx, const So2eArgs& a, const float* W, uint4* wpack, hipStream_t st) {
  const int E = ctx->desc.channels;
  const long n_lanes = so2e_blocks(ctx) * 128;
  hipLaunchKernelGGL(so2e_pack_kernel<LMAX>, dim3((unsigned)((n_lanes + 255) / 256)), dim3(256), 0, st, W, E, 3 * (E / SO2E_CE),
                     n_lanes, a.w_max, wpack);
  EGNN_LAUNCH_CHECK(ctx, "so2e_pack_kernel");
  constexpr int D = (LMAX + 1) * (LMAX + 1), Y = D * 16 * SO2E_LDY * 4, A = D * SO2E_COMP, lds = Y > A ? Y : A;
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(so2e_block_kernel<LMAX>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return egnn_check_hip(ctx, e, "hipFuncSetAttribute(so2e_block_kernel)");
  }
  hipLaunchKernelGGL(so2e_block_kernel<LMAX>, dim3(8u * a.per_xcd * a.n_cb), dim3(SO2E_THREADS), lds, st, a);
  EGNN_LAUNCH_CHECK(ctx, "so2e_block_kernel");
  return EGNN_OK;
}

int so2e_edge_block(egnn_ctx* ctx, const egnn_graph* g, const float* rhat_d, const float* x, const float* T_in, const float* W,
                    float* T_out, unsigned* w_max, uint4* wpack, hipStream_t st) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  int rc;
  if ((rc = so2_launch_wmax(ctx, W, w_max, st))) return rc;
  So2eArgs a;
  a.src = g->src; a.dst = g->dst; a.rhat_d = reinterpret_cast<const float4*>(rhat_d); a.x = x;
  a.x_bytes = (unsigned)((size_t)g->n_total * (lmax + 1) * (lmax + 1) * E * 4);
  a.T_in = T_in; a.T_out = T_out; a.w = wpack; a.w_max = w_max; a.n_edges = g->n_edges;
  a.n_tiles = (int)((g->n_edges + SO2E_EDGES - 1) / SO2E_EDGES); a.per_xcd = (a.n_tiles + 7) / 8;
  a.n_cb = (E + 31) / 32; a.log2E = ctx->log2_channels; a.r_cut = ctx->desc.r_cut;
  switch (lmax) {
    case 0: return so2e_launch<0>(ctx, a, W, wpack, st);
    case 1: return so2e_launch<1>(ctx, a, W, wpack, st);
    case 2: return so2e_launch<2>(ctx, a, W, wpack, st);
    case 3: return so2e_launch<3>(ctx, a, W, wpack, st);
    default: return so2e_launch<4>(ctx, a, W, wpack, st);
  }
}
