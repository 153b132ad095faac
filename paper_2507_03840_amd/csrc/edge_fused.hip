// S3 + S4 in one kernel: the radial weights of an (edge, channel) come off the matrix cores into the registers of the lane that
// uses them; no weight tensor in memory.
//
//   a[j] = nbar^-1/2 sum_{k: dst(k)=j} sum_p w_k[p][c] (C_p . h_src(k) . Yhat(rhat_k)),
//   w_k[p][c] = fc(d_k) alpha_p (W_r2 SiLU(W_r1 B(d_k)))[p*E + c]
// (Sec. 3 "Message passing"; coupling of Sec. 2.2 / Eq. 1 in the bond frame of Sec. 2.1 / Fig. 2(d)).
//
// Through memory, w is the largest object of a layer: at 3,000 atoms, 32 channels and lmax 4 it took 1.7 GB of writes (353 us)
// and 3.4 GB of reads (640 us).  Here, same case: 500 to 600 us for the kernel below (passes one after the other; 525 between
// pauses) and 50 us of preparation; 12,000 + 8,000 atoms at 64 channels 7.4 -> 4.5 ms.
//
// Work: a wavefront takes a destination node and 4 channels and walks the node's edges 16 at a time.  The 16x16x32 tiles have the
// rows of W_r2 as rows (4 paths x 4 channels) and the 16 edges as columns, so result register r of lane (n, q) is path 4 t + r
// of edge n and channel 4 group + q: 11 tiles of 6 products give a lane the 42 weights of its (edge, channel), which then runs the
// bond-frame product as S4 does.  (A tile of 32 edges x 2 channels, 32x32x16, takes fewer LDS reads but leaves more lanes idle
// at a node's end and more lines per gathered row: 1,180 against 1,058 ns for the arithmetic of 64 lanes.)  The lane keeps
// its 25 sums until the node ends; then the 16 edges are added.  No atomics, a fixed order.
//
// What bounds it: issue, at the clock that the chip holds under it.  Counters of that launch: 1.76 GHz (2.3 on zeros), vector
// instructions, matrix ones among them, issue in 90 % of the SIMD-cycles, the matrix cores are busy in 36 %, the vector cache in 30 %, LDS in
// 24 % of a CU's, 0.4 GB fetched.  The products (66 x 16 cycles a tile) and the vector work (555 instructions) of the two
// wavefronts of a SIMD overlap in part; a copy of the loop without its memory accesses took 347 us.  What the layout is for:
//   * W_r2 of 4 channels (45 KB at lmax 4) stays on the compute unit: high pieces in registers, low pieces in LDS.  With all of it
//     in LDS (44 reads of 1 KB a tile and wavefront) LDS and the products took turns.
//   * Both gathered streams go from memory straight to LDS one tile ahead, four neighbouring lanes per 64 bytes.  As loads to
//     registers in the products' lane order, neighbouring lanes were different edges, every 16 bytes an access of its own:
//     728 accesses a tile, and the vector cache, one a cycle, was the limit (1.0 of 1.1 M cycles).
//   * The hidden activations (256 bytes a row of weights) are read once per group of channels: two groups share an XCD, so
//     that its L2 serves one of them (misses halve; no difference beyond two).
#include "egnn_internal.h"
#include "bond_frame.h"
#include "half_scales.h"
#include "edge_vector.h"
#include "edge_fused.h"

__device__ __forceinline__ uint4 ef_pack8(const float (&x)[8], uint4& lo) {
  uint32_t h[8], l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const _Float16 a = (_Float16)x[i];
    const _Float16 b = (_Float16)(x[i] - (float)a);
    h[i] = __builtin_bit_cast(unsigned short, a);
    l[i] = __builtin_bit_cast(unsigned short, b);
  }
  lo = make_uint4(l[0] | (l[1] << 16), l[2] | (l[3] << 16), l[4] | (l[5] << 16), l[6] | (l[7] << 16));
  return make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
}

// First preparation.  Per edge the rotation into its frame (cos p, sin p, cos t, sin t of the azimuth and polar angle), per row
// of radial weights the length and the cutoff envelope; the last HS_BLOCKS workgroups take the parts of the operands' scalings.
struct EfFirst {
  const int* src;
  const int* dst;
  const int8_t* shift;
  const float* pos;
  const int* w_row;
  const float* W_r1;
  const float* W_r2;
  float4* frame;
  float2* length;
  float* scales;
  float4* rhat_d;                 // may be NULL (see edge_fused.h)
  float r_cut;
  double bx, by, bz;
  long n_edges;
  int n_rbf, PE, log2E;
  PathAlpha alpha;
};
__global__ __launch_bounds__(256) void ef_first_kernel(EfFirst g) {
  const int part = (int)blockIdx.x - ((int)gridDim.x - HS_BLOCKS);
  if (part >= 0) {
    half_scales_part(part, g.W_r1, g.W_r2, g.n_rbf, g.PE, g.log2E, g.alpha, g.scales);
    return;
  }
  const long k = (long)blockIdx.x * 256 + threadIdx.x;
  if (k >= g.n_edges) return;
  const EdgeVector v = egnn_edge_vector(g.pos, g.shift, k, g.src[k], g.dst[k], g.bx, g.by, g.bz);
  const double inv = 1.0 / v.d, rho = sqrt(v.rho2);
  const bool polar = rho <= 1e-15 * v.d;                // (the azimuth is free there)
  const double irho = polar ? 0.0 : 1.0 / rho;
  g.frame[k] = make_float4(polar ? 1.0f : (float)(v.x * irho), (float)(v.y * irho), (float)(v.z * inv), (float)(rho * inv));
  const int r = g.w_row ? g.w_row[k] : (int)k;
  if (r >= 0) g.length[r] = make_float2((float)v.d, egnn_envelope((float)v.d, g.r_cut));
  if (g.rhat_d) g.rhat_d[k] = egnn_edge_record(v, inv);
}

// Second preparation: both operands of the radial contraction, scaled and cut into two half-precision pieces.  The contraction
// runs over the 64 hidden units in two steps of 32; octet q of a step is what a lane (n, q) holds.
//   rec  [row][step][piece][q] of 16 bytes: hidden activations of a row times the cutoff envelope
//   A    [group of 4 channels][tile of 4 paths][step][piece][lane] of 16 bytes: alpha W_r2; lane (m, q) holds path
//        4 tile + m % 4, channel 4 group + m / 4
// A thread takes an octet of units of two rows, W_r1 from LDS.  What bounds it: the vector ALU (busy throughout by the counters, 1.7 GHz;
// 34 us for 313,000 rows of 16 Gaussians; sixteen lanes a row that share out its exponentials, rows asked for ahead and stores
// without a test measured the same).  (With the fp32 products on
// the matrix cores the weights came out less exact: their gradient summed over all edges was off by 2.03e-7 instead of 1.69e-7.)
// The next workgroups write A, the last ones (if w2s) scalings and pieces as S3 takes them.
struct EfSecond {
  const float2* length;
  const float* W_r1;
  const float* W_r2;
  const float* scales;
  uint4* rec;
  uint4* A;
  long n_rows;
  int n_rbf, P, NT, log2E, row_blocks, a_blocks;
  float r_cut;
  PathAlpha alpha;
  float* w2s;
};

__global__ __launch_bounds__(256) void ef_second_kernel(EfSecond g) {
  float s_w, s_g, inv;
  half_scales_of(g.scales, s_w, s_g, inv);
  const int lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
  const int ab = (int)blockIdx.x - g.row_blocks;
  if (ab >= g.a_blocks) {
    const int i = (ab - g.a_blocks) * 256 + threadIdx.x;
    if (i == 0) { g.w2s[0] = s_w; g.w2s[1] = s_g; g.w2s[2] = inv; }
    if (i < (g.P << g.log2E) * EGNN_HIDDEN)
      half_piece_of_w2(g.W_r2[i], i, s_w, reinterpret_cast<uint16_t*>(g.w2s + 64), g.log2E, g.alpha);
    return;
  }
  if (ab >= 0) {
    const int idx = ab * 256 + threadIdx.x;      // [group][tile][step][lane]
    const int ks = (idx >> 6) & 1, tile = (idx >> 7) % g.NT, cg = (idx >> 7) / g.NT;
    if (cg >= (1 << g.log2E) / 4) return;
    const int p = 4 * tile + (n & 3), c = 4 * cg + (n >> 2);
    const float f = p < g.P ? g.alpha.a[p] * s_w : 0.0f;
    const float* W = g.W_r2 + ((size_t)((p < g.P ? p : 0) << g.log2E) + c) * EGNN_HIDDEN;
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = p < g.P ? f * W[32 * ks + 8 * q + i] : 0.0f;
    uint4 lo;
    const uint4 hi = ef_pack8(x, lo);
    uint4* out = g.A + ((size_t)(cg * g.NT + tile) * 2 + ks) * 128 + lane;
    out[0] = hi;
    out[64] = lo;
    return;
  }
  __shared__ float sW1[32 * EGNN_HIDDEN];                // [Gaussian][unit]
  for (int i = threadIdx.x; i < g.n_rbf * EGNN_HIDDEN; i += 256) sW1[i] = g.W_r1[(i & 63) * g.n_rbf + (i >> 6)];
  __syncthreads();
  const int o = threadIdx.x & 7;
  const float step_r = g.r_cut / (float)(g.n_rbf - 1);
  const float inv2s2 = 0.5f / (step_r * step_r);
  for (long r0 = (long)blockIdx.x * 64 + (threadIdx.x >> 3); r0 < g.n_rows; r0 += (long)g.row_blocks * 64) {
    const bool two = r0 + 32 < g.n_rows;
    const float2 row[2] = {g.length[r0], g.length[two ? r0 + 32 : r0]};
    float pre[2][8];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 8; ++i) pre[t][i] = 0.0f;
    for (int b = 0; b < g.n_rbf; ++b) {
      const float4* wr = reinterpret_cast<const float4*>(sW1 + b * EGNN_HIDDEN + 8 * o);
      const float4 w0 = wr[0], w1 = wr[1];
      const float w[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const float u = row[t].x - (float)b * step_r;
        const float B = __expf(-u * u * inv2s2);
#pragma unroll
        for (int i = 0; i < 8; ++i) pre[t][i] += w[i] * B;
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float fc = s_g * row[t].y;
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        // SiLU by a reciprocal and one Newton step (a large exponential is cut off at 1e30, where the quotient is zero)
        const float y = 1.0f + fminf(__expf(-pre[t][i]), 1e30f);
        const float r = __builtin_amdgcn_rcpf(y);
        x[i] = fc * pre[t][i] * __builtin_fmaf(__builtin_fmaf(-y, r, 1.0f), r, r);
      }
      uint4 lo;
      const uint4 hi = ef_pack8(x, lo);
      if (t == 0 || two) {
        uint4* out = g.rec + (r0 + 32 * t) * 16 + (o >> 2) * 8 + (o & 3);
        out[0] = hi;
        out[4] = lo;
      }
    }
  }
}

template <int CTRL>
__device__ __forceinline__ float ef_dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}


// Sums of N values over the 16 lanes of a row, shared out among them: each of the four steps adds a lane's partner's part and
// keeps one half of the values (3 instructions for each that is kept, against one per value and step of a full sum, and the
// results lie in the lanes that store them).  Lane n ends with values ef_slot(n) .. of x[0 ..].
template <int N> struct EfHalves {
  static constexpr int H1 = (N + 1) / 2, H2 = (H1 + 1) / 2, H3 = (H2 + 1) / 2, H4 = (H3 + 1) / 2;
};
template <int N, int H, int CTRL>
__device__ __forceinline__ void ef_halve(float* x, bool upper) {
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const float lo = x[i], hi = i + H < N ? x[i + H] : 0.0f;
    const float keep = upper ? hi : lo, give = upper ? lo : hi;
    x[i] = keep + ef_dpp<CTRL>(give);
  }
}
template <int N>
__device__ __forceinline__ void ef_sum16(float* x, int n) {
  using S = EfHalves<N>;
  ef_halve<N, S::H1, 0x140>(x, n & 8);          // lane 15 - n
  ef_halve<S::H1, S::H2, 0x141>(x, n & 4);      // lane 7 - n of the eight
  ef_halve<S::H2, S::H3, 0x4E>(x, n & 2);       // lane ^ 2
  ef_halve<S::H3, S::H4, 0xB1>(x, n & 1);       // lane ^ 1
}
// index of value r of lane n, or -1
template <int N>
__device__ __forceinline__ int ef_slot(int n, int r) {
  using S = EfHalves<N>;
  const int i4 = r + ((n & 1) ? S::H4 : 0), i3 = i4 + ((n & 2) ? S::H3 : 0), i2 = i3 + ((n & 4) ? S::H2 : 0),
            i1 = i2 + ((n & 8) ? S::H1 : 0);
  return i4 < S::H3 && i3 < S::H2 && i2 < S::H1 && i1 < N ? i1 : -1;
}

template <int LMAX, bool HALF, bool SHARED>
__global__ __launch_bounds__(256, EF_WG_PER_CU) void ef_layer_kernel(
    const int* __restrict__ row_ptr, const int* __restrict__ src, const int* __restrict__ w_row,
    const float4* __restrict__ frame, const uint4* __restrict__ rec, const uint4* __restrict__ A,
    const float4* __restrict__ h4, const float* __restrict__ scales, float* __restrict__ a, int n_owned, int n_edges,
    int log2E, int parts, float scale) {
  using Mid = typename LayerMid<LMAX>::T;
  constexpr int D = (LMAX + 1) * (LMAX + 1), P = Mid::P, NT = (P + 3) / 4, NQ = (D + 3) / 4;
  __shared__ uint4 sLo[NT * 2 * 64];         // low pieces of W_r2
  __shared__ uint4 sRec[4][4 * 64];          // per wavefront: the operand of its next tile
  __shared__ uint4 sH[4][NQ * 64];           //                and the features
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = 1 << (log2E - 2);
  // channel group and part of the nodes, see the launch
  const int xcd = blockIdx.x & 7, i_x = blockIdx.x >> 3;
  const int per = min(G, EF_CGX), sets = G / per;         // groups that share an XCD, sets of them
  int cg, part;
  if (sets >= 8) {
    const int turns = sets >> 3;
    cg = (xcd + 8 * ((i_x / per) % turns)) * per + i_x % per;
    part = i_x / (per * turns);
  } else {
    cg = (xcd % sets) * per + i_x % per;
    part = (i_x / per) * (8 / sets) + xcd / sets;
  }
  const uint4* Ag = A + (size_t)cg * NT * 256;
  for (int i = tid; i < NT * 2 * 64; i += 256) sLo[i] = Ag[(i >> 6) * 128 + 64 + (i & 63)];
  uint4 ah[NT][2];                           // high pieces
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) ah[t][ks] = Ag[(t * 2 + ks) * 128 + lane];
  float s_w, s_g, unscale;
  half_scales_of(scales, s_w, s_g, unscale);
  // the scalings of the operands are undone half before and half after the product (a whole power of two each)
  const int ex = ilogbf(unscale), exh = ex / 2;
  const float f = HALF ? 1.0f : ldexpf(1.0f, exh);
  const float fin = HALF ? scale : scale * ldexpf(1.0f, ex - 2 * exh);
  __syncthreads();

  const int n = lane & 15, q = lane >> 4;
  const int stride = parts * 4;
  int j = part * 4 + wave;
  if (j >= n_owned) return;
  const int last = n_edges - 1;
  float acc[D];
#pragma unroll
  for (int i = 0; i < D; ++i) acc[i] = 0.0f;

  // Tiles of 16 edges, three of them under way: tile 0 is worked on, the operand and the features of tile 1 are being
  // loaded, so are the indices of tile 2.  (k, k1): first edge of a tile and end of its node's edges; (kb, kb1): edges of the
  // node that follows tile 2's node.
  int k0 = row_ptr[j], k0_1 = row_ptr[j + 1], k1, k1_1, k2, k2_1, jn = j, kb, kb1;
  auto fetch_node = [&]() {
    jn += stride;
    const int jj = min(jn, n_owned - 1);
    kb = row_ptr[jj];
    kb1 = row_ptr[jj + 1];
  };
  auto advance = [&](int k, int k_1, int& kn, int& kn_1) {
    if (k + 16 >= k_1) {
      kn = kb;
      kn_1 = kb1;
      fetch_node();
    } else {
      kn = k + 16;
      kn_1 = k_1;
    }
  };
  fetch_node();
  advance(k0, k0_1, k1, k1_1);
  advance(k1, k1_1, k2, k2_1);

  // Memory to LDS: four neighbouring lanes bring the 64 bytes that the four channels (octets of units) of one edge need, so that
  // a request is a whole one; lane (q, n) then reads piece q of edge n.  The order of the four inside an edge is turned by
  // the edge's quad, which spreads the reads over the banks.
  const int e4 = lane >> 2, p4 = (lane & 3) ^ (lane >> 4), at4 = 4 * n + (q ^ (n >> 2));
  uint4* const myRec = sRec[wave];
  uint4* const myH = sH[wave];
  auto load_rec = [&](int raw) {
    const uint4* p = rec + (size_t)(SHARED && raw < 0 ? ~raw : raw) * 16 + p4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p + 4 * i),
                                       (__attribute__((address_space(3))) void*)(myRec + 64 * i), 16, 0, 0);
  };
  auto load_h = [&](int s) {
    const float4* p = h4 + ((size_t)s * G + cg) * (NQ * 4) + p4;
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p + 4 * i),
                                       (__attribute__((address_space(3))) void*)(myH + 64 * i), 16, 0, 0);
  };
  float4 fr;
  int s1, r1;
  {
    const int kk = min(k0 + e4, last);
    const int kk1 = min(k1 + e4, last);
    const int s = src[kk], r = SHARED ? w_row[kk] : kk;
    s1 = src[kk1];
    r1 = SHARED ? w_row[kk1] : kk1;
    fr = frame[min(k0 + n, last)];
    load_rec(r);
    load_h(s);
  }
  // The sums of a finished node are stored early in the next tile: a store in flight would hold up that tile's wait for its
  // operands.
  constexpr int H4 = EfHalves<D>::H4;
  float done[H4];
  int j_done = -1;
  auto store_node = [&]() {
    float* out = a + (((size_t)j_done * D) << log2E) + 4 * cg + q;
#pragma unroll
    for (int i = 0; i < H4; ++i) {
      const int at = ef_slot<D>(n, i);
      if (at >= 0) out[(size_t)at << log2E] = done[i];
    }
    j_done = -1;
  };
  while (true) {
    const bool node_done = k0 + 16 >= k0_1;
    ef_wait_arrived();
    uint4 b[2][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i >> 1][i & 1] = myRec[64 * i + at4];
    float v[NQ * 4], o[D];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const uint4 x = myH[64 * i + at4];
      v[4 * i] = __uint_as_float(x.x); v[4 * i + 1] = __uint_as_float(x.y);
      v[4 * i + 2] = __uint_as_float(x.z); v[4 * i + 3] = __uint_as_float(x.w);
    }
    const int kk2 = min(k2 + e4, last);
    const int s2 = src[kk2];
    const int r2 = SHARED ? w_row[kk2] : kk2;
    const float4 frn = frame[min(k1 + n, last)];
    ef_wait_read();                  // (before the next ones may arrive)
    if (j_done >= 0) store_node();
    load_rec(r1);
    load_h(s1);
    __builtin_amdgcn_sched_barrier(0);

    int at = lane;
    asm volatile("" : "+v"(at));     // (the operand stays in LDS: read ahead of the loop it would not fit the registers)
    ef_f4 c[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) c[t] = ef_f4{0.0f, 0.0f, 0.0f, 0.0f};
    // (the four correction products first: then the sum is rounded at its full size twice, not six times)
    ef_h8 bh[2], bl[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) { bh[ks] = __builtin_bit_cast(ef_h8, b[ks][0]); bl[ks] = __builtin_bit_cast(ef_h8, b[ks][1]); }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
        c[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(ef_h8, ah[t][ks]), bl[ks], c[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < NT; ++t)
        c[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(ef_h8, sLo[(t * 2 + ks) * 64 + at]), bh[ks], c[t], 0, 0, 0);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        c[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(ef_h8, ah[t][ks]), bh[ks], c[t], 0, 0, 0);
    float w[NT * 4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) w[4 * t + r] = HALF ? (float)(_Float16)(c[t][r] * unscale) : c[t][r];
    __builtin_amdgcn_sched_barrier(0);

    BondTrig t;
    t.cp[0] = 1.0f; t.sp[0] = 0.0f; t.ct[0] = 1.0f; t.st[0] = 0.0f;
    t.cp[1] = fr.x; t.sp[1] = fr.y; t.ct[1] = fr.z; t.st[1] = fr.w;
#pragma unroll
    for (int m = 2; m <= LMAX; ++m) {
      t.cp[m] = t.cp[m - 1] * fr.x - t.sp[m - 1] * fr.y;
      t.sp[m] = t.sp[m - 1] * fr.x + t.cp[m - 1] * fr.y;
      t.ct[m] = t.ct[m - 1] * fr.z - t.st[m - 1] * fr.w;
      t.st[m] = t.st[m - 1] * fr.z + t.ct[m - 1] * fr.w;
    }
    if (!HALF) {
#pragma unroll
      for (int m = 1; m <= LMAX; ++m) { t.cp[m] *= f; t.sp[m] *= f; }
#pragma unroll
      for (int l = 0; l <= LMAX; ++l) v[l * l + l] *= f;
    }
    egnn_to_bond_frame<LMAX>(v, t);
    Mid::run(v, w, o);
    egnn_from_bond_frame<LMAX>(o, t);
    if (!HALF) {
#pragma unroll
      for (int l = 0; l <= LMAX; ++l) o[l * l + l] *= f;
    }
    if (node_done) {      // (lanes past the node's last edge hold other edges: left out)
      const bool valid = k0 + n < k0_1;
#pragma unroll
      for (int i = 0; i < D; ++i) acc[i] += valid ? o[i] : 0.0f;
      ef_sum16<D>(acc, n);
#pragma unroll
      for (int i = 0; i < H4; ++i) done[i] = fin * acc[i];
      j_done = j;
#pragma unroll
      for (int i = 0; i < D; ++i) acc[i] = 0.0f;
      j += stride;
      if (j >= n_owned) break;
    } else {
#pragma unroll
      for (int i = 0; i < D; ++i) acc[i] += o[i];
    }
    k0 = k1; k0_1 = k1_1; k1 = k2; k1_1 = k2_1;
    advance(k1, k1_1, k2, k2_1);
    fr = frn;
    s1 = s2;
    r1 = r2;
  }
  ef_wait_arrived();                 // (nothing is on its way to LDS when the workgroup gives it back)
  store_node();
}

// Where this kernel is the faster one, measured on 48 .. 3,000 atoms of 13 .. 209 edges, whole calls against the two kernels: the one
// that makes the weights for itself, and the one that also writes them for the reverse pass.  Both give the same bits, so one
// rule holds for both; the second runs S3 as well, on what was prepared for the sums.
//   lmax 2 to 4, up to 64 channels: 1.06 to 2.9 times; keeping the weights 0.92 to 1.6, median 1.05 to 1.1, below 0.97 at lmax 2 on
//     graphs without shared rows.  Where a node has about 19 edges, which leave every second tile of 16 nearly empty, keeping
//     them 0.87 to 0.98 (2 to 20 us of the call, up to 3 % of a training step of the layer), not keeping them 1.06 to 1.4.
//   lmax 2, 128 channels, whose 32 groups of channels read the hidden activations 32 times: up to 300 nodes 1.05 to 1.8, keeping them
//     0.91 to 1.56; on more from 60 edges a node 1.06 to 1.46 and 0.96 to 1.2, from 800 nodes and 25 edges a node 1.06 to 1.46 and
//     0.98 to 1.07.  Between them 0.94 to 1.14 and 0.85 to 1.04, from 800 nodes below 25 edges 1.02 to 1.06 and 0.96 to 1.0: not taken.
//   lmax 1, where w is small: up to 800 nodes x 32 channels and 46,000 edges x 32 channels 1.11 to 1.45, keeping them 0.98 to 1.23;
//     beyond, 0.95 to 1.27 and 0.78 to 0.98: not taken.  128 channels 0.89 to 1.7: not taken.
//   lmax 0, where one path takes a tile of four, 0.58 to 1.0 for 37,000 edges and more: not taken.
// The scratch is the room of a weight tensor in memory, which is not needed then; whether it is large enough is asked for one row
// per edge, so that a graph with shared rows goes the same way as one without (lmax 1: from 32 channels on).
bool egnn_edge_fused_fits(const egnn_ctx* ctx, const egnn_graph* g) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  const bool small = (int64_t)g->n_owned * E <= 800 * 32 && g->n_edges * E <= 46000 * 32;
  if (lmax == 0 || (lmax == 1 && (E > 64 || !small))) return false;
  if (lmax == 2 && E == 128 && g->n_owned > 300 && g->n_edges < (int64_t)(g->n_owned < 800 ? 60 : 25) * g->n_owned) return false;
  return g->n_edges > 0 && g->n_owned > 0 &&
         egnn_ef_carve(ctx, g, 0, nullptr).bytes <= (size_t)g->n_edges * ctx->n_paths[0] * E * sizeof(float);
}

static PathAlpha ef_alpha(const egnn_ctx* ctx, int which) {
  PathAlpha al;
  for (int p = 0; p < EGNN_MAX_PATHS; ++p) al.a[p] = p < ctx->n_paths[which] ? ctx->alpha[which][p] : 0.0f;
  return al;
}

int egnn_launch_edge_fused_first(egnn_ctx* ctx, const egnn_graph* g, int which, const float* pos, const float box[3],
                                 const float* W_r1, const float* W_r2, void* scratch, hipStream_t stream, float* rhat_d) {
  const EfScratch s = egnn_ef_carve(ctx, g, which, scratch);
  const EfFirst x = {g->src, g->dst, g->shift, pos, g->w_row, W_r1, W_r2, s.frame, s.length, s.scales,
                     reinterpret_cast<float4*>(rhat_d), ctx->desc.r_cut,
                     (double)box[0], (double)box[1], (double)box[2], (long)g->n_edges, ctx->desc.n_rbf,
                     ctx->n_paths[which] * ctx->desc.channels, ctx->log2_channels, ef_alpha(ctx, which)};
  hipLaunchKernelGGL(ef_first_kernel, dim3((unsigned)((g->n_edges + 255) / 256 + HS_BLOCKS)), dim3(256), 0, stream, x);
  EGNN_LAUNCH_CHECK(ctx, "ef_first_kernel");
  return EGNN_OK;
}

int egnn_launch_edge_fused_second(egnn_ctx* ctx, const egnn_graph* g, int which, const float* W_r1, const float* W_r2,
                                  void* scratch, hipStream_t stream, void* w2s) {
  const EfScratch s = egnn_ef_carve(ctx, g, which, scratch);
  const long n_rows = g->w_row ? g->n_w_rows : g->n_edges;
  const int NT = ef_tiles(ctx, which), a_blocks = (ctx->desc.channels / 4 * NT * 128 + 255) / 256;
  const long groups = (n_rows + 63) / 64;                // of four wavefronts
  const int row_blocks = (int)(groups < 4 * EGNN_CUS ? groups : 4 * EGNN_CUS);
  const int w2_blocks = w2s ? (ctx->n_paths[which] * ctx->desc.channels * EGNN_HIDDEN + 255) / 256 : 0;
  const EfSecond x = {s.length, W_r1, W_r2, s.scales, s.rec, s.A, n_rows, ctx->desc.n_rbf, ctx->n_paths[which], NT,
                      ctx->log2_channels, row_blocks, a_blocks, ctx->desc.r_cut, ef_alpha(ctx, which), (float*)w2s};
  hipLaunchKernelGGL(ef_second_kernel, dim3((unsigned)(row_blocks + a_blocks + w2_blocks)), dim3(256), 0, stream, x);
  EGNN_LAUNCH_CHECK(ctx, "ef_second_kernel");
  return EGNN_OK;
}

int egnn_launch_edge_fused_features(egnn_ctx* ctx, const egnn_graph* g, const float* x_in, const float* W_pre, void* scratch,
                                    hipStream_t stream, float* h) {
  return egnn_launch_node_mix(ctx, x_in, W_pre, nullptr, nullptr, h, g->n_total, stream, 0,
                              egnn_ef_carve(ctx, g, 0, scratch).h4, ef_quads(ctx));
}

int egnn_launch_edge_fused_sum(egnn_ctx* ctx, const egnn_graph* g, void* scratch, float* a, bool half, hipStream_t stream) {
  const EfScratch s = egnn_ef_carve(ctx, g, 0, scratch);
  const int G = ctx->desc.channels / 4;
  const float4* h4 = reinterpret_cast<const float4*>(s.h4);
  const float* scales = s.scales;
  const float scale = 1.0f / sqrtf(ctx->desc.agg_norm);
  // Workgroups: EF_WG_PER_CU on every compute unit, fewer where there are not that many nodes for their wavefronts.  EF_CGX channel
  // groups share an XCD; the sets of them are dealt to the XCDs, and where there are fewer than eight sets, so are the nodes.
  const int per = G < EF_CGX ? G : EF_CGX, sets = G / per;
  const int turns = sets >= 8 ? sets / 8 : 1;
  const int mult = per * turns;                              // workgroups of an XCD that make up one part
  const int parts_per = sets >= 8 ? 1 : 8 / sets;            // parts that the eight XCDs bring at a time
  int i_max = (EGNN_CUS / 8) * EF_WG_PER_CU / mult;
  const int need = (g->n_owned + 3) / 4;                     // parts that still have a node for every wavefront
  const int i_need = (need + parts_per - 1) / parts_per;
  if (i_max < 1) i_max = 1;
  if (i_max > i_need) i_max = i_need;
  const int parts = i_max * parts_per;
  const dim3 grid(8 * i_max * mult), block(256);
#define KERNEL(L, H, S)                                                                                                   \
  hipLaunchKernelGGL((ef_layer_kernel<L, H, S>), grid, block, 0, stream, g->row_ptr, g->src, g->w_row,                      \
                     s.frame, s.rec, s.A, h4, scales, a, \
                     g->n_owned, (int)g->n_edges, ctx->log2_channels,     \
                     parts, scale)
#define LAUNCH(L)                                       \
  case L:                                               \
    if (half && g->w_row) KERNEL(L, true, true);        \
    else if (half) KERNEL(L, true, false);              \
    else if (g->w_row) KERNEL(L, false, true);          \
    else KERNEL(L, false, false);                       \
    break;
  switch (ctx->desc.lmax) {
    LAUNCH(1) LAUNCH(2) LAUNCH(3) LAUNCH(4)
    default: return egnn_fail(ctx, EGNN_EINVAL, "edge_fused: lmax out of range");
  }
#undef LAUNCH
#undef KERNEL
  EGNN_LAUNCH_CHECK(ctx, "ef_layer_kernel");
  return EGNN_OK;
}
