// Reverse pass of the readout where the radial weights' gradient is summed per length interval (grid route, radial_grid.hip): no
// gradient of the weights in memory, channels collapsed and spread on the matrix cores.
//
// Forward (' = in the bond frame, rotated by D_k):  u = D^T Mid(D z ; w),  q[o][M] = sum_c V[o][c] u[(L,M)][c],  H = C q.  Three kernels:
//   ra_couple  dq = C^T dH per edge, by straight-line code per pair of shells (uncouple_gen.inc), in the order of the rows of V;
//   ra_edges   dV[o][c] += sum_M dq[o][M] u[(L,M)][c];   du[(L,M)][c] = sum_o V[o][c] dq[o][M],   dz = D^T Mid^T(w ; D du);
//   ra_bins    dw = Mid^T(D z ; D du) of the edges of an interval, added to six sums per (path, channel) as in tp_bins.hip.
// In the last two a lane is (channel of 16, edge of 4): u[(L,M)] is then the operand (edge, channel) of a 16x16x4 fp32 product with
// 16 rows of V as rows, which gives dV; and du comes out of the products with (edge, order) as rows, V's rows contracted, in the
// lane that goes on with it.
//
// 313,000 edges, lmax 4, 32 channels, 13 orbitals: 95 + 705 + 410 us, in place of 1,550 for the adjoint that wrote dw and 333 for reading it.
// What bounds them, by counters: ra_edges the memory beyond the L2s (3.7 GB of lines miss: weights twice, dz, dq; 5.3 TB/s), with vector
// instructions issuing in 47 % of the SIMD-cycles, matrix cores busy in 17, 15 % of a wavefront's life in waits (775 us and 34 % where an entry of
// w_row was touched in the turn that loads it and four registers were spilled); ra_bins the issue of vector instructions (85 %; 1,200 per
// four edges and 16 channels, two wavefronts a SIMD) and the hand-over from the matrix cores.
#include <algorithm>
#include <type_traits>
#include "egnn_internal.h"
#include "bond_frame.h"
#include "edge_fused.h"
#include "radial_grid.h"
#include "uncouple_gen.inc"

#define RA_D 25                      // (L_READOUT + 1)^2
// dq of an edge: per coupled degree L room for so many rows of V, 2 L + 1 values each, zero past the last row
static constexpr int ra_room[5] = {16, 20, 16, 8, 4};
static constexpr int ra_off[5] = {0, 16, 76, 156, 212};
#define RA_S 248
#define RA_PAST 128                  // words after the last edge's that reads of rows past the last one may touch
#define RA_MAX_Q 192
#define RA_MAX_BLOCKS 64
struct RaRows {                      // rows of V of a degree, first of them
  int n[5], v[5];
};
struct RaTabs {
  int16_t perm[RA_MAX_Q];            // entry of a block -> place among the values in order of the pairs of shells
  int16_t place[RA_S];               // word of dq -> the same, or -1
  int16_t blk[RA_MAX_BLOCKS];        // first value of a pair, the pairs in order of (l_a, l_b)
  int n_blk[9], nq;
};

// ---------------------------------------------------------------------------------------------- dq
// A wavefront takes 16 edges.  out [n_edges + 16][RA_S], the 16 rows past the last edge zero.  Bound by memory: 0.7 + 1 KB an edge.
// (A lane keeps its places of an edge's values; with places looked up per value 196 instead of 97 us for 313,000 edges.)
__global__ __launch_bounds__(256) void ra_couple_kernel(const float* __restrict__ dH, RaTabs tb, float* __restrict__ out, long n_edges,
                                                        const int* __restrict__ route) {
  if (!route[0]) return;
  extern __shared__ float ra_lds[];
  __shared__ int s_perm[RA_MAX_Q], s_place[256], s_blk[RA_MAX_BLOCKS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 15, q = lane >> 4;
  if (tid < RA_MAX_Q) s_perm[tid] = tb.perm[tid];
  s_place[tid] = tid < RA_S ? tb.place[tid] : -1;
  if (tid < RA_MAX_BLOCKS) s_blk[tid] = tb.blk[tid];
  __syncthreads();
  const int nq = tb.nq, nqs = nq | 1;
  float* const mine = ra_lds + (size_t)wave * 16 * nqs;
  const long k0 = ((long)blockIdx.x * 4 + wave) * 16;
  if (k0 >= n_edges + 16) return;                                      // (no barrier beyond)
  {
    int to[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) to[i] = lane + 64 * i < nq ? s_perm[lane + 64 * i] : -1;
    const float* in = dH + k0 * nq + lane;
#pragma unroll
    for (int e0 = 0; e0 < 16; e0 += 8) {
      float x[8][3];
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < 3; ++i)
          x[e][i] = to[i] >= 0 && k0 + e0 + e < n_edges ? __builtin_nontemporal_load(in + (e0 + e) * nq + 64 * i) : 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < 3; ++i)
          if (to[i] >= 0) mine[(e0 + e) * nqs + to[i]] = x[e][i];
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  {
    int first = 0;
    auto couple = [&](auto size, int kind, auto turn) {
      constexpr int N = decltype(size)::value;
      const int count = tb.n_blk[kind];
      for (int r = q; r < count; r += 4) {
        float* x = mine + n * nqs + s_blk[first + r];
        float y[N];
#pragma unroll
        for (int i = 0; i < N; ++i) y[i] = x[i];
        turn(y);
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = y[i];
      }
      first += count;
    };
#define PAIR(a, b) couple(std::integral_constant<int, (2 * a + 1) * (2 * b + 1)>(), 3 * a + b, [](float* y) { egnn_couple_##a##b(y); });
    PAIR(0, 0) PAIR(0, 1) PAIR(0, 2) PAIR(1, 0) PAIR(1, 1) PAIR(1, 2) PAIR(2, 0) PAIR(2, 1) PAIR(2, 2)
#undef PAIR
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  int from[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) from[i] = s_place[lane + 64 * i];
  const int rows = (int)min(16L, n_edges + 16 - k0);
  float* to = out + k0 * RA_S + lane;
#pragma unroll 4
  for (int e = 0; e < rows; ++e)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (lane + 64 * i < RA_S) to[e * RA_S + 64 * i] = from[i] >= 0 ? mine[e * nqs + from[i]] : 0.0f;
}

// ---------------------------------------------------------------------------------------------- what the two kernels share
struct RaArgs {
  const int *src, *dst, *w_row;
  const float4* rhat_d;
  const float *zs, *zt, *w, *V, *dq;
  float *dz, *partial;
  const int *bin_ptr, *perm;
  float* Zp;
  const int* route;
  RaRows rows;
  long n_edges, items_per_xcd;
  int n_vrows;
  float inv_h;
};
constexpr int ra_es(int D) { return ((D * 16 - 16 + 63) / 64) * 64 + 16; }    // an edge's room: banks differ from edge to edge
constexpr int ra_bins_words(int D) { return 8 * ra_es(D) + 4 * RA_S + RA_PAST; }      // of LDS per wavefront
constexpr int ra_edges_words(int D) { return 4 * ra_es(D) + 8 * RA_S + RA_PAST; }
constexpr int ra_log2nb(int LE) { return LE - 4 < 2 ? LE - 4 : 2; }                    // 2^ blocks of 16 channels a workgroup

typedef const __attribute__((address_space(1))) void* ra_gp;
typedef __attribute__((address_space(3))) void* ra_lp;

// rows of four nodes (node of the lane's own edge in j), 16 channels each, from memory to LDS
template <int D, int LE>
__device__ __forceinline__ void ra_load_rows(const float* z, int j, float* to, int lane) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float* r = z + (((size_t)__builtin_amdgcn_readlane(j, 16 * e) * D) << LE);
#pragma unroll
    for (int i = 0; i < (4 * D + 63) / 64; ++i) {
      const int q = 64 * i + lane;
      if (64 * i + 64 <= 4 * D || q < 4 * D)
        __builtin_amdgcn_global_load_lds((ra_gp)(r + (((q >> 2) << LE) + 4 * (q & 3))), (ra_lp)(to + e * ra_es(D) + 256 * i), 16, 0, 0);
    }
  }
}
// V as the products with contracted rows take it: lane (channel, k) holds row 4 s + k of a step, zero past the last
struct RaV { float x[4 + 5 + 4 + 2 + 1]; };
template <int L> constexpr int ra_steps() { return ra_room[L] / 4; }
template <int L> constexpr int ra_step0() { return L == 0 ? 0 : L == 1 ? 4 : L == 2 ? 9 : L == 3 ? 13 : 15; }
template <int L, int LE>
__device__ __forceinline__ void ra_load_v(const RaArgs& g, int ch, int k, RaV& V) {
#pragma unroll
  for (int s = 0; s < ra_steps<L>(); ++s) {
    const int o = 4 * s + k;
    V.x[ra_step0<L>() + s] = o < g.rows.n[L] ? g.V[((size_t)(g.rows.v[L] + o) << LE) + ch] : 0.0f;
  }
}
// du of degree L: rows of a product are (edge, order 4 j + r), so a lane (channel, edge) gets the orders of its own edge
template <int L>
__device__ __forceinline__ void ra_spread(const float* sq, int lane, const RaV& V, float* du) {
  constexpr int W = 2 * L + 1, J = (W + 3) / 4;
  const int r = lane & 3;
  const float* p = sq + ((lane & 15) >> 2) * RA_S + ra_off[L] + (lane >> 4) * W;
  ef_f4 d[J];
#pragma unroll
  for (int j = 0; j < J; ++j) d[j] = ef_f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < ra_steps<L>(); ++s)
#pragma unroll
    for (int j = 0; j < J; ++j)       // (an order past the last: the last again, not used)
      d[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[4 * s * W + (4 * j + 3 < W ? 4 * j + r : 4 * j + min(r, W - 1 - 4 * j))],
                                                  V.x[ra_step0<L>() + s], d[j], 0, 0, 0);
#pragma unroll
  for (int i = 0; i < W; ++i) du[i] = d[i / 4][i % 4];
}
// dV of degree L: += sum over the four edges and the orders of dq[o][M] u[(L,M)][c], 16 rows o (rows past the last: not used)
template <int L>
__device__ __forceinline__ void ra_collapse(const float* sq, int lane, const float* u, int tile, ef_f4& dV) {
  constexpr int W = 2 * L + 1;
  const float* p = sq + (lane >> 4) * RA_S + ra_off[L] + (lane & 15) * W + 16 * W * tile;
  ef_f4 x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int M = 0; M < W; ++M) x = __builtin_amdgcn_mfma_f32_16x16x4f32(p[M], u[M], x, 0, 0, 0);
  dV += x;
}
static_assert(3 * RA_S + 212 + 15 * 9 + 8 < 4 * RA_S + RA_PAST, "reads of rows past the last");
template <int LMAX, int L1>
struct RaDegree {
  using Mid = typename ReadoutMid<LMAX>::T;
  static constexpr int first = Mid::CHUNK_FIRST[L1], count = Mid::CHUNK_COUNT[L1];
  __device__ __forceinline__ static void fwd(const float* v, const float* w, float* u) {
    Mid::template run_l1<L1>(v + L1 * L1, w + first, u);
    if constexpr (L1 < LMAX) RaDegree<LMAX, L1 + 1>::fwd(v, w, u);
  }
  // gradient of the features (the other one is not asked for)
  __device__ __forceinline__ static void feature(const float* w, const float* du, float* gv) {
    float v[2 * L1 + 1], gw[count];
#pragma unroll
    for (int i = 0; i < 2 * L1 + 1; ++i) v[i] = 0.0f;
    Mid::template run_bwd_l1<L1>(v, w + first, du, gv + L1 * L1, gw);
    if constexpr (L1 < LMAX) RaDegree<LMAX, L1 + 1>::feature(w, du, gv);
  }
  __device__ __forceinline__ static void weight(const float* v, const float* du, float* gw) {
    float w[count], gv[2 * L1 + 1];
#pragma unroll
    for (int p = 0; p < count; ++p) w[p] = 0.0f;
    Mid::template run_bwd_l1<L1>(v + L1 * L1, w, du, gv, gw + first);
    if constexpr (L1 < LMAX) RaDegree<LMAX, L1 + 1>::weight(v, du, gw);
  }
};

// ---------------------------------------------------------------------------------------------- dV and dz
template <int LMAX, int LE>        // 2^LE channels
__global__ __launch_bounds__(256, 2) void ra_edges_kernel(RaArgs g) {
  if (!g.route[0]) return;
  using Mid = typename ReadoutMid<LMAX>::T;
  constexpr int D = (LMAX + 1) * (LMAX + 1), P = Mid::P, ES = ra_es(D);
  extern __shared__ __align__(16) float ra_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, e = lane >> 4;
  constexpr int LNB = ra_log2nb(LE), nb = 1 << LNB, phases = 4 >> LNB;
  const int phase = wave >> LNB;
  const int ch0 = ((int)blockIdx.y * nb + (wave & (nb - 1))) * 16, ch = ch0 + c;
  float* const myS = ra_lds + (size_t)wave * ra_edges_words(D);
  float* const myQ = myS + 4 * ES;                                     // two of them
  RaV V;
  ra_load_v<0, LE>(g, ch, e, V); ra_load_v<1, LE>(g, ch, e, V); ra_load_v<2, LE>(g, ch, e, V); ra_load_v<3, LE>(g, ch, e, V); ra_load_v<4, LE>(g, ch, e, V);
  ef_f4 dV[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) dV[i] = ef_f4{0.0f, 0.0f, 0.0f, 0.0f};
  const bool two = g.rows.n[1] > 16;

  // consecutive items (the same destinations, neighbouring sources) go to the same XCD
  const long items = (g.n_edges + 4 * phases - 1) / (4 * phases);
  const long step = gridDim.x >> 3, i0 = (long)(blockIdx.x & 7) * g.items_per_xcd, i1 = min(i0 + g.items_per_xcd, items);
  const unsigned last = (unsigned)(g.n_edges - 1);
  auto first_edge = [&](long it) { return (it * phases + phase) * 4; };
  auto edge = [&](long it) -> unsigned { return min((unsigned)min(first_edge(it), g.n_edges - 1) + e, last); };
  auto load_q = [&](long it, float* to) {                              // (up to 16 rows of zeros follow the last edge's)
    const float* p = g.dq + min(first_edge(it), g.n_edges) * RA_S;
#pragma unroll
    for (int i = 0; i < RA_S; i += 64)
      if (i + 64 <= RA_S || i + lane < RA_S)
        __builtin_amdgcn_global_load_lds((ra_gp)(p + 4 * (i + lane)), (ra_lp)(to + 4 * i), 16, 0, 0);
  };
  long it = i0 + (blockIdx.x >> 3);
  if (it < i1) {
    float w[P], v[D];
    const unsigned k1 = edge(it), k2 = edge(it + step);
    // (the entry of w_row is decoded only where it becomes an address, a turn after its load: see tp_bins.hip)
    auto row_of = [&](unsigned k) { return g.w_row ? g.w_row[k] : (int)k; };
    auto weights = [&](int row) { return g.w + ((size_t)(row < 0 ? ~row : row) * P << LE) + ch; };
    auto target = [&](int d) { return g.zt + ((size_t)d * D << LE) + ch; };
    float4 r1 = g.rhat_d[k1];
    ra_load_rows<D, LE>(g.zs + ch0, g.src[k1], myS, lane);
    load_q(it, myQ);
    {
      const float* const tp = target(g.dst[k1]);
      const float* const wp = weights(row_of(k1));
#pragma unroll
      for (int i = 0; i < D; ++i) v[i] = tp[i << LE];
#pragma unroll
      for (int p = 0; p < P; ++p) w[p] = wp[p << LE];
    }
    int s2 = g.src[k2], d2 = g.dst[k2];
    int w2 = row_of(k2);
    float4 r2 = g.rhat_d[k2];
    float dz[D];
    long done = -1;                    // first edge of the group whose dz is not stored yet
    int turn = 0;
    const int out_at = ((e * D << LE) + ch) * 4;
    auto store = [&]() {               // (stores past the last edge are dropped; addresses per lane were spilled)
      const auto out = __builtin_amdgcn_make_buffer_rsrc(g.dz + ((size_t)done * D << LE), 0,
                                                         ((int)min(4L, g.n_edges - done) * D << LE) * 4, 0x00020000);
#pragma unroll
      for (int i = 0; i < D; ++i) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dz[i]), out, out_at, i << (LE + 2), 2 /* nt */);
    };
    ef_wait_arrived();
    for (; it < i1; it += step) {
      // (The one wait for loads of a turn, weights included, which were asked for in the middle of the turn before.  Leaving those in
      // flight gains nothing: to copy them, or to use them past loads to LDS, the compiler waits for everything.)
      ef_wait_arrived();
      float u[RA_D], wn[P];
#pragma unroll
      for (int i = 0; i < D; ++i) v[i] += myS[e * ES + i * 16 + c];
      const float4 r = r1;
      const float* const sq = myQ + turn * 4 * RA_S;
      turn ^= 1;
      ef_wait_read();
      // (stored only now: a store in flight would hold up the wait above)
      if (done >= 0) store();
      ra_load_rows<D, LE>(g.zs + ch0, s2, myS, lane);                  // (past the last item: its edges once more, not used)
      load_q(it + step, myQ + turn * 4 * RA_S);
      const float *const tp = target(d2), *const wp = weights(w2);
      r1 = r2;
      const unsigned k3 = edge(it + 2 * step);
      s2 = g.src[k3];
      d2 = g.dst[k3];
      w2 = row_of(k3);
      r2 = g.rhat_d[k3];
      __builtin_amdgcn_sched_barrier(0);
      BondTrig t;
      egnn_bond_trig<4>(r.x, r.y, r.z, t);
      egnn_to_bond_frame<LMAX>(v, t);
#pragma unroll
      for (int i = 0; i < RA_D; ++i) u[i] = 0.0f;
      RaDegree<LMAX, 0>::fwd(v, w, u);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < D; ++i) v[i] = tp[i << LE];
      // (the wavefronts of the two halves of a 128-byte line of weights stay together: 40 us less of 835 with the former waits; with
      // loads that bypass the caches 1,020, every line fetched twice)
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < P; ++p) wn[p] = wp[p << LE];
      __builtin_amdgcn_sched_barrier(0);
      egnn_from_bond_frame<4>(u, t);
      ra_collapse<0>(sq, lane, u, 0, dV[0]);
      ra_collapse<1>(sq, lane, u + 1, 0, dV[1]);
      if (two) ra_collapse<1>(sq, lane, u + 1, 1, dV[2]);
      ra_collapse<2>(sq, lane, u + 4, 0, dV[3]);
      ra_collapse<3>(sq, lane, u + 9, 0, dV[4]);
      ra_collapse<4>(sq, lane, u + 16, 0, dV[5]);
      ra_spread<0>(sq, lane, V, u);
      ra_spread<1>(sq, lane, V, u + 1);
      ra_spread<2>(sq, lane, V, u + 4);
      ra_spread<3>(sq, lane, V, u + 9);
      ra_spread<4>(sq, lane, V, u + 16);
      egnn_to_bond_frame<4>(u, t);
      RaDegree<LMAX, 0>::feature(w, u, dz);
      egnn_from_bond_frame<LMAX>(dz, t);
      done = first_edge(it) < g.n_edges ? first_edge(it) : -1;
#pragma unroll
      for (int p = 0; p < P; ++p) w[p] = wn[p];
    }
    if (done >= 0) store();
    ef_wait_arrived();                 // (nothing is on its way to LDS when it is used for the sums)
  }
  // one partial [n_vrows][channels] per workgroup: its wavefronts of the same channels added in fixed order
  __syncthreads();
  float* const red = ra_lds + (size_t)wave * g.n_vrows * 16;
  auto put = [&](int L, int tile, const ef_f4& x) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (16 * tile + 4 * e + r < g.rows.n[L]) red[(g.rows.v[L] + 16 * tile + 4 * e + r) * 16 + c] = x[r];
  };
  put(0, 0, dV[0]); put(1, 0, dV[1]); put(1, 1, dV[2]); put(2, 0, dV[3]); put(3, 0, dV[4]); put(4, 0, dV[5]);
  __syncthreads();
  for (int i = tid; i < (g.n_vrows * 16) << LNB; i += 256) {
    const int b = i / (g.n_vrows * 16), x = i - b * g.n_vrows * 16;
    float sum = 0.0f;
    for (int p = 0; p < phases; ++p) sum += ra_lds[(size_t)(p * nb + b) * g.n_vrows * 16 + x];
    g.partial[(((size_t)blockIdx.x * g.n_vrows + (x >> 4)) << LE) + ((int)blockIdx.y * nb + b) * 16 + (x & 15)] = sum;
  }
}

// ---------------------------------------------------------------------------------------------- dw, per interval of lengths
// rows[i] of lane row r <-> rows[r] of lane row i
__device__ __forceinline__ void ra_turn(float& a, float& b, float& c, float& d) {
  auto s32 = [](float& x, float& y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
  };
  auto s16 = [](float& x, float& y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
  };
  s32(a, c); s32(b, d);
  s16(a, b); s16(c, d);
}

template <int LMAX, int LE>        // 2^LE channels
__global__ __launch_bounds__(256, 2) void ra_bins_kernel(RaArgs g) {
  if (!g.route[0]) return;
  using Mid = typename ReadoutMid<LMAX>::T;
  constexpr int D = (LMAX + 1) * (LMAX + 1), P = Mid::P, QP = (P + 3) / 4, ES = ra_es(D);
  extern __shared__ __align__(16) float ra_lds[];
  const int m = RG_BINS - 1 - (int)blockIdx.x;                         // longest (fullest) intervals first
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, e = lane >> 4;
  constexpr int LNB = ra_log2nb(LE), nb = 1 << LNB, phases = 4 >> LNB;
  const int phase = wave >> LNB;
  const int ch0 = ((int)blockIdx.y * nb + (wave & (nb - 1))) * 16, ch = ch0 + c;
  float* const myS = ra_lds + (size_t)wave * ra_bins_words(D);
  float* const myT = myS + 4 * ES;
  float* const myQ = myT + 4 * ES;
  const int c0 = g.bin_ptr[m], c1 = g.bin_ptr[m + 1], PE = P << LE;
  float acc[QP][RG_PTS];
#pragma unroll
  for (int i = 0; i < QP; ++i)
#pragma unroll
    for (int k = 0; k < RG_PTS; ++k) acc[i][k] = 0.0f;
  const int begin = c0 + 4 * phase, step = 4 * phases;
  if (begin < c1) {
    RaV V;
    ra_load_v<0, LE>(g, ch, e, V); ra_load_v<1, LE>(g, ch, e, V); ra_load_v<2, LE>(g, ch, e, V); ra_load_v<3, LE>(g, ch, e, V); ra_load_v<4, LE>(g, ch, e, V);
    // (in range only where it becomes an index, a turn after its load: see tp_bins.hip)
    auto edge_at = [&](int at) { return g.perm[min(at + e, c1 - 1)]; };
    auto in_range = [&](int k) { return min(max(k, 0), (int)g.n_edges - 1); };
    auto load_q = [&](int k) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float* p = g.dq + (size_t)__builtin_amdgcn_readlane(k, 16 * i) * RA_S;
        if (lane < RA_S / 4) __builtin_amdgcn_global_load_lds((ra_gp)(p + 4 * lane), (ra_lp)(myQ + i * RA_S), 16, 0, 0);
      }
    };
    const int k1 = in_range(edge_at(begin));
    int k2 = in_range(edge_at(begin + step)), k3 = edge_at(begin + 2 * step);
    int s2 = g.src[k2], d2 = g.dst[k2];
    float4 r1 = g.rhat_d[k1], r2 = g.rhat_d[k2];
    ra_load_rows<D, LE>(g.zs + ch0, g.src[k1], myS, lane);
    ra_load_rows<D, LE>(g.zt + ch0, g.dst[k1], myT, lane);
    load_q(k1);
    for (int at = begin; at < c1; at += step) {
      ef_wait_arrived();
      float v[D], du[RA_D], gw[4 * QP];
#pragma unroll
      for (int i = 0; i < D; ++i) v[i] = myS[e * ES + i * 16 + c] + myT[e * ES + i * 16 + c];
      const float4 r = r1;
      const bool valid = at + e < c1;
      ra_spread<0>(myQ, lane, V, du);
      ra_spread<1>(myQ, lane, V, du + 1);
      ra_spread<2>(myQ, lane, V, du + 4);
      ra_spread<3>(myQ, lane, V, du + 9);
      ra_spread<4>(myQ, lane, V, du + 16);
      ef_wait_read();
      // (the last group's are loaded once more by the ones after it)
      ra_load_rows<D, LE>(g.zs + ch0, s2, myS, lane);
      ra_load_rows<D, LE>(g.zt + ch0, d2, myT, lane);
      load_q(k2);
      r1 = r2;
      k2 = in_range(k3);
      s2 = g.src[k2];
      d2 = g.dst[k2];
      r2 = g.rhat_d[k2];
      k3 = edge_at(at + 3 * step);
      __builtin_amdgcn_sched_barrier(0);
      BondTrig t;
      egnn_bond_trig<4>(r.x, r.y, r.z, t);
      egnn_to_bond_frame<LMAX>(v, t);
      egnn_to_bond_frame<4>(du, t);
#pragma unroll
      for (int p = P; p < 4 * QP; ++p) gw[p] = 0.0f;
      RaDegree<LMAX, 0>::weight(v, du, gw);
      float phi[RG_PTS], ph[4][RG_PTS];
      rg_weights(r.w * g.inv_h - (float)m, phi);
#pragma unroll
      for (int k = 0; k < RG_PTS; ++k) {
        const float x = valid ? phi[k] : 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) ph[i][k] = x;
        ra_turn(ph[0][k], ph[1][k], ph[2][k], ph[3][k]);
      }
#pragma unroll
      for (int i = 0; i < QP; ++i) {
        ra_turn(gw[i], gw[QP + i], gw[2 * QP + i], gw[3 * QP + i]);    // the lane's quarter of the paths, of four edges
#pragma unroll
        for (int k = 0; k < RG_PTS; ++k)
#pragma unroll
          for (int x = 0; x < 4; ++x) acc[i][k] += ph[x][k] * gw[x * QP + i];
      }
    }
    ef_wait_arrived();                 // (nothing is on its way to LDS when it is used for the sums)
  }
  float* const red = ra_lds;           // [wave][value][lane]
#pragma unroll
  for (int k = 0; k < RG_PTS; ++k) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < QP; ++i) red[(wave * QP + i) * 64 + lane] = acc[i][k];
    __syncthreads();
    float* out = g.Zp + ((size_t)m * RG_PTS + k) * PE + (int)blockIdx.y * nb * 16;
    for (int x = tid; x < (P * 16) << LNB; x += 256) {
      const int cc = x & (16 * nb - 1), p = x >> (4 + LNB), b = cc >> 4;
      float sum = 0.0f;
      for (int f = 0; f < phases; ++f) sum += red[((f * nb + b) * QP + p % QP) * 64 + 16 * (p / QP) + (cc & 15)];
      out[((size_t)p << LE) + cc] = sum;
    }
  }
}

// ---------------------------------------------------------------------------------------------- host side
static int ra_vrows(const egnn_ctx* ctx) {
  int n = 0;
  for (int L = 0; L <= EGNN_L_READOUT; ++L) n += ctx->n_out[L];
  return n;
}
// workgroups per XCD of ra_edges: two on every compute unit, fewer where there are not that many items
static long ra_per_xcd(const egnn_ctx* ctx, int64_t n_edges, long* items_per_xcd) {
  const int lnb = ra_log2nb(ctx->log2_channels), edges = 16 >> lnb, ny = (ctx->desc.channels / 16) >> lnb;
  const long items = (n_edges + edges - 1) / edges;
  *items_per_xcd = (items + 7) / 8;
  return std::min<long>(*items_per_xcd, EGNN_CUS / 8 * 2 / ny);
}

// The fewest edges from which these kernels are the faster ones, whole adjoint calls against the kernels with dw in memory, 60 .. 2,500 atoms,
// 19 .. 107 edges an atom.  Room for the rows of V is fixed, so that few orbitals gain less, and every interval costs a workgroup.
//   12 and 13 orbitals, from 12,000 edges: 16 channels (lmax 3, 4) 1.00 .. 1.50, 32 (lmax 2 to 4) 1.01 .. 1.32, 64 1.12 .. 1.52, at lmax 4 1.35 ..
//     2.0, 128 1.13 .. 1.9.  At 5,700 edges 0.92 (32 channels) .. 1.22.
//   4, 8 and 9: lmax 4 with 64 and 128 channels 1.09 .. 1.63 from 5,700 edges; with 16 and 32 0.95 .. 1.01 at 19,000, 1.00 .. 1.30 from 42,000
//     on.  lmax 3 with 128 channels 1.1 .. 1.3 from 19,000; with 64 1.01 .. 1.10 from there (4 orbitals 0.97 .. 1.05: not taken); with 32
//     1.01 .. 1.08 from 42,000 (4 orbitals 0.96 .. 1.01: not taken); with 16 1.02 .. 1.24 from 42,000.  lmax 1 and 2 0.74 .. 1.03: not taken.
static int64_t ra_least_edges(int lmax, int E, int n_orb) {
  const int64_t never = INT64_MAX;
  if (n_orb >= 12) return 12000;
  if (lmax == 4) return E >= 64 ? 12000 : 40000;
  if (lmax == 3) return E == 128 ? 18000 : E == 16 ? 40000 : n_orb < 8 ? never : E == 64 ? 18000 : 40000;
  return never;
}

bool egnn_readout_adjoint_fits(const egnn_ctx* ctx, int64_t n_edges) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels, nq = ctx->n_orb * ctx->n_orb;
  if (lmax < 1 || E < 16 || nq < 1 || nq > RA_MAX_Q || ctx->desc.n_orb_shells * ctx->desc.n_orb_shells > RA_MAX_BLOCKS) return false;
  if (n_edges < ra_least_edges(lmax, E, ctx->n_orb)) return false;
  for (int L = 0; L <= EGNN_L_READOUT; ++L)
    if (ctx->n_out[L] > ra_room[L]) return false;
  const int D = (lmax + 1) * (lmax + 1), P = ctx->n_paths[1];
  long items;
  return ra_vrows(ctx) * 16 <= ra_edges_words(D) && (P + 3) / 4 * 64 <= ra_bins_words(D) && (n_edges + 16) * RA_S <= n_edges * P * E &&
         (size_t)8 * ra_per_xcd(ctx, n_edges, &items) * ra_vrows(ctx) * E * sizeof(float) <= egnn_readout_backward_partial_bytes(ctx, n_edges);
}

static RaArgs ra_args(const egnn_ctx* ctx, const egnn_graph* g, const ReadoutAdjoint& a) {
  RaArgs x = {};
  x.src = g->src; x.dst = g->dst; x.w_row = a.shared_rows ? g->w_row : nullptr;
  x.rhat_d = reinterpret_cast<const float4*>(a.rhat_d);
  x.zs = a.zs; x.zt = a.zt; x.w = a.w; x.V = a.V; x.dq = a.dq; x.dz = a.dz; x.partial = a.partial; x.route = a.route;
  for (int L = 0, v = 0; L <= EGNN_L_READOUT; ++L) { x.rows.n[L] = ctx->n_out[L]; x.rows.v[L] = v; v += ctx->n_out[L]; }
  x.n_edges = g->n_edges; x.n_vrows = ra_vrows(ctx);
  x.inv_h = (float)RG_BINS / ctx->desc.r_cut;
  return x;
}
template <int LMAX, int LE>
static int ra_launch(egnn_ctx* ctx, bool bins, dim3 grid, const RaArgs& x, hipStream_t st) {
  constexpr int D = (LMAX + 1) * (LMAX + 1);
  const auto kernel = bins ? ra_bins_kernel<LMAX, LE> : ra_edges_kernel<LMAX, LE>;
  const int shmem = 16 * (bins ? ra_bins_words(D) : ra_edges_words(D));
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, shmem);
  if (e != hipSuccess) return egnn_check_hip(ctx, e, "hipFuncSetAttribute(readout adjoint)");
  hipLaunchKernelGGL(kernel, grid, dim3(256), shmem, st, x);
  EGNN_LAUNCH_CHECK(ctx, bins ? "ra_bins_kernel" : "ra_edges_kernel");
  return EGNN_OK;
}
static int ra_launch(egnn_ctx* ctx, bool bins, unsigned grid_x, const RaArgs& x, hipStream_t st) {
  const dim3 grid(grid_x, (ctx->desc.channels / 16) >> ra_log2nb(ctx->log2_channels));
#define BY_CHANNELS(L)                                                          \
  case L:                                                                       \
    switch (ctx->log2_channels) {                                               \
      case 4: return ra_launch<L, 4>(ctx, bins, grid, x, st);                   \
      case 5: return ra_launch<L, 5>(ctx, bins, grid, x, st);                   \
      case 6: return ra_launch<L, 6>(ctx, bins, grid, x, st);                   \
      case 7: return ra_launch<L, 7>(ctx, bins, grid, x, st);                   \
    }                                                                           \
    break;
  switch (ctx->desc.lmax) {
    BY_CHANNELS(1) BY_CHANNELS(2) BY_CHANNELS(3) BY_CHANNELS(4)
  }
#undef BY_CHANNELS
  return egnn_fail(ctx, EGNN_EINVAL, "readout adjoint: lmax or channels out of range");
}

int egnn_launch_readout_adjoint(egnn_ctx* ctx, const egnn_graph* g, const ReadoutAdjoint& a, const float* dH, float* dV, hipStream_t st) {
  RaTabs tb = {};
  const int nq = ctx->n_orb * ctx->n_orb, ns = ctx->desc.n_orb_shells;
  const int* ol = ctx->desc.orb_l;
  RaArgs x = ra_args(ctx, g, a);
  tb.nq = nq;
  for (int i = 0; i < RA_S; ++i) tb.place[i] = -1;
  for (int i = 0; i < ctx->n_slots; ++i) {
    const int L = ctx->slot_L[i];
    for (int M = 0; M < 2 * L + 1; ++M)
      tb.place[ra_off[L] + (ctx->slot_vrow[i] - x.rows.v[L]) * (2 * L + 1) + M] = (int16_t)(ctx->slot_qoff[i] + M);
  }
  int n_blk = 0;
  for (int kind = 0; kind < 9; ++kind)
    for (int s = 0, at = 0, row = 0; s < ns; row += 2 * ol[s] + 1, ++s)
      for (int t = 0, col = 0; t < ns; col += 2 * ol[t] + 1, ++t) {
        const int nt = 2 * ol[t] + 1;
        if (3 * ol[s] + ol[t] == kind) {
          tb.blk[n_blk++] = (int16_t)at;
          tb.n_blk[kind]++;
          for (int i = 0; i < (2 * ol[s] + 1) * nt; ++i) tb.perm[(row + i / nt) * ctx->n_orb + col + i % nt] = (int16_t)(at + i);
        }
        at += (2 * ol[s] + 1) * nt;
      }
  const long groups = (g->n_edges + 16 + 15) / 16;
  hipLaunchKernelGGL(ra_couple_kernel, dim3((unsigned)((groups + 3) / 4)), dim3(256), 64 * (nq | 1) * sizeof(float), st, dH, tb,
                     const_cast<float*>(a.dq), (long)g->n_edges, a.route);
  EGNN_LAUNCH_CHECK(ctx, "ra_couple_kernel");
  const long per_xcd = ra_per_xcd(ctx, g->n_edges, &x.items_per_xcd);
  const int rc = ra_launch(ctx, false, (unsigned)(8 * per_xcd), x, st);
  if (rc) return rc;
  return egnn_launch_reduce_partials(ctx, a.partial, (int)(8 * per_xcd), (long)x.n_vrows * ctx->desc.channels, dV, 1.0f, st, a.route + 1);
}

int egnn_launch_readout_bins(egnn_ctx* ctx, const egnn_graph* g, const ReadoutAdjoint& a, const int* bin_ptr, const int* perm, float* Zp,
                             hipStream_t st) {
  RaArgs x = ra_args(ctx, g, a);
  x.bin_ptr = bin_ptr; x.perm = perm; x.Zp = Zp;
  return ra_launch(ctx, true, RG_BINS, x, st);
}
