// S3 + S6 in one kernel: the readout with its radial weights made on the matrix cores in the registers of the lanes that use them,
// as in edge_fused.hip, and the channels collapsed on the matrix cores from where the product leaves them.
//
// Work: a wavefront takes 16 edges and goes through all groups of 4 channels; eight wavefronts share the pieces of W_r2, which
// come group by group from memory to LDS while the vector work of the group before runs (a barrier on either side).  After the
// product a lane (n, q) holds, of degree L and order M, the value of edge n and channel 4 group + q: that is the second
// operand of a 16x16x4 fp32 product with 16 rows of V_L.  9 products do degrees 0 to 2; degrees 3 and 4 (up to 5 rows and 1)
// and a 17th row of degree 1 are vector work, 47 sums a lane (as products their 16-row tiles would be nearly empty).  After the
// last group the collapsed values go through LDS: every pair of shells is turned into its block by straight-line code with the
// coupling constants (uncouple_gen.inc), and 16 blocks leave as one contiguous run.  With a list of coefficients per entry, as
// in readout.hip, that last part took 235 of 790 us.
//
// Before: weights through memory (1.0 GB written and read in half precision at 1,777 atoms, 371,000 edges, 32 channels, lmax 4)
// and the collapse from LDS: 297 + 577 us, now 630 + 45 of preparation; 1,000 atoms, lmax 3: 45 + 177 -> 140 + 19.  What bounds it:
// the matrix-core and the vector work of a group in turn (copies without the one took 600 of 790 us, without the other 655), 44
// LDS reads of 1 KB a group and wavefront, and the waits at the barriers.  Counters at 1,777 atoms: 2.0 GHz, vector instructions issue
// in 54 % of the SIMD-cycles, matrix cores busy in 20 %, LDS in 21 %, waiting 27 % of a wave's life.
#include <type_traits>
#include "egnn_internal.h"
#include "bond_frame.h"
#include "half_scales.h"
#include "edge_fused.h"
#include "uncouple_gen.inc"

#define RF_WAVES 8
#define RF_D 25                     // (L_READOUT + 1)^2
// rows of V per coupled degree that the kernel has room for: 16 in a matrix-core tile for L <= 2 (and one more for L = 1), the
// others as vector work
static constexpr int rf_room[5] = {16, 17, 16, 5, 1};
#define RF_MAX_Q 192                 // 16 + 3 * 17 + 5 * 16 + 7 * 5 + 9 = 191 collapsed values at most
#define RF_MAX_BLOCKS 56             // a pair of shells has a row of V of its own in some degree
// What the kernel knows of the orbitals, passed by value.
// pos: where the collapsed value of (degree, order, row of V) goes: 9 (degree, order) pairs of 16 rows for the matrix cores'
// results, then 48 for the vector work's: 3 orders of the 17th row of degree 1, 7 orders x 5 rows of degree 3, 9 orders of
// degree 4, one unused; values without a place go to word nq.  perm: where the entry u of a block lies among the values of
// its edge, which are in order of the pairs of shells.  blk: first value of a pair, the pairs in order of (l_a, l_b), n_blk of each.
#define RF_POS (9 * 16 + 48)
struct RfTabs {
  int16_t pos[RF_POS], perm[RF_MAX_Q], blk[RF_MAX_BLOCKS];
  int n_blk[9], nq;
  int n[5], off[5];                  // rows of V of a degree, index of the first of them
};

// Sums over the four rows of 16 lanes, shared out: row r ends with values 12 r .. 12 r + 11 in x[0 .. 11].  A swap of halves
// leaves each half with the two parts of one of the two values.
__device__ __forceinline__ void rf_sum_rows(float (&x)[48]) {
#pragma unroll
  for (int i = 0; i < 24; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i + 24]), false, false);
    x[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[i]), __float_as_uint(x[i + 12]), false, false);
    x[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
}

template <int LMAX, bool HALF>
__global__ __launch_bounds__(64 * RF_WAVES, 2) void rf_kernel(
    const int* __restrict__ src, const int* __restrict__ dst, const int* __restrict__ w_row,
    const float4* __restrict__ frame, const uint4* __restrict__ rec, const uint4* __restrict__ A,
    const float4* __restrict__ s4, const float4* __restrict__ t4, const float* __restrict__ scales,
    const float* __restrict__ V, RfTabs tb, float* __restrict__ H, long n_edges, int log2E, int stage_words,
    long batches_per_xcd) {
  using Mid = typename ReadoutMid<LMAX>::T;
  constexpr int D = (LMAX + 1) * (LMAX + 1), P = Mid::P, NT = (P + 3) / 4, NQ = (D + 3) / 4;
  extern __shared__ uint4 smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = 1 << (log2E - 2), E = 1 << log2E;
  uint4* const sA = smem;                                              // [NT][2 steps][2 pieces][64]
  float* const stage0 = reinterpret_cast<float*>(sA + NT * 256);       // per wavefront: features, then collapsed values
  float* const sVm = stage0 + RF_WAVES * stage_words;                  // [3][G][64]  V as the matrix cores take it
  float* const sVv = sVm + 3 * G * 64;                                 // [G][4][8]   the rows of the vector work
  int* const s_pos = reinterpret_cast<int*>(sVv + G * 32);             // [RF_POS]
  int* const s_perm = s_pos + RF_POS;                                  // [RF_MAX_Q]
  int* const s_blk = s_perm + RF_MAX_Q;                                // [RF_MAX_BLOCKS]
  const int nq = tb.nq, nqs = (nq + 1) | 1;
  for (int i = tid; i < 3 * G * 64; i += 64 * RF_WAVES) {
    const int L = i / (G * 64), cg = (i >> 6) & (G - 1), m = i & 15, k = (i >> 4) & 3;
    sVm[i] = m < tb.n[L] ? V[(size_t)(tb.off[L] + m) * E + 4 * cg + k] : 0.0f;
  }
  for (int i = tid; i < G * 32; i += 64 * RF_WAVES) {
    const int u = i & 7, c = (i >> 3);                                 // c = channel
    const int L = u == 0 ? 1 : u < 6 ? 3 : 4, m = u == 0 ? 16 : u < 6 ? u - 1 : 0;
    sVv[i] = u < 7 && m < tb.n[L] ? V[(size_t)(tb.off[L] + m) * E + c] : 0.0f;
  }
  for (int i = tid; i < RF_POS; i += 64 * RF_WAVES) s_pos[i] = tb.pos[i];
  for (int i = tid; i < RF_MAX_Q; i += 64 * RF_WAVES) s_perm[i] = tb.perm[i];
  for (int i = tid; i < RF_MAX_BLOCKS; i += 64 * RF_WAVES) s_blk[i] = tb.blk[i];
  __syncthreads();
  float s_w, s_g, unscale;
  half_scales_of(scales, s_w, s_g, unscale);
  const int ex = ilogbf(unscale), exh = ex / 2;                        // (undone half before and half after the product)
  const float f = HALF ? 1.0f : ldexpf(1.0f, exh);
  const float fin = HALF ? 1.0f : ldexpf(1.0f, ex - 2 * exh);

  const int n = lane & 15, q = lane >> 4;
  const int e4 = lane >> 2, p4 = (lane & 3) ^ (lane >> 4), at4 = 4 * n + (q ^ (n >> 2));
  uint4* const myS = reinterpret_cast<uint4*>(stage0 + (size_t)wave * stage_words);
  float* const sq = stage0 + (size_t)wave * stage_words;
  const unsigned last = (unsigned)(n_edges - 1);
  auto edge = [&](long k, int i) -> unsigned { return min((unsigned)min(k, n_edges - 1) + i, last); };   // k + i, or the last one
  auto load_A = [&](int cg) {
    const uint4* p = A + (size_t)cg * NT * 256 + lane;
#pragma unroll
    for (int i = 0; i < (NT * 4 + RF_WAVES - 1) / RF_WAVES; ++i) {
      const int c = i * RF_WAVES + wave;
      if (c < NT * 4)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p + 64 * c),
                                         (__attribute__((address_space(3))) void*)(sA + 64 * c), 16, 0, 0);
    }
  };
  auto load_s = [&](int s, int cg) {
    const float4* p = s4 + ((size_t)s * G + cg) * (NQ * 4) + p4;
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p + 4 * i),
                                       (__attribute__((address_space(3))) void*)(myS + 64 * i), 16, 0, 0);
  };
  // consecutive batches of 8 x 16 edges (the same destinations, neighbouring sources) go to the same XCD
  const long b_first = (long)(blockIdx.x & 7) * batches_per_xcd, b_step = gridDim.x >> 3;
  const long b_end = min(b_first + batches_per_xcd, (n_edges + 16 * RF_WAVES - 1) / (16 * RF_WAVES));
  long batch = b_first + (blockIdx.x >> 3);
  if (batch >= b_end) return;
  // of a tile: the source of the edge that the lane brings to LDS, destination, row of weights and frame of the edge it works on
  int s_e, d, raw;
  float4 fr;
  uint4 b[2][2];
  auto load_rec = [&]() {
    const uint4* rp = rec + (size_t)(w_row && raw < 0 ? ~raw : raw) * 16 + q;
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i >> 1][i & 1] = rp[4 * i];
  };
  {
    const long k0 = (batch * RF_WAVES + wave) * 16;
    const unsigned kk = edge(k0, n);
    s_e = src[edge(k0, e4)];
    d = dst[kk];
    raw = w_row ? w_row[kk] : (int)kk;
    fr = frame[kk];
    load_rec();
  }
  load_A(0);
  load_s(s_e, 0);
  for (; batch < b_end; batch += b_step) {
    const long k0 = (batch * RF_WAVES + wave) * 16;                    // (past the last edge: works on it, stores nothing)
    // (of the wavefront's next tile; past its last: some edge's, not used)
    const long k_next = k0 + b_step * (16 * RF_WAVES);
    const unsigned kk_next = edge(k_next, n);
    const int s_next = src[edge(k_next, e4)], d_next = dst[kk_next], raw_next = w_row ? w_row[kk_next] : (int)kk_next;
    ef_f4 m0 = {0.0f, 0.0f, 0.0f, 0.0f}, m1[3], m2[5];
    float pv[48];
#pragma unroll
    for (int i = 0; i < 3; ++i) m1[i] = m0;
#pragma unroll
    for (int i = 0; i < 5; ++i) m2[i] = m0;
#pragma unroll
    for (int i = 0; i < 48; ++i) pv[i] = 0.0f;

    for (int cg = 0; cg < G; ++cg) {
      ef_wait_arrived();
      __builtin_amdgcn_s_barrier();                                    // all parts of W_r2's group are there
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
      float4 zt[NQ];
      {
        const float4* tp = t4 + ((size_t)d * G + cg) * (NQ * 4) + q;
#pragma unroll
        for (int i = 0; i < NQ; ++i) zt[i] = tp[4 * i];
      }
      __builtin_amdgcn_sched_barrier(0);
      ef_f4 c[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) c[t] = ef_f4{0.0f, 0.0f, 0.0f, 0.0f};
      // (the four correction products first: then the sum is rounded at its full size twice, not six times)
      ef_h8 bh[2], bl[2];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) { bh[ks] = __builtin_bit_cast(ef_h8, b[ks][0]); bl[ks] = __builtin_bit_cast(ef_h8, b[ks][1]); }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        ef_h8 hi[2], lo[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          hi[ks] = __builtin_bit_cast(ef_h8, sA[(t * 2 + ks) * 128 + lane]);
          lo[ks] = __builtin_bit_cast(ef_h8, sA[(t * 2 + ks) * 128 + 64 + lane]);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          c[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi[ks], bl[ks], c[t], 0, 0, 0);
          c[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo[ks], bh[ks], c[t], 0, 0, 0);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) c[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi[ks], bh[ks], c[t], 0, 0, 0);
      }
      float w[NT * 4];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) w[4 * t + r] = HALF ? (float)(_Float16)(c[t][r] * unscale) : c[t][r];
      float v[NQ * 4], o[RF_D];
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const uint4 x = myS[64 * i + at4];
        v[4 * i] = __uint_as_float(x.x) + zt[i].x; v[4 * i + 1] = __uint_as_float(x.y) + zt[i].y;
        v[4 * i + 2] = __uint_as_float(x.z) + zt[i].z; v[4 * i + 3] = __uint_as_float(x.w) + zt[i].w;
      }
      __builtin_amdgcn_sched_barrier(0);
      ef_wait_read();
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      __builtin_amdgcn_s_barrier();                                    // all wavefronts have read it
      load_A(cg + 1 < G ? cg + 1 : 0);
      if (cg + 1 < G) load_s(s_e, cg + 1);
      BondTrig t;
      t.cp[0] = 1.0f; t.sp[0] = 0.0f; t.ct[0] = 1.0f; t.st[0] = 0.0f;
      t.cp[1] = fr.x; t.sp[1] = fr.y; t.ct[1] = fr.z; t.st[1] = fr.w;
#pragma unroll
      for (int m = 2; m <= 4; ++m) {
        t.cp[m] = t.cp[m - 1] * fr.x - t.sp[m - 1] * fr.y;
        t.sp[m] = t.sp[m - 1] * fr.x + t.cp[m - 1] * fr.y;
        t.ct[m] = t.ct[m - 1] * fr.z - t.st[m - 1] * fr.w;
        t.st[m] = t.st[m - 1] * fr.z + t.ct[m - 1] * fr.w;
      }
      if (!HALF) {
#pragma unroll
        for (int m = 1; m <= 4; ++m) { t.cp[m] *= f; t.sp[m] *= f; }
#pragma unroll
        for (int l = 0; l <= LMAX; ++l) v[l * l + l] *= f;
      }
      egnn_to_bond_frame<LMAX>(v, t);
      Mid::run(v, w, o);
      egnn_from_bond_frame<4>(o, t);
      if (!HALF) {
#pragma unroll
        for (int l = 0; l <= 4; ++l) o[l * l + l] *= f;
      }
      // collapse of the group's channels: what a lane holds of degree L and order M is the operand's element (channel, edge)
      const float a0 = sVm[cg * 64 + lane], a1 = sVm[(G + cg) * 64 + lane], a2 = sVm[(2 * G + cg) * 64 + lane];
      // (each product from zero: the running sums of 16 .. 128 channels are then rounded once per group, not per channel)
      const ef_f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
      m0 += __builtin_amdgcn_mfma_f32_16x16x4f32(a0, o[0], zero, 0, 0, 0);
#pragma unroll
      for (int M = 0; M < 3; ++M) m1[M] += __builtin_amdgcn_mfma_f32_16x16x4f32(a1, o[1 + M], zero, 0, 0, 0);
#pragma unroll
      for (int M = 0; M < 5; ++M) m2[M] += __builtin_amdgcn_mfma_f32_16x16x4f32(a2, o[4 + M], zero, 0, 0, 0);
      const float4 va = *reinterpret_cast<const float4*>(sVv + (cg * 4 + q) * 8), vb = *reinterpret_cast<const float4*>(sVv + (cg * 4 + q) * 8 + 4);
#pragma unroll
      for (int M = 0; M < 3; ++M) pv[M] += va.x * o[1 + M];
#pragma unroll
      for (int M = 0; M < 7; ++M) {
        pv[3 + 5 * M] += va.y * o[9 + M];
        pv[4 + 5 * M] += va.z * o[9 + M];
        pv[5 + 5 * M] += va.w * o[9 + M];
        pv[6 + 5 * M] += vb.x * o[9 + M];
        pv[7 + 5 * M] += vb.y * o[9 + M];
      }
#pragma unroll
      for (int M = 0; M < 9; ++M) pv[38 + M] += vb.z * o[16 + M];
    }

    raw = raw_next;
    d = d_next;
    fr = frame[kk_next];
    load_rec();
    // collapsed values to LDS (where the features were), then the blocks
    float* const mine = sq + n * nqs;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const int4 at = *reinterpret_cast<const int4*>(s_pos + 16 * i + 4 * q);
      const ef_f4 x = i == 0 ? m0 : i < 4 ? m1[i - 1] : m2[i - 4];
      mine[at.x] = x[0];
      mine[at.y] = x[1];
      mine[at.z] = x[2];
      mine[at.w] = x[3];
    }
    rf_sum_rows(pv);
#pragma unroll
    for (int i = 0; i < 12; i += 4) {
      const int4 at = *reinterpret_cast<const int4*>(s_pos + 144 + 12 * q + i);
      mine[at.x] = pv[i];
      mine[at.y] = pv[i + 1];
      mine[at.z] = pv[i + 2];
      mine[at.w] = pv[i + 3];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    // the coupled values of a pair of shells become its block in place, a lane at a time: four pairs of a kind by the four rows
    {
      int first = 0;
      auto uncouple = [&](auto size, int kind, auto turn) {
        constexpr int N = decltype(size)::value;
        const int count = tb.n_blk[kind];
        for (int r = 0; r < count; r += 4)
          if (r + q < count) {
            float* x = mine + s_blk[first + r + q];
            float y[N];
#pragma unroll
            for (int i = 0; i < N; ++i) y[i] = x[i];
            turn(y);
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = y[i];
          }
        first += count;
      };
#define PAIR(a, b) \
  uncouple(std::integral_constant<int, (2 * a + 1) * (2 * b + 1)>(), 3 * a + b, [](float* y) { egnn_uncouple_##a##b(y); });
      PAIR(0, 0) PAIR(0, 1) PAIR(0, 2) PAIR(1, 0) PAIR(1, 1) PAIR(1, 2) PAIR(2, 0) PAIR(2, 1) PAIR(2, 2)
#undef PAIR
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    {
      float* out = H + k0 * nq;
      const int m20 = ((1 << 20) + nq - 1) / nq;                       // i / nq = i * m20 >> 20 for i < 16 * 191
#pragma unroll 4
      for (int i = lane; i < 16 * nq; i += 64) {
        const int e = (i * m20) >> 20;
        const float x = fin * sq[e * nqs + s_perm[i - e * nq]];
        if (k0 + e < n_edges) __builtin_nontemporal_store(x, out + i);
      }
    }
    s_e = s_next;
    ef_wait_read();
    load_s(s_e, 0);                                                    // (past the wavefront's last batch: read and not used)
  }
  ef_wait_arrived();                 // (nothing is on its way to LDS when the workgroup gives it back)
}

static size_t rf_stage_words(const egnn_ctx* ctx) {
  const size_t nq = (size_t)ctx->n_orb * ctx->n_orb, a = (size_t)ef_quads(ctx) * 256, b = 16 * ((nq + 1) | 1);
  return ((a > b ? a : b) + 3) & ~(size_t)3;
}
static size_t rf_lds_bytes(const egnn_ctx* ctx) {
  const size_t G = ctx->desc.channels / 4;
  return (size_t)ef_tiles(ctx, 1) * 4096 + 4 * (RF_WAVES * rf_stage_words(ctx) + 3 * G * 64 + G * 32 + RF_POS + RF_MAX_Q + RF_MAX_BLOCKS);
}

// The fewest orbitals an atom from which this kernel is the faster one: the old kernel's collapse grows with them, this one's does not.
// Measured as whole calls against the two kernels, 48 .. 2,600 atoms (1,000 .. 546,000 edges), 4 .. 13 orbitals, for the call that
// keeps the weights (S3 runs as well, on the same preparation) and the one that does not; both give the same bits, so that one
// rule holds for both, and the lines lie where the call that keeps them turns slower.  A round is the 32,768 edges that the
// chip's wavefronts take at a time.  Times of the old kernels over the new ones, keeping / not keeping:
//   64 channels, from 150,000 edges: 12 and 13 orbitals 1.00 .. 1.67 / 1.4 .. 1.9, 9 and 10 0.92 .. 1.05 / 1.16 .. 1.67 (lmax 1 1.13 ..
//     1.25 / 1.3 .. 1.5), 8 0.80 .. 1.03.  Below, where a wavefront goes through 16 groups one after the other, 13 orbitals 0.75 .. 1.2.
//   32 channels: one round 8 orbitals 1.00 .. 1.19 / 1.15 .. 1.7, 4 0.93 .. 1.5.  Up to half of a second one, which takes as long as a
//     whole one, 13 1.00 .. 1.30 / 1.23 .. 1.46, 12 0.96 .. 1.06 (lmax 1 1.2), 8 .. 10 0.91 .. 1.02.  More: lmax 2 10 orbitals 0.99 ..
//     1.05, 9 0.93 .. 0.98, 8 0.86 .. 0.93; lmax 3 9 1.00 .. 1.04, 8 0.95 .. 1.01; lmax 4 8 0.98 .. 1.07; lmax 1 9 1.0 .. 1.1, 8
//     0.95 .. 0.98.
//   16 channels: one round 4 orbitals 1.17 .. 1.3; more: lmax 2 9 1.1, 8 0.95 .. 0.98, 5 0.90 .. 1.1; lmax 1 8 1.0, 5 0.92 .. 0.96;
//     lmax 3 and 4 4 orbitals 1.00 .. 1.1.
//   8 channels: 4 orbitals 1.0 .. 2.
static int rf_least_orbitals(int lmax, int E, int64_t n_edges) {
  const int64_t round = 16 * RF_WAVES * EGNN_CUS;
  const int never = 1000;
  if (E == 64) return n_edges < 150000 ? never : lmax == 1 ? 9 : 12;
  if (E == 32) return n_edges <= round ? 8 : n_edges <= round + round / 2 ? 13 : lmax == 4 ? 8 : lmax == 2 ? 10 : 9;
  if (E == 16) return n_edges > round && lmax <= 2 ? (lmax == 2 ? 9 : 8) : 1;
  return E == 8 ? 1 : never;
}

bool egnn_readout_fused_fits(const egnn_ctx* ctx, const egnn_graph* g) {
  if (ctx->desc.lmax < 1 || g->n_edges <= 0 || ctx->n_orb < rf_least_orbitals(ctx->desc.lmax, ctx->desc.channels, g->n_edges) ||
      rf_lds_bytes(ctx) > 160 * 1024)
    return false;
  for (int L = 0; L <= EGNN_L_READOUT; ++L)
    if (ctx->n_out[L] > rf_room[L]) return false;
  return egnn_ef_carve(ctx, g, 1, nullptr).bytes <= (size_t)g->n_edges * ctx->n_paths[1] * ctx->desc.channels * sizeof(float);
}

int egnn_launch_readout_fused(egnn_ctx* ctx, const egnn_graph* g, void* scratch, const float* V, float* H, bool half,
                              hipStream_t stream) {
  const EfScratch s = egnn_ef_carve(ctx, g, 1, scratch);
  const int nq = ctx->n_orb * ctx->n_orb;
  RfTabs tb = {};
  tb.nq = nq;
  for (int L = 0, at = 0; L <= EGNN_L_READOUT; ++L) { tb.n[L] = ctx->n_out[L]; tb.off[L] = at; at += ctx->n_out[L]; }
  for (int i = 0; i < RF_POS; ++i) tb.pos[i] = (int16_t)nq;
  for (int i = 0; i < ctx->n_slots; ++i) {
    const int L = ctx->slot_L[i], m = ctx->slot_vrow[i] - tb.off[L];
    for (int M = 0; M < 2 * L + 1; ++M) {
      const int p = L <= 2 && m < 16 ? (L * L + M) * 16 + m : 144 + (L == 1 ? M : L == 3 ? 3 + 5 * M + m : 38 + M);
      tb.pos[p] = (int16_t)(ctx->slot_qoff[i] + M);
    }
  }
  const int ns = ctx->desc.n_orb_shells;
  const int* ol = ctx->desc.orb_l;
  int n_blk = 0;
  for (int kind = 0; kind < 9; ++kind)
    for (int a = 0, at = 0, row = 0; a < ns; row += 2 * ol[a] + 1, ++a)
      for (int b = 0, col = 0; b < ns; col += 2 * ol[b] + 1, ++b) {
        const int nb = 2 * ol[b] + 1;
        if (3 * ol[a] + ol[b] == kind) {
          tb.blk[n_blk++] = (int16_t)at;
          tb.n_blk[kind]++;
          for (int i = 0; i < (2 * ol[a] + 1) * nb; ++i)
            tb.perm[(row + i / nb) * ctx->n_orb + col + i % nb] = (int16_t)(at + i);
        }
        at += (2 * ol[a] + 1) * nb;
      }
  const size_t shmem = rf_lds_bytes(ctx);
  const long batches = (g->n_edges + 16 * RF_WAVES - 1) / (16 * RF_WAVES), per_xcd = (batches + 7) / 8;
  const int wg_per_xcd = (int)(per_xcd < EGNN_CUS / 8 ? per_xcd : EGNN_CUS / 8);
#define KERNEL(L, HF)                                                                                                       \
  do {                                                                                                                     \
    auto kern = rf_kernel<L, HF>;                                                                                          \
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,    \
                                       (int)shmem);                                                                        \
    if (e != hipSuccess) return egnn_check_hip(ctx, e, "hipFuncSetAttribute(rf_kernel)");                                  \
    hipLaunchKernelGGL(kern, dim3(8 * wg_per_xcd), dim3(64 * RF_WAVES), shmem, stream, g->src, g->dst, g->w_row, s.frame,  \
                       s.rec, s.A, reinterpret_cast<const float4*>(s.h4), reinterpret_cast<const float4*>(s.t4), s.scales, \
                       V, tb, H, (long)g->n_edges, ctx->log2_channels, (int)rf_stage_words(ctx), per_xcd);           \
  } while (0)
#define LAUNCH(L)                     \
  case L:                             \
    if (half) KERNEL(L, true);        \
    else KERNEL(L, false);            \
    break;
  switch (ctx->desc.lmax) {
    LAUNCH(1) LAUNCH(2) LAUNCH(3) LAUNCH(4)
    default: return egnn_fail(ctx, EGNN_EINVAL, "readout_fused: lmax out of range");
  }
#undef LAUNCH
#undef KERNEL
  EGNN_LAUNCH_CHECK(ctx, "rf_kernel");
  return EGNN_OK;
}
