// The SO(2) message sums with the channel mixing moved from the edges to the nodes.
//
// A message is D^T (sum_m W_m acting on the +-m components) D x with weights that all edges share, and the matrix
// D_lo^T P^m D_li of a pair of degrees is a function of the edge direction alone: sum_L beta_L^m C^(lo li L) . Yhat_L.
// So the sum over the incoming edges of a node needs, per edge, only the products of the harmonics Yhat_LM, L <= 2 lmax,
// with the features of the source,
//     S[LM][(li, mi)][c] = sum_k f_k Yhat_LM(r_k) x_src(k)[(li, mi)][c]            (so2n_gather_kernel, matrix cores)
// and coupling and channel mixing follow once per node:
//     T[lo][mo][(li, L)][c] = sum_{M, mi} C^(lo li L)[mo][mi][M] S[LM][(li, mi)][c]  (same kernel, constants in code)
//     a[(lo, mo)][c_out]    = sum_{li, L, c} (sum_m beta_L^m W_m)[c_out][c] T        (so2n_mix_kernel, matrix cores)
// The destination's own embedding is the same for all of the edges: its S is the outer product of x_j with
// g_j[LM] = sum_k f_k Yhat_LM(r_k) (so2n_sums_kernel).  The L = 0 plane of the initial edge embedding, W_e B(d), enters through
// G_j[LM][b] = sum_k f_k Yhat_LM(r_k) B_b(d_k), L <= lmax (same kernel), as columns W_e G of T beside the features' (it has
// their size there, and the weights of both are plain W); persistent edge embeddings (node block) are gathered like the
// sources', each edge its own row.
#include "so2_node.h"
#include "stream_gemm.h"
#include "so2_node_gen.inc"

#define SO2N_BATCH 256     // edges whose harmonics are staged in LDS at a time
#define SO2N_THREADS 512
#define SO2N_INLINE __attribute__((always_inline))

__host__ __device__ constexpr int so2n_nlm(int lmax) { return (2 * lmax + 1) * (2 * lmax + 1); }
__host__ __device__ constexpr int so2n_mt(int lmax) { return (so2n_nlm(lmax) + 31) / 32; }
// bytes of one 16-edge step of the staged harmonics: per tile of 32 (L, M) two pieces of two half-waves of 32 x 16 bytes,
// each padded by 16 bytes (and the step of two tiles by 64) so that the writes of 64 edges fall into 64 different banks
__host__ __device__ constexpr int so2n_step_bytes(int lmax) {
  return so2n_mt(lmax) * 2112 + (so2n_mt(lmax) == 2 ? 64 : 0);
}
// rows [(mi, LM)] of S of one degree li, and first row of li within its round
__host__ __device__ constexpr int so2n_srows(int lmax, int li) { return (2 * li + 1) * (lmax + li + 1) * (lmax + li + 1); }
__host__ __device__ constexpr int so2n_srow0(int lmax, int li) {
  int n = 0;
  for (int q = (li == 4 ? 4 : 0); q < li; ++q) n += so2n_srows(lmax, q);
  return n;
}
__host__ __device__ constexpr int so2n_cs(int E) { return E < 32 ? E : 32; }
// LDS: staged harmonics or, later, S
__host__ __device__ constexpr size_t so2n_lds_main(int lmax, int cs) {
  int rows = 0;
  for (int li = 0; li <= (lmax < 3 ? lmax : 3); ++li) rows += so2n_srows(lmax, li);
  if (lmax == 4 && so2n_srows(4, 4) > rows) rows = so2n_srows(4, 4);
  const size_t s = (size_t)rows * cs * 4, y = (size_t)(SO2N_BATCH / 16) * so2n_step_bytes(lmax);
  return s > y ? s : y;
}
__host__ __device__ constexpr size_t so2n_lds_bytes(int lmax, int E) {
  return so2n_lds_main(lmax, so2n_cs(E)) + SO2N_BATCH * 4 + 96 * 4 + 64 + (size_t)(lmax + 1) * (lmax + 1) * so2n_cs(E) * 4;
}

typedef _Float16 so2n_h2 __attribute__((ext_vector_type(2)));
typedef float so2n_f4u __attribute__((ext_vector_type(4), aligned(4)));   // (a caller's array: any alignment of its type)
typedef __amdgpu_buffer_rsrc_t so2n_rsrc;

__device__ __forceinline__ uint32_t so2n_split(float x) {   // high piece in the low half, rest in the high half
  const _Float16 h = (_Float16)x;
  const _Float16 l = (_Float16)(x - (float)h);
  return (uint32_t)__builtin_bit_cast(unsigned short, h) | ((uint32_t)__builtin_bit_cast(unsigned short, l) << 16);
}

// exponent of the power of two that brings a largest magnitude into [2^13, 2^14); 0 for zero, infinite or NaN
__device__ __forceinline__ int so2n_exp(float m) {
  if (!(m > 0.0f && m < 3.0e38f)) return 0;
  const int e = 13 - ilogbf(m);
  return e < -120 ? -120 : (e > 120 ? 120 : e);
}

// eight words (piece pairs) -> the two operand registers
__device__ __forceinline__ void so2n_pieces(const uint32_t (&w)[8], uint4& hi, uint4& lo) {
  hi.x = __builtin_amdgcn_perm(w[1], w[0], 0x05040100); lo.x = __builtin_amdgcn_perm(w[1], w[0], 0x07060302);
  hi.y = __builtin_amdgcn_perm(w[3], w[2], 0x05040100); lo.y = __builtin_amdgcn_perm(w[3], w[2], 0x07060302);
  hi.z = __builtin_amdgcn_perm(w[5], w[4], 0x05040100); lo.z = __builtin_amdgcn_perm(w[5], w[4], 0x07060302);
  hi.w = __builtin_amdgcn_perm(w[7], w[6], 0x05040100); lo.w = __builtin_amdgcn_perm(w[7], w[6], 0x07060302);
}

// Harmonics of order |m| in [M0, M1] up to degree NL - 1, times a factor: emit(index, value)
template <int NL, int M0, int M1, class F>
__device__ __forceinline__ void so2n_harmonics(float x, float y, float z, float factor, F&& emit) {
  float re = factor, im = 0.0f;
#pragma unroll
  for (int m = 0; m <= M1; ++m) {
    if (m > 0) {
      const float t = re * x - im * y;
      im = re * y + im * x;
      re = t;
    }
    if (m >= M0 && m < NL) {
      float p2 = 0.0f, p1 = SO2N_START[m];
#pragma unroll
      for (int l = m; l < NL; ++l) {
        if (l > m) {
          const float p = SO2N_A[l][m] * z * p1 - SO2N_B[l][m] * p2;
          p2 = p1;
          p1 = p;
        }
        emit(l * l + l + m, p1 * re);
        if (m > 0) emit(l * l + l - m, p1 * im);
      }
    }
  }
}

// Which of the 8 waves couples block (li, L): blocks dealt out largest first to the least loaded wave, per round
template <int LMAX>
struct So2nOwners {
  int w[5][9];
  constexpr So2nOwners() : w{} {
    for (int round = 0; round < 2; ++round) {
      const int first = LMAX == 4 && round == 0 ? 3 : 0;   // (waves 0-2 still hold degree 4 then)
      int load[8] = {};
      bool done[5][9] = {};
      for (;;) {
        int bl = -1, bL = -1, bc = -1;
        for (int li = round ? 4 : 0; li <= (round ? LMAX : (LMAX < 3 ? LMAX : 3)); ++li)
          for (int L = 0; L <= LMAX + li; ++L) {
            int outs = 0;
            for (int lo = 0; lo <= LMAX; ++lo)
              if (L >= (lo > li ? lo - li : li - lo) && L <= lo + li) outs += 2 * lo + 1;
            const int cost = (2 * L + 1) * (2 * li + 1) * 2 + outs * (2 * (2 * L + 1 < 2 * li + 1 ? 2 * L + 1 : 2 * li + 1));
            if (!done[li][L] && cost > bc) { bc = cost; bl = li; bL = L; }
          }
        if (bl < 0) break;
        int best = first;
        for (int q = first + 1; q < 8; ++q)
          if (load[q] < load[best]) best = q;
        w[bl][bL] = best;
        load[best] += bc;
        done[bl][bL] = true;
      }
    }
  }
};

// a workgroup barrier that may sit in different branches of different waves, with the LDS writes before it visible after it
__device__ __forceinline__ void so2n_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS written and read by one wave alone
__device__ __forceinline__ void so2n_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

struct So2nArgs {
  const int* ptr;            // segments: edges (or positions in perm) of node j
  const int* perm;           // NULL: the edges of node j are ptr[j] .. ptr[j + 1] themselves
  const int* index;          // feature row of edge k
  const float4* rhat_d;
  const float* alpha;        // optional further weight per edge
  const uint32_t* packed;    // feature rows in pieces, every row scaled by
  const int* row_exp;        // this power of two, which its edges' weights take back
  unsigned packed_bytes;
  const float* rows;         // OWN: the edges' own rows (fp32)
  const float* x_self;       // rows of the nodes themselves (fp32); NULL: that group is zero
  const int* self_ptr;       // incoming edges of the nodes that have a self group
  const float* g;            // [n_self] sums of the harmonics over them
  float* T;
  unsigned* t_max;           // per node: largest |T| as bits, raised here
  const unsigned* rows_max;  // OWN: largest |rows|
  int j_begin, j_end;        // nodes of this launch; T and t_max start at j_begin
  int n_self;                // nodes that have a self group
  int per_xcd, E, n_slices, form;
  float r_cut;
};

// One workgroup (8 waves) per node and slice of 32 channels.  The contraction over the node's edges runs in steps of 16
// (v_mfma_f32_32x32x16_f16, two half-precision pieces per operand, three products): operand A = harmonics of 32 (L, M) from
// LDS, operand B = 32 columns (l, m, c) of the gathered rows, which a lane reads as one word per edge, both pieces, and
// only has to permute.  Degree li couples to L <= lmax + li: at lmax 4 the 9 column tiles of li = 4 need 3 row tiles and go
// to waves 0-2, the other 16 need 2 and go to waves 3-6, wave 7 only stages harmonics; 177 matrix instructions per 16 edges,
// 51 on the busiest SIMD.
// S of the node then goes through LDS to be coupled by straight runs of multiply-adds with constants in the code, every
// wave its own blocks (li, L), lanes = (group, channel).
// lmax 4, 32 channels, 3,000 nodes, 628,000 edges: 430 us (the per-edge form: gather, five products and scatter, 3.2 ms).  With
// one part left out (of 445, when wave 7 summed the harmonics): contraction 124 us, coupling 127, harmonics 61; the rest is what
// one workgroup of 8 waves x 250 registers per compute unit cannot overlap (loads of the node's edges, barriers, starting the next workgroup).  Matrix cores at the
// contraction alone: 92 us.  Coupling on the matrix cores as well, with tables in memory: 630 us (chains of dependent loads);
// persistent workgroups that request the next node's edges early: 532 us (67 registers spilled).
// OWN: the rows are the edges' own, fp32 and read once from memory (2 GB: 560 us), cut into pieces on the way to the matrix
// cores, for the third group alone.
template <int LMAX, int CS, bool OWN>
__global__ __launch_bounds__(SO2N_THREADS, 2) void so2n_gather_kernel(So2nArgs p) {
  constexpr int D = (LMAX + 1) * (LMAX + 1), NL = 2 * LMAX + 1, NLM = NL * NL, MT = so2n_mt(LMAX);
  constexpr int STEP = so2n_step_bytes(LMAX);
  constexpr int NT = (D * CS + 31) / 32;                   // column tiles
  constexpr int TA0 = LMAX == 4 ? 16 * CS / 32 : NT;       // first tile of degree 4
  constexpr int NA = LMAX == 4 ? (NT - TA0 + 2) / 3 : 0;   // tiles per wave 0-2
  constexpr int WB0 = LMAX == 4 ? 3 : 0;                   // first wave of the lower degrees
  constexpr int NB = LMAX == 4 ? (TA0 + 3) / 4 : (NT + 6) / 7;   // tiles per wave WB0 .. 6
  constexpr int MTB = LMAX == 4 ? 2 : MT;
  constexpr So2nOwners<LMAX> owners{};
  extern __shared__ uint4 so2n_smem[];
  char* s_y = reinterpret_cast<char*>(so2n_smem);
  float* s_s = reinterpret_cast<float*>(so2n_smem);
  unsigned* s_off = reinterpret_cast<unsigned*>(s_y + so2n_lds_main(LMAX, CS));
  float* s_g = reinterpret_cast<float*>(s_off + SO2N_BATCH);
  float* s_red = s_g + 96;
  float* s_x = s_red + 16;                         // the node's own row

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = lane >> 5, l32 = lane & 31;
  const int slot = (int)(blockIdx.x >> 3);
  const int slice = slot % p.n_slices;
  const int node = (int)(blockIdx.x & 7) * p.per_xcd + slot / p.n_slices;     // relative to j_begin
  if (slot / p.n_slices >= p.per_xcd || p.j_begin + node >= p.j_end) return;
  const int j = p.j_begin + node;
  const int E = p.E;
  const int k0 = p.ptr[j], deg = p.ptr[j + 1] - k0;

  // The node's own row, the first batch of edges (their rows' offsets and lengths to LDS; direction and weight stay in
  // registers until the scaling is known) and the largest edge weight, whose power of two scales the harmonics.
  // (without incoming edges there is no message that the node's own row could enter, whatever it holds)
  const bool has_self = p.x_self != nullptr && j < p.n_self && p.self_ptr[j + 1] > p.self_ptr[j];
  for (int i = tid; i < D * CS; i += SO2N_THREADS)
    s_x[i] = has_self ? p.x_self[((size_t)j * D + i / CS) * E + slice * CS + i % CS] : 0.0f;
  for (int i = tid; i < NLM; i += SO2N_THREADS) s_g[i] = has_self ? p.g[(size_t)j * NLM + i] : 0.0f;
  const int e_own = tid & (SO2N_BATCH - 1);
  float4 g_own = make_float4(0.0f, 0.0f, 1.0f, 1.0f);
  float f_own = 0.0f;
  auto weight = [&](int k, int row, float d) SO2N_INLINE {
    const float f = egnn_envelope(d, p.r_cut) * (p.alpha ? p.alpha[k] : 1.0f);
    return OWN ? f : ldexpf(f, -p.row_exp[row]);
  };
  auto load_edge = [&](int b0) SO2N_INLINE {
    const int nb = deg - b0 < SO2N_BATCH ? deg - b0 : SO2N_BATCH;
    if (e_own < ((nb + 15) & ~15)) {
      // (the last step of 16 is filled up with copies of the last edge, of weight zero)
      const int at = k0 + b0 + (e_own < nb ? e_own : nb - 1);
      const int k = p.perm ? p.perm[at] : at;
      const int row = OWN ? at - k0 - b0 : p.index[k];
      g_own = p.rhat_d[k];
      f_own = e_own < nb ? weight(k, row, g_own.w) : 0.0f;
      if (tid < SO2N_BATCH) s_off[e_own] = (unsigned)row * (unsigned)(D * E * 4);
    }
  };
  load_edge(0);
  float wmax = f_own;
  for (int e = SO2N_BATCH + e_own; e < deg; e += SO2N_BATCH) {
    const int k = p.perm ? p.perm[k0 + e] : k0 + e;
    wmax = fmaxf(wmax, weight(k, OWN ? 0 : p.index[k], p.rhat_d[k].w));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) wmax = fmaxf(wmax, __shfl_xor(wmax, off));
  if (lane == 0) s_red[wave] = wmax;
  if (tid == 0) s_red[8] = 0.0f;                   // largest |T|, as bits
  so2n_barrier();
#pragma unroll
  for (int q = 0; q < 8; ++q) wmax = fmaxf(wmax, s_red[q]);
  // |Yhat_LM| <= sqrt(17): three bits below the range the scaling of a maximum aims at
  const int ey = so2n_exp(wmax) - 3;
  const int ex = OWN ? sgh_scale_exp(*p.rows_max) : 0;
  const float y_scale = ldexpf(1.0f, ey), unscale = ldexpf(1.0f, -ex) * ldexpf(1.0f, -ey);
  // (rows of the edges themselves lie together: those of a batch are addressed from its first)
  auto rows_of = [&](int b0) SO2N_INLINE {
    if (!OWN) return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p.packed), 0, (int)p.packed_bytes, 0x00020000);
    const int nb = deg - b0 < SO2N_BATCH ? deg - b0 : SO2N_BATCH;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.rows + (size_t)(k0 + b0) * (D * E)), 0, nb * (D * E * 4), 0x00020000);
  };
  const float x_scale = ldexpf(1.0f, ex);
  const unsigned lane_col = (unsigned)(slice * 32 + l32) * 4u;
  const unsigned tile_bytes = (unsigned)(CS == 32 ? E : 32) * 4u;
  float amax = 0.0f;

  // harmonics of the batch of edges at hand -> LDS; two threads per edge, one for the orders |m| <= LMAX / 2
  auto stage = [&](auto part_c, int n_steps) SO2N_INLINE {
    constexpr int PART = decltype(part_c)::value;
    if (e_own >= n_steps * 16) return;
    // pairs of edges share a word: the even one writes the high pieces of both, the odd one the low pieces
    char* base = s_y + (e_own >> 4) * STEP + (e_own & 1) * 1056 + ((e_own >> 3) & 1) * 528 + ((e_own & 7) >> 1) * 4;
    const uint32_t sel = (e_own & 1) ? 0x03020706u : 0x05040100u;
    auto put = [&](int lm, float v) SO2N_INLINE {
      const uint32_t u = so2n_split(v);
      const uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)u, 0xB1, 0xF, 0xF, true);   // lane ^ 1
      *reinterpret_cast<uint32_t*>(base + (lm >> 5) * 2112 + (lm & 31) * 16) = __builtin_amdgcn_perm(o, u, sel);
    };
    const float f = f_own * y_scale;
    if (PART == 0 || (PART == 2 && wave < 4)) so2n_harmonics<NL, 0, LMAX / 2>(g_own.x, g_own.y, g_own.z, f, put);
    else so2n_harmonics<NL, LMAX / 2 + 1, 2 * LMAX>(g_own.x, g_own.y, g_own.z, f, put);
  };
  const char* frag = s_y + hh * 528 + l32 * 16;
#define SO2N_A(t, piece) (*reinterpret_cast<const uint4*>(frag + s * STEP + (t) * 2112 + (piece) * 1056))

  // coupling of the blocks this wave owns: lane = (group, channel), group 0 reads S, group 1 forms g x on the spot
  const int c = lane % CS, grp = lane / CS;
  // (masks: as factors of 0 and 1 they would let one group's infinities reach the other, and take 12 us more; compares 78)
  const uint32_t from_s = grp == 0 ? ~0u : 0u, from_x = grp == 1 ? ~0u : 0u;
  auto only = [](float v, uint32_t mask) SO2N_INLINE { return __uint_as_float(__float_as_uint(v) & mask); };
  const int form = p.form;
  const int node_floats = so2n_node_off(LMAX, E, LMAX + 1, form);
  float* T = p.T + (size_t)node * node_floats;
  const so2n_rsrc tr = __builtin_amdgcn_make_buffer_rsrc(T, 0, node_floats * 4, 0x00020000);
  auto couple = [&](auto li_c, auto L_c) SO2N_INLINE {
    constexpr int li = decltype(li_c)::value, L = decltype(L_c)::value;
    constexpr int nl = (LMAX + li + 1) * (LMAX + li + 1);
    if (wave != owners.w[li][L]) return;
    float xv[2 * li + 1];
#pragma unroll
    for (int q = 0; q < 2 * li + 1; ++q) xv[q] = only(s_x[(li * li + q) * CS + c], from_x);
    float o[D];
#pragma unroll
    for (int i = 0; i < D; ++i) o[i] = 0.0f;
    const float* rows = s_s + (size_t)so2n_srow0(LMAX, li) * CS + c;
    So2Couple<LMAX, li, L>::run(
        [&](int M, float* v) SO2N_INLINE {
          const int lm = L * L + M;
          const float gl = s_g[lm];
#pragma unroll
          for (int mi = 0; mi < 2 * li + 1; ++mi) {
            const float sv = rows[(mi * nl + lm) * CS];
            v[mi] = gl * xv[mi] + only(sv, from_s);
          }
        },
        o);
#pragma unroll
    for (int lo = 0; lo <= LMAX; ++lo) {
      if (L >= (lo > li ? lo - li : li - lo) && L <= lo + li) {
        const int path = so2n_path_base(lo, li) + L - (lo > li ? lo - li : li - lo);
        const int np = so2n_paths(LMAX, lo), ld = so2n_ld(LMAX, E, lo, form);
        const int at0 = so2n_node_off(LMAX, E, lo, form) + path * E + slice * 32;
        // (lanes past the two groups: an offset the range check drops)
        const int lane_at = grp < (OWN ? 1 : 2) ? ((OWN ? 2 : grp) * np * E + c) * 4 : node_floats * 4;
#pragma unroll
        for (int mo = 0; mo < 2 * lo + 1; ++mo) {
          const float v = o[lo * lo + mo];
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), tr, lane_at, (at0 + mo * ld) * 4, 0);
          amax = fmaxf(amax, fabsf(v));
        }
      }
    }
  };
#define SO2N_C(li, L) couple(std::integral_constant<int, li>{}, std::integral_constant<int, L>{});
#define SO2N_IF(li, L) if constexpr (li <= LMAX && L <= LMAX + li) SO2N_C(li, L)
#define SO2N_ROW(li) SO2N_IF(li, 0) SO2N_IF(li, 1) SO2N_IF(li, 2) SO2N_IF(li, 3) SO2N_IF(li, 4) SO2N_IF(li, 5) SO2N_IF(li, 6) SO2N_IF(li, 7)

  // Each kind of wave has a branch of its own from the first step until its S is in LDS, so that no accumulator lives in
  // another kind's code; every branch passes the same barriers.
  // N column tiles of M row tiles from tile0 on (a wave whose last tiles do not exist repeats the last one that does)
  auto contract = [&](auto nt_c, auto mt_c, auto part_c, int tile0, int t_end, auto&& finish) SO2N_INLINE {
    constexpr int N = decltype(nt_c)::value, M = decltype(mt_c)::value;
    float16v acc[N * M];
#pragma unroll
    for (int t = 0; t < N * M; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
    unsigned tb[N];
#pragma unroll
    for (int i = 0; i < N; ++i) tb[i] = (unsigned)(tile0 + i < t_end ? tile0 + i : t_end - 1) * tile_bytes;
    for (int b0 = 0; b0 < deg; b0 += SO2N_BATCH) {
      const int nb = deg - b0 < SO2N_BATCH ? deg - b0 : SO2N_BATCH;
      const int n_steps = (nb + 15) >> 4;
      if (b0) {
        so2n_barrier();                             // the previous batch is consumed
        load_edge(b0);
        so2n_barrier();
      }
      const so2n_rsrc xr = rows_of(b0);
      uint32_t w[N][8];
      unsigned o[8];
      auto offsets = [&](int s) SO2N_INLINE {
        const uint4 o0 = *reinterpret_cast<const uint4*>(s_off + s * 16 + 8 * hh);
        const uint4 o1 = *reinterpret_cast<const uint4*>(s_off + s * 16 + 8 * hh + 4);
        o[0] = o0.x + lane_col; o[1] = o0.y + lane_col; o[2] = o0.z + lane_col; o[3] = o0.w + lane_col;
        o[4] = o1.x + lane_col; o[5] = o1.y + lane_col; o[6] = o1.z + lane_col; o[7] = o1.w + lane_col;
      };
      // (buffer loads: a plain load of the next step's words would be moved over the loop's back edge to their use)
      auto fetch = [&](int i) SO2N_INLINE {
#pragma unroll
        for (int q = 0; q < 8; ++q) w[i][q] = __builtin_amdgcn_raw_buffer_load_b32(xr, (int)o[q], (int)tb[i], 0);
      };
      offsets(0);
#pragma unroll
      for (int i = 0; i < N; ++i) fetch(i);
      stage(part_c, n_steps);
      so2n_barrier();
      for (int s = 0; s < n_steps; ++s) {
        uint4 ah[M], al[M];
#pragma unroll
        for (int t = 0; t < M; ++t) { ah[t] = SO2N_A(t, 0); al[t] = SO2N_A(t, 1); }
        offsets(s + 1 < n_steps ? s + 1 : s);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          uint4 bh, bl;
          if (OWN) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = __uint_as_float(w[i][q]);
            sgh_split8(v, x_scale, bh, bl);
          } else {
            so2n_pieces(w[i], bh, bl);
          }
          fetch(i);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int t = 0; t < M; ++t)
            acc[i * M + t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(al[t]), sgh_as_h8(bh), acc[i * M + t], 0, 0, 0);
#pragma unroll
          for (int t = 0; t < M; ++t)
            acc[i * M + t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(ah[t]), sgh_as_h8(bl), acc[i * M + t], 0, 0, 0);
#pragma unroll
          for (int t = 0; t < M; ++t)
            acc[i * M + t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(ah[t]), sgh_as_h8(bh), acc[i * M + t], 0, 0, 0);
        }
      }
    }
    so2n_barrier();                                 // the staged harmonics are consumed: S takes their place
    finish(acc);
  };
  // S of one wave's tiles -> LDS rows [(mi, LM)][c] of degree li
  auto spill = [&](auto nt_c, auto mt_c, int tile0, int t_end, const float16v* acc) SO2N_INLINE {
    constexpr int N = decltype(nt_c)::value, M = decltype(mt_c)::value;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int n = (tile0 + i) * 32 + l32;
      const int lm_in = CS == 32 ? tile0 + i : n / CS, cc = CS == 32 ? l32 : n % CS;   // (one (l, m) per tile: scalar)
      if (tile0 + i < t_end && lm_in < D) {
        const int li = lm_in < 1 ? 0 : lm_in < 4 ? 1 : lm_in < 9 ? 2 : lm_in < 16 ? 3 : 4;
        const int nl = (LMAX + li + 1) * (LMAX + li + 1);
        const int row0 = li == 0 ? 0 : li == 1 ? so2n_srow0(LMAX, 1) : li == 2 ? so2n_srow0(LMAX, 2) : li == 3 ? so2n_srow0(LMAX, 3) : 0;
        float* out = s_s + (size_t)(row0 + (lm_in - li * li) * nl + 4 * hh) * CS + cc;
#pragma unroll
        for (int t = 0; t < M; ++t)
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            const int lm = t * 32 + 8 * (q >> 2) + (q & 3);   // of the first half-wave; the second holds lm + 4
            if (lm + 4 < nl) out[lm * CS] = unscale * acc[i * M + t][q];
            else if (lm < nl && hh == 0) out[lm * CS] = unscale * acc[i * M + t][q];
          }
      }
    }
  };
  // the wave without tiles
  auto stage_only = [&]() SO2N_INLINE {
    for (int b0 = 0; b0 < deg; b0 += SO2N_BATCH) {
      const int nb = deg - b0 < SO2N_BATCH ? deg - b0 : SO2N_BATCH;
      if (b0) {
        so2n_barrier();
        load_edge(b0);
        so2n_barrier();
      }
      stage(std::integral_constant<int, 1>{}, (nb + 15) >> 4);
      so2n_barrier();
    }
  };
  // Two rounds at lmax 4, because S of all degrees exceeds the LDS: waves 0-2 hold degree 4 in registers during the first,
  // so the others couple the lower degrees alone.
  if (LMAX == 4 && wave < 3) {
    if constexpr (LMAX == 4) {
      const int t0 = TA0 + wave * NA;
      contract(std::integral_constant<int, NA>{}, std::integral_constant<int, 3>{}, std::integral_constant<int, 0>{}, t0, NT,
               [&](const float16v* acc) SO2N_INLINE {
                 so2n_barrier();
                 so2n_barrier();
                 spill(std::integral_constant<int, NA>{}, std::integral_constant<int, 3>{}, t0, NT, acc);
               });
    }
  } else {
    if (wave == 7) {
      stage_only();
      so2n_barrier();                               // the staged harmonics are consumed
    } else {
      const int t0 = (wave - WB0) * NB;
      contract(std::integral_constant<int, NB>{}, std::integral_constant<int, MTB>{}, std::integral_constant<int, 2>{}, t0, TA0,
               [&](const float16v* acc) SO2N_INLINE {
                 spill(std::integral_constant<int, NB>{}, std::integral_constant<int, MTB>{}, t0, TA0, acc);
               });
    }
    so2n_barrier();
    SO2N_ROW(0) SO2N_ROW(1) SO2N_ROW(2) SO2N_ROW(3)
    if constexpr (LMAX == 4) so2n_barrier();
  }
  if constexpr (LMAX == 4) {
    so2n_barrier();
    SO2N_ROW(4) SO2N_IF(4, 8)
  }
#undef SO2N_ROW
#undef SO2N_IF
#undef SO2N_C
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  if (lane == 0) atomicMax(reinterpret_cast<unsigned*>(s_red + 8), __float_as_uint(amax));
  so2n_barrier();
  if (tid == 0) atomicMax(p.t_max + node, __float_as_uint(s_red[8]));   // (no result is waited for)
}

// ---------------------------------------------------------------------------------------------- sums of the harmonics
#define SO2N_SUM_WAVES 4
struct So2nSums {
  const int* ptr;
  const float4* rhat_d;
  const float* alpha;        // optional further weight per edge
  const float* W_e;          // transposed, [SO2N_AUX][E]: the edge embedding's columns of T (form SO2N_GAUSS); NULL: none
  float* g;                  // [n_owned][(2 lmax + 1)^2]
  float* G;                  // [n_owned][(lmax + 1)^2][SO2N_AUX] sums with the Gaussian basis; NULL: not kept
  float* T;
  unsigned* t_max;           // per node: largest |T| (raised here) or |G| (set here) as bits
  unsigned* G_max;
  int n_rbf, log2E;          // n_rbf = 0: g alone
  float r_cut;
};

// One workgroup per node, a quarter of its edges per wave, a lane an edge: the harmonics go from the lane's registers to LDS,
// half a wavefront's edges at a time (all 64 of two waves would leave room for six waves per compute unit), where they are
// summed, lane = (L, M), and contracted with the Gaussian basis on the fp32 matrix cores (v_mfma_f32_32x32x2_f32), all in 32
// bits.  3,000 nodes, 628,000 edges, lmax 4, 32 channels: 46 us, without the basis 22; latency of the node's few edges.
template <int LMAX>
__global__ __launch_bounds__(64 * SO2N_SUM_WAVES) void so2n_sums_kernel(So2nSums p) {
  constexpr int D = (LMAX + 1) * (LMAX + 1), NL = 2 * LMAX + 1, NLM = NL * NL;     // (NLM odd: lanes write different banks)
  constexpr int NY = 32 * NLM + (NLM < 32 ? 32 : 0);      // (rows 25 .. 31 of the contraction read on; nobody uses them)
  constexpr int THREADS = 64 * SO2N_SUM_WAVES;
  __shared__ float s_y[SO2N_SUM_WAVES][NY > 32 * 33 ? NY : 32 * 33];
  __shared__ float s_d[SO2N_SUM_WAVES][64];
  __shared__ float s_sum[SO2N_SUM_WAVES][NLM];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = lane >> 5, l32 = lane & 31, j = blockIdx.x;
  const int k0 = p.ptr[j], deg = p.ptr[j + 1] - k0;
  const int share = (deg + SO2N_SUM_WAVES - 1) / SO2N_SUM_WAVES, b_end = min((wave + 1) * share, deg);
  const float rbf_step = p.n_rbf > 1 ? p.r_cut / (float)(p.n_rbf - 1) : 1.0f;
  const float rbf_inv = 0.5f / (rbf_step * rbf_step);
  float* y = s_y[wave];
  constexpr int R = (NLM + 63) / 64;
  float sum[R][4];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[r][q] = 0.0f;
  float16v acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
  for (int b0 = wave * share; b0 < b_end; b0 += 64) {
    float4 e = make_float4(0.0f, 0.0f, 1.0f, 1.0f);
    float f = 0.0f;                                    // (edges past the last are zero)
    if (b0 + lane < b_end) {
      const int k = k0 + b0 + lane;
      e = p.rhat_d[k];
      f = egnn_envelope(e.w, p.r_cut) * (p.alpha ? p.alpha[k] : 1.0f);
    }
    float v[NLM];
    so2n_harmonics<NL, 0, 2 * LMAX>(e.x, e.y, e.z, f, [&](int lm, float h) SO2N_INLINE { v[lm] = h; });
    s_d[wave][lane] = e.w;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int nb = min(b_end - b0 - 32 * half, 32);
      if (nb <= 0) break;
      if (hh == half)
#pragma unroll
        for (int i = 0; i < NLM; ++i) y[l32 * NLM + i] = v[i];
      so2n_wave_sync();
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int lm = r * 64 + lane;
        if (lm < NLM)
          for (int q = 0; q < nb; q += 8)
#pragma unroll
            for (int u = 0; u < 8; ++u) sum[r][u & 3] += y[(q + u) * NLM + lm];
      }
      if (p.n_rbf > 0)
        for (int q0 = 0; q0 < nb; q0 += 8) {
#pragma unroll
          for (int t = 0; t < 8; t += 2) {
            const int q = q0 + t + hh;
            const float u = s_d[wave][32 * half + q] - (float)l32 * rbf_step;
            const float basis = l32 < p.n_rbf ? __expf(-u * u * rbf_inv) : 0.0f;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(y[q * NLM + l32], basis, acc, 0, 0, 0);
          }
        }
      so2n_wave_sync();
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r * 64 + lane < NLM) s_sum[wave][r * 64 + lane] = (sum[r][0] + sum[r][1]) + (sum[r][2] + sum[r][3]);
#pragma unroll
  for (int i = 0; i < 16; ++i) y[(8 * (i >> 2) + 4 * hh + (i & 3)) * 33 + l32] = acc[i];
  __syncthreads();
  for (int i = tid; i < NLM; i += THREADS) p.g[(size_t)j * NLM + i] = (s_sum[0][i] + s_sum[1][i]) + (s_sum[2][i] + s_sum[3][i]);
  if (p.n_rbf == 0) return;
  float mx = 0.0f;
  for (int i = tid; i < D * SO2N_AUX; i += THREADS) {
    const int at = (i >> 5) * 33 + (i & 31);
    const float v = (s_y[0][at] + s_y[1][at]) + (s_y[2][at] + s_y[3][at]);
    s_y[0][at] = v;
    mx = fmaxf(mx, fabsf(v));
    if (p.G) p.G[(size_t)j * (D * SO2N_AUX) + i] = v;
  }
  if (p.W_e) {
    __syncthreads();
    mx = 0.0f;
    const int E = 1 << p.log2E, c = tid & (E - 1);
    float w[SO2N_AUX];
#pragma unroll
    for (int b = 0; b < SO2N_AUX; ++b) w[b] = p.W_e[(b << p.log2E) + c];
    float* T = p.T + (size_t)j * so2n_node_off(LMAX, E, LMAX + 1, SO2N_GAUSS) + c - E;
    for (int i = tid >> p.log2E; i < D; i += THREADS >> p.log2E) {
      float v = 0.0f;
#pragma unroll
      for (int b = 0; b < SO2N_AUX; ++b) v += s_y[0][i * 33 + b] * w[b];
      const int lo = i < 1 ? 0 : i < 4 ? 1 : i < 9 ? 2 : i < 16 ? 3 : 4;
      T[so2n_node_off(LMAX, E, lo, SO2N_GAUSS) + (i - lo * lo + 1) * so2n_ld(LMAX, E, lo, SO2N_GAUSS)] = v;
      mx = fmaxf(mx, fabsf(v));
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if (lane == 0) s_d[0][wave] = mx;
  __syncthreads();
  if (tid == 0) {
    const unsigned bits = __float_as_uint(fmaxf(fmaxf(s_d[0][0], s_d[0][1]), fmaxf(s_d[0][2], s_d[0][3])));
    if (p.W_e) atomicMax(p.t_max + j, bits);
    else p.G_max[j] = bits;
  }
}
static_assert(SO2N_SUM_WAVES == 4 && SO2N_AUX == 32, "so2n_sums_kernel adds four waves' sums of 32 columns");

// ---------------------------------------------------------------------------------------------- attention scores
// score[k] = sum_c w_att[c] leaky(y0[k][c]) with y0 = the L = 0 plane of edge k's message: that plane needs only the m = 0
// component of every degree in the bond frame, sum_M Yhat_lM x_lM / sqrt(2 l + 1), of the three rows (edge, source,
// destination), and the first E rows of W_0.  A workgroup takes 32 consecutive edges and the three groups one after
// another: threads (edge, channel) form the components in LDS, four waves share the contraction over (l, channel)
// (v_mfma_f32_32x32x2_f32, lane = edge).  Bound: the edge rows, read here and once more by the gathering kernel, because
// the softmax stands in between; 628,000 edges, lmax 4, 32 channels: 660 us, of which matrix cores 122 and vector ALU about
// 235 (all three groups in LDS at once, two workgroups per compute unit: 937).  The largest magnitude among them is kept
// for that kernel's scaling.
template <int LMAX>
__global__ __launch_bounds__(256) void so2n_score_kernel(const int* __restrict__ src, const int* __restrict__ dst,
                                                         const float4* __restrict__ rhat_d, const float* __restrict__ x,
                                                         unsigned x_bytes, const float* __restrict__ T_edge, const float* __restrict__ W,
                                                         const float* __restrict__ w_att, float* __restrict__ score,
                                                         long n_edges, int log2E, unsigned* __restrict__ t_max) {
  constexpr int D = (LMAX + 1) * (LMAX + 1), NL = LMAX + 1;
  extern __shared__ float so2n_sf[];
  __shared__ float s_h[32][D + 1];
  __shared__ float s_part[4][32];
  __shared__ float s_mx[4];
  const int E = 1 << log2E, K = NL * E, ldq = K + 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, hh = lane >> 5;
  const long e0 = (long)blockIdx.x * 32;
  const int ne = n_edges - e0 < 32 ? (int)(n_edges - e0) : 32;
  if (tid < 32) {
    const float4 g = rhat_d[e0 + (tid < ne ? tid : ne - 1)];
    so2n_harmonics<NL, 0, LMAX>(g.x, g.y, g.z, 1.0f, [&](int lm, float v) SO2N_INLINE { s_h[tid][lm] = v; });
  }
  __syncthreads();
  const int c = tid & (E - 1), slot = tid >> log2E, n_slots = 256 >> log2E;
  float mx = 0.0f;
  // The contraction runs in steps of 8 columns, four of them per half-wave.  Up to 32 channels the waves share the columns and
  // their sums meet in LDS before the non-linearity; with 64, waves 0 and 1 (2 and 3) share those of a block of 32 channels.
  const int n_cb = E > 32 ? 2 : 1, cb = E > 32 ? wave >> 1 : 0, part = E > 32 ? wave & 1 : wave, parts = 4 / n_cb;
  const int n_steps = K / 8, per = (n_steps + parts - 1) / parts;
  const int s1 = (part + 1) * per < n_steps ? (part + 1) * per : n_steps;
  float16v acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
  const bool live = cb * 32 + l32 < E;
  const float* w_row = W + (size_t)(live ? cb * 32 + l32 : 0) * (3 * K) + 4 * hh;
  const float* q_row = so2n_sf + (size_t)l32 * ldq + 4 * hh;
  constexpr int U = 5;
  const so2n_rsrc xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, (int)x_bytes, 0x00020000);
  const so2n_rsrc tr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(T_edge + (((size_t)e0 * D) << log2E)), 0,
                                                         (ne * D) << (log2E + 2), 0x00020000);
  auto group = [&](auto grp_c) SO2N_INLINE {
    constexpr int GRP = decltype(grp_c)::value;         // as in the weights: 0 source, 1 destination, 2 edge
    for (int e = slot; e < 32; e += n_slots) {
      const long k = e0 + (e < ne ? e : ne - 1);        // (the copies of the last edge are not stored)
      // (buffer loads: the 25 offsets within a row are scalars; formed per lane they were half of the kernel's instructions)
      const unsigned row = GRP == 2 ? (unsigned)(k - e0) : (unsigned)(GRP == 0 ? src[k] : dst[k]);
      const int at = (int)(((row * D) << (log2E + 2)) + 4 * c);
      float v[D];
#pragma unroll
      for (int i = 0; i < D; ++i)
        v[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(GRP == 2 ? tr : xr, at, i << (log2E + 2), GRP == 2 ? 2 : 0));
      float* q = so2n_sf + (size_t)e * ldq + c;
#pragma unroll
      for (int l = 0; l <= LMAX; ++l) {
        constexpr float inv[5] = {1.0f, 0.57735026918962576f, 0.44721359549995794f, 0.37796447300922722f, 0.33333333333333333f};
        float a = 0.0f;
#pragma unroll
        for (int i = l * l; i < (l + 1) * (l + 1); ++i) {
          a += s_h[e][i] * v[i];
          if (GRP == 2) mx = fmaxf(mx, fabsf(v[i]));
        }
        q[l << log2E] = a * inv[l];
      }
    }
    __syncthreads();
    for (int s = part * per; s < s1; s += U) {
      sg_f4 wv[U], qv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int su = s + u < s1 ? s + u : s1 - 1, l = (su * 8) >> log2E;
        wv[u] = *reinterpret_cast<const so2n_f4u*>(w_row + su * 8 + (2 * l + GRP) * E);
        qv[u] = *reinterpret_cast<const sg_f4*>(q_row + su * 8);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s + u < s1)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(live ? wv[u][t] : 0.0f, qv[u][t], acc, 0, 0, 0);
    }
    __syncthreads();
  };
  group(std::integral_constant<int, 2>{});
  group(std::integral_constant<int, 0>{});
  group(std::integral_constant<int, 1>{});
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if (lane == 0) s_mx[wave] = mx;
  // (the components are consumed: partial sums take their place)
#pragma unroll
  for (int i = 0; i < 16; ++i) so2n_sf[(wave * 16 + i) * 64 + lane] = acc[i];
  __syncthreads();
  if (tid == 0) egnn_raise_max(t_max, fmaxf(fmaxf(s_mx[0], s_mx[1]), fmaxf(s_mx[2], s_mx[3])));
  float sc = 0.0f;
  for (int r = wave; r < 16 * n_cb; r += 4) {
    const int b = r >> 4, i = r & 15, co = b * 32 + 8 * (i >> 2) + 4 * hh + (i & 3);
    float v = 0.0f;
    for (int z = 0; z < parts; ++z) v += so2n_sf[((b * parts + z) * 16 + i) * 64 + lane];
    if (co < E) sc += w_att[co] * (v > 0.0f ? v : 0.2f * v);
  }
  sc += __shfl_xor(sc, 32);
  if (hh == 0) s_part[wave][l32] = sc;
  __syncthreads();
  if (tid < ne) score[e0 + tid] = (s_part[0][tid] + s_part[1][tid]) + (s_part[2][tid] + s_part[3][tid]);
}

// scores -> attention weights, in place; a wavefront per node
__global__ __launch_bounds__(256) void so2n_softmax_kernel(const int* __restrict__ row_ptr, float* __restrict__ alpha, int n_owned) {
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= n_owned) return;
  const int k0 = row_ptr[j], k1 = row_ptr[j + 1];
  float mx = -3.0e38f;
  for (int k = k0 + lane; k < k1; k += 64) mx = fmaxf(mx, alpha[k]);
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  float sum = 0.0f;
  for (int k = k0 + lane; k < k1; k += 64) {
    const float e = __expf(alpha[k] - mx);
    alpha[k] = e;                               // read again by this lane alone
    sum += e;
  }
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  const float inv = 1.0f / sum;
  for (int k = k0 + lane; k < k1; k += 64) alpha[k] *= inv;
}

// ---------------------------------------------------------------------------------------------- features in pieces
// One wavefront per row: its largest magnitude, the power of two from that and the row in pieces.  A power of two for all rows
// would have to leave out those that no edge reads, and lose the small ones beside the large (and take two kernels: 19 instead
// of 10 us on 2.4 million values).
//
// With X_max the scales of a weight gradient come from here too: sums over the nodes n of X_n y_n with y the rows (X = the coupled
// sums T and y = the features; X = G and y = da), X_n scaled by 2^node_exp[n] from its own largest value and y_n by the inverse
// of that and 2^C for all.  C brings the largest y_n 2^-node_exp[n] to 2^13; its exponent (plus SO2N_EXP0) goes to *used.  Nodes
// whose X is zero, those without edges (incoming ones of the first n_ptr nodes, outgoing ones with col_ptr) among them, and those
// that fill up a multiple of 16 are marked.
#define SO2N_UNUSED (-1000000)
#define SO2N_EXP0 4096
struct So2nPack {
  const float* x;
  int n_rows, row_floats;
  uint32_t* out;                 // NULL: scales only
  int* row_exp;
  const unsigned* X_max;         // largest |X| of every node; NULL: rows only
  const int* ptr;
  int n_ptr;
  const int* col_ptr;            // may be NULL
  int* node_exp;
  unsigned* used;
};
__global__ __launch_bounds__(256) void so2n_pack_kernel(So2nPack p) {
  __shared__ unsigned s_used[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned used = 0u;
  const int n_all = p.X_max ? (p.n_rows + 15) & ~15 : p.n_rows;
  for (int i = blockIdx.x * 4 + wave; i < n_all; i += gridDim.x * 4) {
    const bool there = i < p.n_rows;
    float mx = 0.0f;
    bool finite = true;
    if (there) {
      const float* row = p.x + (size_t)i * p.row_floats;
#pragma unroll 4
      for (int q = lane; q < p.row_floats; q += 64) {
        const float v = fabsf(row[q]);
        mx = fmaxf(mx, v);
        finite = finite && v < __builtin_inff();
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
      if (p.out) {
        const int e = so2n_exp(mx);
        if (lane == 0) p.row_exp[i] = e;
        const float sc = ldexpf(1.0f, e);
#pragma unroll 4
        for (int q = lane; q < p.row_floats; q += 64) p.out[(size_t)i * p.row_floats + q] = so2n_split(row[q] * sc);
      }
    }
    if (!p.X_max) continue;
    finite = __all(finite);
    const bool edges = there && ((i < p.n_ptr && p.ptr[i + 1] > p.ptr[i]) || (p.col_ptr && p.col_ptr[i + 1] > p.col_ptr[i]));
    const float X = edges ? __uint_as_float(p.X_max[i]) : 0.0f;
    const int e = so2n_exp(X);
    // (an infinite or NaN row shows in the result unless its node has no edges)
    const bool unused = !edges || (X == 0.0f && finite);
    if (lane == 0) p.node_exp[i] = unused ? SO2N_UNUSED : e;
    if (!unused && finite && mx > 0.0f && X > 0.0f) used = max(used, (unsigned)(ilogbf(mx) - e + SO2N_EXP0));
  }
  if (!p.X_max) return;
  if (lane == 0) s_used[wave] = used;
  __syncthreads();
  if (threadIdx.x == 0) atomicMax(p.used, max(max(s_used[0], s_used[1]), max(s_used[2], s_used[3])));
}

// ---------------------------------------------------------------------------------------------- path weights
struct So2nW {
  int k_first[6];        // first contraction row of every output degree
  int K[5];              // contraction length (2 paths E + aux)
  size_t off[6];         // first weight W_0 / (Wr_m, Wi_m) of every order
};

// Weight of contraction row (group, path, channel) of output degree a into channel col.  Transposed (reverse pass): a is the
// input degree of the forward pass, the paths run over its output degrees; swapping the two degrees of a coupling tensor
// changes its sign with the parity of the degrees.
__device__ float so2n_weight(const float* __restrict__ W, const So2nW& s, int lmax, int E, int a, int k, int col, int form,
                             bool transposed) {
  const int np = so2n_paths(lmax, a);
  if (k >= so2n_groups(form) * np * E)   // W_0, edge columns of degree 0
    return W[(size_t)(a * E + col) * ((lmax + 1) * 3 * E) + 2 * E + (k - so2n_groups(form) * np * E)] / sqrtf((float)(2 * a + 1));
  const int g = k / (np * E), r = k - g * np * E;
  const int path = r / E, kc = r - path * E;
  int b = 0;
  while (path >= so2n_path_base(a, b + 1)) ++b;
  const int d = a > b ? a - b : b - a;
  const int L = d + path - so2n_path_base(a, b);
  const int lo = transposed ? b : a, li = transposed ? a : b;
  const int co = transposed ? kc : col, ci = transposed ? col : kc;
  const int odd = (a + b + L) & 1;
  float sum = 0.0f;
  for (int m = odd; m <= (a < b ? a : b); ++m) {
    const int nl = lmax + 1 - m;
    const size_t at = (size_t)((lo - m) * E + co) * (nl * 3 * E) + (size_t)(li - m) * 3 * E + g * E + ci;
    sum += SO2N_BETA[lo][li][L - d][m] * W[s.off[m] + (odd ? (size_t)nl * E * nl * 3 * E : 0) + at];
  }
  return transposed && odd ? -sum : sum;
}

// out: the path weights and then, with W_e, its transpose padded to SO2N_AUX rows
__global__ __launch_bounds__(256) void so2n_weights_kernel(const float* __restrict__ W, const float* __restrict__ W_e, So2nW s,
                                                           int lmax, int E, int n_rbf, int form, bool transposed,
                                                           float* __restrict__ out, unsigned* __restrict__ w_max) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x, n = (long)s.k_first[lmax + 1] * E;
  float v = 0.0f;
  if (W_e && i >= n && i < n + SO2N_AUX * E) {
    const int b = (int)(i - n) / E, c = (int)(i - n) % E;
    out[i] = b < n_rbf ? W_e[c * n_rbf + b] : 0.0f;
  }
  if (i < n) {
    const int row = (int)(i / E), col = (int)(i - (long)row * E);
    int a = 0;
    while (row >= s.k_first[a + 1]) ++a;
    v = so2n_weight(W, s, lmax, E, a, row - s.k_first[a], col, form, transposed);
    out[i] = v;
  }
  float mx = fabsf(v);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if ((threadIdx.x & 63) == 0) egnn_raise_max(w_max, mx);
}

// operand order of so2n_mix_kernel: [step of 16][column block][piece][lane][8 halves], per output degree
struct So2nSteps { int first[6]; };   // first step of every output degree
__global__ __launch_bounds__(256) void so2n_wpack_kernel(const float* __restrict__ w, So2nW s, So2nSteps st, int lmax, int E,
                                                         int n_cb, const unsigned* __restrict__ w_max, uint4* __restrict__ out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long)st.first[lmax + 1] * n_cb * 64) return;
  const int lane = (int)(i & 63);
  const int blk = (int)(i >> 6), step = blk / n_cb, cb = blk - step * n_cb;
  int a = 0;
  while (step >= st.first[a + 1]) ++a;
  const int k = (step - st.first[a]) * 16 + 8 * (lane >> 5), col = cb * 32 + (lane & 31);
  float v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = (k + q < s.K[a] && col < E) ? w[(size_t)(s.k_first[a] + k + q) * E + col] : 0.0f;
  uint4 hi, lo;
  sgh_split8(v, ldexpf(1.0f, sgh_scale_exp(*w_max)), hi, lo);
  out[((size_t)blk * 2) * 64 + lane] = hi;
  out[((size_t)blk * 2 + 1) * 64 + lane] = lo;
}

// ---------------------------------------------------------------------------------------------- channel mixing per node
struct So2nMix {
  const float* T;
  int node_floats, off[5], ld[5];
  const uint4* w;
  So2nSteps st;
  int blocks[6];        // first row block of every output degree
  int K[5];
  int n_nodes, lmax, E;
  float scale;
  float* out;           // [n_nodes][(lmax+1)^2][E]
  const unsigned* t_max;
  const unsigned* w_max;
};

// out[(n, (lo, mo))][col] = scale sum_k T[lo][n (2 lo + 1) + mo][k] w[lo][k][col].  A workgroup takes 32 rows, its four
// waves a quarter of the contraction each (rows are 1,632 values long at lmax 4 and 32 channels, up to 6,528 in all, while there
// are only (lmax+1)^2 of them per node: without the split a few thousand waves would each walk a hundred dependent steps);
// partial sums meet in LDS in a fixed order.  Bound: T, written by the gathering kernel and read here; 413 MB at 3,000 nodes,
// lmax 4, 32 channels: 117 us.  128 channels are two workgroups of two column blocks each: one of four has no registers for
// three sums, and even with two the whole call took 1,000 instead of 866 us on 1,000 nodes.
template <int NCB>
__global__ __launch_bounds__(256, 2) void so2n_mix_kernel(So2nMix p) {
  __shared__ float s_part[3][NCB * 16 * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, hh = lane >> 5;
  int lo = 0;
  while ((int)blockIdx.x >= p.blocks[lo + 1]) ++lo;
  const long rows = (long)p.n_nodes * (2 * lo + 1), r0 = ((long)blockIdx.x - p.blocks[lo]) * 32;
  const int K = p.K[lo], n_steps = (K + 15) / 16;
  const int per = (n_steps + 3) / 4;
  const int s0 = wave * per, s1 = s0 + per < n_steps ? s0 + per : n_steps;
  const long row = r0 + l32 < rows ? r0 + l32 : rows - 1;
  const long node = row / (2 * lo + 1);
  const float* a = p.T + (size_t)node * p.node_floats + p.off[lo] + (size_t)(row - node * (2 * lo + 1)) * p.ld[lo] + 8 * hh;
  const int n_cb = gridDim.y * NCB, cb0 = blockIdx.y * NCB;
  const uint4* w = p.w + ((size_t)p.st.first[lo] * n_cb + cb0) * 128 + lane;
  // (a scale per node: beside others' large sums, small ones, of features or edges near the cutoff, keep their accuracy)
  const int ea = so2n_exp(__uint_as_float(p.t_max[node])), eb = sgh_scale_exp(*p.w_max);
  const float a_scale = ldexpf(1.0f, ea);
  // Even steps, odd steps, and the products of a high and a low piece, 2^-11 of the others: the rounding of the running sums is the
  // largest part of the error (with one sum for all 2.75e-7 of the message sum at lmax 4, 32 channels and 209 edges a node, so
  // 2.0e-7; no slower).
  float16v sums[3][NCB];
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) sums[q][cb][i] = 0.0f;
  constexpr int U = 4;
  for (int s = s0; s < s1; s += U) {
    sg_f4 x0[U], x1[U];
    uint4 b[U][NCB][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int su = s + u < s1 ? s + u : s1 - 1;
      // (a contraction length that is an odd multiple of 8 ends in half a step: its second half repeats the first, with
      // zero weights)
      const int k = su * 16 + 8 * hh < K ? su * 16 : su * 16 - 8;
      x0[u] = *reinterpret_cast<const sg_f4*>(a + k);
      x1[u] = *reinterpret_cast<const sg_f4*>(a + k + 4);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        b[u][cb][0] = w[((size_t)su * n_cb + cb) * 128];
        b[u][cb][1] = w[((size_t)su * n_cb + cb) * 128 + 64];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s + u < s1) {
        const float v[8] = {x0[u][0], x0[u][1], x0[u][2], x0[u][3], x1[u][0], x1[u][1], x1[u][2], x1[u][3]};
        uint4 ah, al;
        sgh_split8(v, a_scale, ah, al);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          sums[2][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(al), sgh_as_h8(b[u][cb][0]), sums[2][cb], 0, 0, 0);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          sums[2][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(ah), sgh_as_h8(b[u][cb][1]), sums[2][cb], 0, 0, 0);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          sums[u % 2][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(ah), sgh_as_h8(b[u][cb][0]), sums[u % 2][cb], 0, 0, 0);
      }
    }
  }
  float16v acc[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) acc[cb] = sums[0][cb] + (sums[1][cb] + sums[2][cb]);
  if (wave > 0) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) s_part[wave - 1][(cb * 16 + i) * 64 + lane] = acc[cb][i];
  }
  __syncthreads();
  if (wave > 0) return;
  const int D = (p.lmax + 1) * (p.lmax + 1);
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const int col = (cb0 + cb) * 32 + l32;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float sum = acc[cb][i] + s_part[0][(cb * 16 + i) * 64 + lane] + s_part[1][(cb * 16 + i) * 64 + lane] +
                        s_part[2][(cb * 16 + i) * 64 + lane];
      const int r32 = 8 * (i >> 2) + 4 * hh + (i & 3);
      const long r = r0 + r32;
      const int e_row = __shfl(ea, r32);
      if (r < rows && col < p.E) {
        const long n = r / (2 * lo + 1);
        p.out[((size_t)n * D + lo * lo + (r - n * (2 * lo + 1))) * p.E + col] = p.scale * ldexpf(sum, -e_row - eb);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------- weight gradient
struct So2nWgrad {
  const float* T;        // form SO2N_PLAIN, of n_nodes nodes
  const float* x;        // [n_nodes][(lmax+1)^2][E]
  const float* G;        // of n_G <= n_nodes nodes
  const float* da;       // [n_G][(lmax+1)^2][E]
  float* partial;
  int node_floats, off[5], ld[5], K[5];   // K: rows of the result, those of T and then SO2N_AUX of G
  int k_tiles[5], chunks[5], per_chunk[5], unit0[6];
  size_t part0[6];       // first float of every degree's partial results
  int n_nodes, n_G, E, n_ct, D;
  const int* node_exp[2];   // scales of T and G (so2n_pack_kernel)
  const unsigned* used;
};

// partial[l][chunk][k][col] = sum over the nodes n of the chunk and m of T[n][(l, m)][k] x[n][(l, m)][col].  T are the sums over
// the outgoing edges that dx is made of (l an input degree of the message, k = (group, path to an output degree, its channel), col
// an input channel): sum_edges Yhat x_src da_dst is the same number whether it is gathered at one end or at the other, so the sums
// over the incoming edges need not be formed again (445 of 1,815 us of a call and its adjoint at 3,000 nodes).  A wave
// owns 128 rows x 32 columns of the result; both operands are read in memory order, the contraction index being the row
// index of both: lane (i, h) fetches 16 bytes of T and 4 of x for the eight nodes of its half-wave and finds in one
// component of them the eight consecutive nodes one operand register wants, so accumulator a holds the rows
// k0 + 4 r + a.  Degrees with more rows per node get fewer nodes per chunk, so that all waves take about equally long.  The
// last wave of every column of tiles takes G and da in the place of T and x, with G's own scales: whichever of the two is the smaller keeps
// its accuracy.
// Bound: T read once (403 MB at 3,000 nodes, lmax 4, 32 channels: 105 us = 3.8 TB/s, of which the scales per node and G take 10;
// per edge it was 2.26 ms).
__global__ __launch_bounds__(256, 2) void so2n_wgrad_kernel(So2nWgrad p) {
  const int lane = threadIdx.x & 63, i32 = lane & 31, hh = lane >> 5;
  const int unit = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  int lo = 0;
  while (lo < 5 && unit >= p.unit0[lo + 1]) ++lo;
  if (lo >= 5) return;                             // (no barrier in this kernel)
  int u = unit - p.unit0[lo];
  const int kt = u % p.k_tiles[lo];
  u /= p.k_tiles[lo];
  const int ct = u % p.n_ct, chunk = u / p.n_ct;
  const bool basis = kt == p.k_tiles[lo] - 1;
  const int k_first = basis ? p.K[lo] - SO2N_AUX : kt * 128, n_mo = 2 * lo + 1;
  const int K = basis ? SO2N_AUX : p.K[lo] - SO2N_AUX - k_first;           // rows this wave can have
  const int n_n = basis ? p.n_G : p.n_nodes;
  const int n0 = chunk * p.per_chunk[lo], n1 = n0 + p.per_chunk[lo] < n_n ? n0 + p.per_chunk[lo] : n_n;
  const int ca = 4 * i32, cy = ct * 32 + i32;
  const bool a_ok = ca < K, y_ok = cy < p.E;
  const unsigned largest = p.used[basis ? 1 : 0];
  const int ey = largest ? 13 + SO2N_EXP0 - (int)largest : 0;
  const int* node_exp = p.node_exp[basis ? 1 : 0];
  const float* T = (basis ? p.G + lo * lo * SO2N_AUX : p.T + p.off[lo] + k_first) + (a_ok ? ca : K - 4);
  const int ld = basis ? SO2N_AUX : p.ld[lo], node_floats = basis ? p.D * SO2N_AUX : p.node_floats;
  const float* Y = (basis ? p.da : p.x) + (size_t)(lo * lo) * p.E + (y_ok ? cy : 0);
  const size_t ys = (size_t)p.D * p.E;
  float16v acc[4], rest[4];      // (as in so2n_mix_kernel)
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[a][i] = rest[a][i] = 0.0f;
  sg_f4 ra[8];
  float ry[8];
  int re[8];
  const int n_blocks = n1 > n0 ? (n1 - n0 + 15) / 16 : 0, total = n_blocks * n_mo;   // (a chunk past G's nodes: zeros)
  auto fetch = [&](int q) SO2N_INLINE {
    const int mo = q / n_blocks, n = n0 + (q - mo * n_blocks) * 16 + 8 * hh;
    const int4 e0 = *reinterpret_cast<const int4*>(node_exp + n), e1 = *reinterpret_cast<const int4*>(node_exp + n + 4);
    re[0] = e0.x; re[1] = e0.y; re[2] = e0.z; re[3] = e0.w; re[4] = e1.x; re[5] = e1.y; re[6] = e1.z; re[7] = e1.w;
    const float* tm = T + (size_t)mo * ld;
    const float* ym = Y + (size_t)mo * p.E;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      // (past the last node: that node again, with zeros for x or da)
      const int nr = n + r < n1 ? n + r : n1 - 1;
      ra[r] = *reinterpret_cast<const sg_f4*>(tm + (size_t)nr * node_floats);
      ry[r] = ym[(size_t)nr * ys];
    }
  };
  if (total) fetch(0);
  for (int q = 0; q < total; ++q) {
    uint4 ah[4], al[4], yh, yl;
    float y[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) y[r] = re[r] != SO2N_UNUSED ? ldexpf(ry[r], ey - re[r]) : 0.0f;
    sgh_split8(y, 1.0f, yh, yl);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      float x[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) x[r] = ldexpf(ra[r][a], re[r]);
      sgh_split8(x, 1.0f, ah[a], al[a]);
    }
    fetch(q + 1 < total ? q + 1 : q);
#pragma unroll
    for (int a = 0; a < 4; ++a) rest[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(al[a]), sgh_as_h8(yh), rest[a], 0, 0, 0);
#pragma unroll
    for (int a = 0; a < 4; ++a) rest[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(ah[a]), sgh_as_h8(yl), rest[a], 0, 0, 0);
#pragma unroll
    for (int a = 0; a < 4; ++a) acc[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(sgh_as_h8(ah[a]), sgh_as_h8(yh), acc[a], 0, 0, 0);
  }
  if (y_ok) {
    float* out = p.partial + p.part0[lo] + ((size_t)chunk * p.K[lo] + k_first) * p.E + cy;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int k = 4 * (8 * (i >> 2) + 4 * hh + (i & 3)) + a;
        if (k < K) out[(size_t)k * p.E] = ldexpf(acc[a][i] + rest[a][i], -ey);
      }
  }
}

// dW of the path weights [k][col], all degrees: the chunks' partial results added in order, times scale
__global__ __launch_bounds__(256) void so2n_wgrad_sum_kernel(So2nWgrad p, So2nW s, int lmax, float scale, float* __restrict__ out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long)s.k_first[lmax + 1] * p.E) return;
  const int row = (int)(i / p.E);
  int lo = 0;
  while (row >= s.k_first[lo + 1]) ++lo;
  const size_t n = (size_t)p.K[lo] * p.E;
  const float* part = p.partial + p.part0[lo] + (i - (long)s.k_first[lo] * p.E);
  float sum = 0.0f;
  int c = 0;
  for (; c + 4 <= p.chunks[lo]; c += 4) {
    const float v0 = part[(size_t)c * n], v1 = part[(size_t)(c + 1) * n], v2 = part[(size_t)(c + 2) * n], v3 = part[(size_t)(c + 3) * n];
    sum += v0;
    sum += v1;
    sum += v2;
    sum += v3;
  }
  for (; c < p.chunks[lo]; ++c) sum += part[(size_t)c * n];
  out[i] = scale * sum;
}

// gradient of the path weights (rows of an input degree, columns its channels: neighbouring threads read neighbouring words; and
// rows of G of an output degree, columns that degree's channels) -> gradient of W_0 / (Wr_m, Wi_m) in their layout; and of W_e, a
// wavefront per element in the last workgroups (a thread per element, 160 products one after the other: 66 us in all)
__global__ __launch_bounds__(256) void so2n_unpack_wgrad_kernel(const float* __restrict__ dwp, So2nW s, int lmax, int E, int n_rbf,
                                                                const float* __restrict__ W, const float* __restrict__ W_e,
                                                                float* __restrict__ dW, float* __restrict__ dW_e) {
  const long n_w = (long)s.off[5], w_blocks = (n_w + 255) / 256;
  if ((long)blockIdx.x >= w_blocks) {
    const int e = (int)(blockIdx.x - w_blocks) * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (e >= E * n_rbf) return;
    const int ci = e / n_rbf, b = e - ci * n_rbf;
    float sum = 0.0f;
    for (int lo = 0; lo <= lmax; ++lo) {
      const float* d = dwp + (size_t)(s.k_first[lo] + 2 * so2n_paths(lmax, lo) * E + b) * E;
      const float* row = W + (size_t)(lo * E) * ((lmax + 1) * 3 * E) + 2 * E + ci;
      float part = 0.0f;
      for (int co = lane; co < E; co += 64) part += row[(size_t)co * ((lmax + 1) * 3 * E)] * d[co];
      sum += part / sqrtf((float)(2 * lo + 1));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) dW_e[e] = sum;
    return;
  }
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_w) return;
  int m = 0;
  while (m < lmax && i >= (long)s.off[m + 1]) ++m;
  long r = i - (long)s.off[m];
  const int nl = lmax + 1 - m, cols = nl * 3 * E;
  const int odd = r >= (long)nl * E * cols ? 1 : 0;
  if (odd) r -= (long)nl * E * cols;
  const int row = (int)(r / cols), col = (int)(r - (long)row * cols);
  const int lo = m + row / E, co = row % E, li = m + col / (3 * E), rem = col % (3 * E), g = rem / E, ci = rem % E;
  const int np = so2n_paths(lmax, lo), d = lo > li ? lo - li : li - lo;
  float sum = 0.0f;
  if (g < 2) {
    for (int L = d; L <= lo + li; ++L)
      if (((lo + li + L) & 1) == odd)
        sum += SO2N_BETA[lo][li][L - d][m] *
               dwp[(size_t)(s.k_first[li] + (g * so2n_paths(lmax, li) + so2n_path_base(li, lo) + L - d) * E + co) * E + ci];
    if (odd) sum = -sum;                 // (swapping the two degrees of a coupling tensor, see so2n_weight)
  } else if (m == 0 && li == 0) {
    // (the edge's other planes are zero on this path, and so are their weights' gradients)
    for (int b = 0; b < n_rbf; ++b)
      sum += dwp[(size_t)(s.k_first[lo] + 2 * np * E + b) * E + co] * W_e[ci * n_rbf + b];
    sum /= sqrtf((float)(2 * lo + 1));
  }
  dW[i] = sum;
}

// ---------------------------------------------------------------------------------------------- host side
static size_t so2n_a256(size_t n) { return (n + 255) & ~(size_t)255; }

static void so2n_w_layout(int lmax, int E, int form, So2nW* s, So2nSteps* st) {
  size_t off = 0;
  s->k_first[0] = st->first[0] = 0;
  for (int m = 0; m < 5; ++m) { s->off[m] = 0; s->K[m] = 0; }
  for (int m = 0; m <= lmax; ++m) {
    s->off[m] = off;
    const size_t nl = lmax + 1 - m;
    off += (m == 0 ? 1 : 2) * (nl * E) * (nl * 3 * E);
  }
  s->off[5] = off;
  for (int lo = 0; lo <= lmax; ++lo) {
    s->K[lo] = so2n_ld(lmax, E, lo, form);
    s->k_first[lo + 1] = s->k_first[lo] + s->K[lo];
    st->first[lo + 1] = st->first[lo] + (s->K[lo] + 15) / 16;
  }
  for (int lo = lmax + 1; lo < 5; ++lo) {
    s->k_first[lo + 1] = s->k_first[lo];
    st->first[lo + 1] = st->first[lo];
  }
}

static size_t so2n_packed_bytes(const egnn_ctx* ctx, long n_rows) {   // (a last, partial tile of columns reads past its row)
  return (size_t)n_rows * (ctx->desc.lmax + 1) * (ctx->desc.lmax + 1) * ctx->desc.channels * 4 + 128;
}

size_t so2n_carve(const egnn_ctx* ctx, int32_t n_owned, int32_t n_rows, int32_t n_t, int form, char* base, So2nCall* out) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  size_t used = 0;
  auto take = [&](size_t bytes) { char* q = base ? base + used : nullptr; used += so2n_a256(bytes); return q; };
  So2nW s;
  So2nSteps st;
  so2n_w_layout(lmax, E, form, &s, &st);
  So2nCall c;
  c.maxima = (unsigned*)take(256 + (size_t)n_t * 4);
  c.t_max = c.maxima ? c.maxima + 64 : nullptr;
  c.packed = (uint32_t*)take(so2n_packed_bytes(ctx, n_rows));
  c.row_exp = (int*)take((size_t)n_rows * 4);
  c.g = (float*)take((size_t)n_owned * so2n_nlm(lmax) * 4);
  c.wpath = (float*)take(((size_t)s.k_first[lmax + 1] + SO2N_AUX) * E * 4);
  c.wpack = (uint4*)take((size_t)st.first[lmax + 1] * ((E + 31) / 32) * 128 * 16);
  c.T = (float*)take((size_t)n_t * so2n_node_off(lmax, E, lmax + 1, form) * 4);
  c.partial = c.dwpath = c.G = nullptr;
  c.G_max = nullptr;
  c.node_exp[0] = c.node_exp[1] = nullptr;
  if (out) *out = c;
  return used;
}

static int so2n_launch_pack(egnn_ctx* ctx, So2nPack p, hipStream_t st) {
  if (p.n_rows <= 0) return EGNN_OK;
  p.row_floats = (ctx->desc.lmax + 1) * (ctx->desc.lmax + 1) * ctx->desc.channels;
  hipLaunchKernelGGL(so2n_pack_kernel, dim3((unsigned)std::min((p.n_rows + 3) / 4, 2048)), dim3(256), 0, st, p);
  EGNN_LAUNCH_CHECK(ctx, "so2n_pack_kernel");
  return EGNN_OK;
}
static int so2n_pack_features(egnn_ctx* ctx, const float* x, int n_rows, const So2nCall& c, hipStream_t st) {
  So2nPack p = {};
  p.x = x; p.n_rows = n_rows; p.out = c.packed; p.row_exp = c.row_exp;
  return so2n_launch_pack(ctx, p, st);
}

static int so2n_pack_weights(egnn_ctx* ctx, const float* W, const float* W_e, int form, bool transposed, const So2nCall& c,
                             hipStream_t st) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  So2nW s;
  So2nSteps steps;
  so2n_w_layout(lmax, E, form, &s, &steps);
  const long n = (long)s.k_first[lmax + 1] * E + (W_e ? SO2N_AUX * E : 0);
  hipLaunchKernelGGL(so2n_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, W, W_e, s, lmax, E,
                     ctx->desc.n_rbf, form, transposed, c.wpath, c.maxima + 1);
  EGNN_LAUNCH_CHECK(ctx, "so2n_weights_kernel");
  const int n_cb = (E + 31) / 32;
  const long m = (long)steps.first[lmax + 1] * n_cb * 64;
  hipLaunchKernelGGL(so2n_wpack_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, c.wpath, s, steps, lmax, E, n_cb,
                     c.maxima + 1, c.wpack);
  EGNN_LAUNCH_CHECK(ctx, "so2n_wpack_kernel");
  return EGNN_OK;
}

template <int LMAX, int CS, bool OWN>
static int so2n_launch_gather_t(egnn_ctx* ctx, const So2nArgs& a, hipStream_t st) {
  constexpr size_t lds = so2n_lds_bytes(LMAX, CS);
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(so2n_gather_kernel<LMAX, CS, OWN>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return egnn_check_hip(ctx, e, "hipFuncSetAttribute(so2n_gather_kernel)");
  }
  hipLaunchKernelGGL((so2n_gather_kernel<LMAX, CS, OWN>), dim3(8u * a.per_xcd * a.n_slices), dim3(SO2N_THREADS), lds, st, a);
  EGNN_LAUNCH_CHECK(ctx, "so2n_gather_kernel");
  return EGNN_OK;
}

template <bool OWN>
static int so2n_launch_gather(egnn_ctx* ctx, So2nArgs a, hipStream_t st) {
  const int n = a.j_end - a.j_begin;
  if (n <= 0) return EGNN_OK;
  a.E = ctx->desc.channels;
  a.r_cut = ctx->desc.r_cut;
  a.n_slices = (a.E + 31) / 32;
  a.per_xcd = (n + 7) / 8;
#define SO2N_L(L)                                                     \
  switch (so2n_cs(a.E)) {                                             \
    case 8: return so2n_launch_gather_t<L, 8, OWN>(ctx, a, st);       \
    case 16: return so2n_launch_gather_t<L, 16, OWN>(ctx, a, st);     \
    default: return so2n_launch_gather_t<L, 32, OWN>(ctx, a, st);     \
  }
  switch (ctx->desc.lmax) {
    case 0: SO2N_L(0)
    case 1: SO2N_L(1)
    case 2: SO2N_L(2)
    case 3: SO2N_L(3)
    default: SO2N_L(4)
  }
#undef SO2N_L
}

// g of the owned nodes and, with n_rbf, the edge embedding's columns of T (after so2n_pack_weights with W_e) or G
static int so2n_launch_sums(egnn_ctx* ctx, const egnn_graph* g, const float* rhat_d, const float* alpha, int n_rbf, bool embed,
                            const So2nCall& c, hipStream_t st) {
  if (g->n_owned <= 0) return EGNN_OK;
  So2nW s;
  So2nSteps steps;
  so2n_w_layout(ctx->desc.lmax, ctx->desc.channels, SO2N_GAUSS, &s, &steps);
  const float* W_e = embed ? c.wpath + (size_t)s.k_first[ctx->desc.lmax + 1] * ctx->desc.channels : nullptr;
  So2nSums p;
  p.ptr = g->row_ptr; p.rhat_d = reinterpret_cast<const float4*>(rhat_d); p.alpha = alpha; p.W_e = W_e; p.g = c.g;
  p.G = W_e ? nullptr : c.G; p.T = c.T; p.t_max = c.t_max; p.G_max = c.G_max; p.n_rbf = n_rbf; p.log2E = ctx->log2_channels; p.r_cut = ctx->desc.r_cut;
  const dim3 grid((unsigned)g->n_owned), block(64 * SO2N_SUM_WAVES);
  switch (ctx->desc.lmax) {
    case 0: hipLaunchKernelGGL(so2n_sums_kernel<0>, grid, block, 0, st, p); break;
    case 1: hipLaunchKernelGGL(so2n_sums_kernel<1>, grid, block, 0, st, p); break;
    case 2: hipLaunchKernelGGL(so2n_sums_kernel<2>, grid, block, 0, st, p); break;
    case 3: hipLaunchKernelGGL(so2n_sums_kernel<3>, grid, block, 0, st, p); break;
    default: hipLaunchKernelGGL(so2n_sums_kernel<4>, grid, block, 0, st, p); break;
  }
  EGNN_LAUNCH_CHECK(ctx, "so2n_sums_kernel");
  return EGNN_OK;
}

static int so2n_launch_mix(egnn_ctx* ctx, const So2nCall& c, int form, int n_nodes, float scale, float* out, hipStream_t st) {
  if (n_nodes <= 0) return EGNN_OK;
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  So2nMix p;
  So2nW s;
  so2n_w_layout(lmax, E, form, &s, &p.st);
  p.T = c.T;
  p.node_floats = so2n_node_off(lmax, E, lmax + 1, form);
  p.w = c.wpack;
  p.n_nodes = n_nodes; p.lmax = lmax; p.E = E; p.scale = scale; p.out = out; p.t_max = c.t_max;
  p.w_max = c.maxima + 1;
  p.blocks[0] = 0;
  for (int lo = 0; lo < 5; ++lo) {
    p.K[lo] = s.K[lo];
    p.ld[lo] = so2n_ld(lmax, E, lo, form);
    p.off[lo] = so2n_node_off(lmax, E, lo, form);
    p.blocks[lo + 1] = p.blocks[lo] + (lo <= lmax ? (int)(((long)n_nodes * (2 * lo + 1) + 31) / 32) : 0);
  }
  const dim3 grid((unsigned)p.blocks[lmax + 1]), block(256);
  if (E <= 32) hipLaunchKernelGGL(so2n_mix_kernel<1>, grid, block, 0, st, p);
  else if (E == 64) hipLaunchKernelGGL(so2n_mix_kernel<2>, grid, block, 0, st, p);
  else hipLaunchKernelGGL(so2n_mix_kernel<2>, dim3(grid.x, 2), block, 0, st, p);
  EGNN_LAUNCH_CHECK(ctx, "so2n_mix_kernel");
  return EGNN_OK;
}

static void so2n_wgrad_plan(const egnn_ctx* ctx, int n_nodes, int n_owned, So2nWgrad* p) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  p->node_floats = so2n_node_off(lmax, E, lmax + 1, SO2N_PLAIN);
  p->n_nodes = n_nodes; p->n_G = n_owned; p->E = E; p->n_ct = (E + 31) / 32; p->D = (lmax + 1) * (lmax + 1);
  int tiles = 0;
  auto k_tiles = [&](int lo) { return (so2n_ld(lmax, E, lo, SO2N_PLAIN) + 127) / 128 + 1; };
  for (int lo = 0; lo <= lmax; ++lo) tiles += (2 * lo + 1) * k_tiles(lo) * p->n_ct;
  // about 2,048 waves (two per SIMD): rows (node, mo) per wave, in steps of 16 nodes
  const long rows = std::max<long>(16, ((long)n_nodes * tiles + 2047) / 2048);
  p->unit0[0] = 0;
  p->part0[0] = 0;
  for (int lo = 0; lo < 5; ++lo) {
    const bool there = lo <= lmax;
    p->K[lo] = there ? so2n_ld(lmax, E, lo, SO2N_GRAD) : 0;
    p->ld[lo] = there ? so2n_ld(lmax, E, lo, SO2N_PLAIN) : 0;
    p->off[lo] = there ? so2n_node_off(lmax, E, lo, SO2N_PLAIN) : 0;
    p->k_tiles[lo] = there ? k_tiles(lo) : 1;
    p->per_chunk[lo] = (int)((rows / (2 * lo + 1) + 15) / 16 * 16);
    if (p->per_chunk[lo] < 16) p->per_chunk[lo] = 16;
    p->chunks[lo] = there ? (n_nodes + p->per_chunk[lo] - 1) / p->per_chunk[lo] : 0;
    p->unit0[lo + 1] = p->unit0[lo] + p->chunks[lo] * p->k_tiles[lo] * p->n_ct;
    p->part0[lo + 1] = p->part0[lo] + (size_t)p->chunks[lo] * p->K[lo] * E;
  }
}

size_t so2n_backward_carve(const egnn_ctx* ctx, int32_t n_owned, int32_t n_total, char* base, So2nCall* out) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  size_t used = so2n_carve(ctx, n_owned, n_total, n_total, SO2N_PLAIN, base, out);
  auto take = [&](size_t bytes) { char* q = base ? base + used : nullptr; used += so2n_a256(bytes); return q; };
  So2nW s;
  So2nSteps st;
  so2n_w_layout(lmax, E, SO2N_GRAD, &s, &st);
  So2nWgrad p;
  so2n_wgrad_plan(ctx, n_total, n_owned, &p);
  float* partial = (float*)take(p.part0[lmax + 1] * 4);
  float* dwpath = (float*)take((size_t)s.k_first[lmax + 1] * E * 4);
  float* G = (float*)take((size_t)n_owned * (lmax + 1) * (lmax + 1) * SO2N_AUX * 4);
  unsigned* G_max = (unsigned*)take((size_t)n_owned * 4);
  int* exps[2];
  for (int z = 0; z < 2; ++z) exps[z] = (int*)take(((size_t)(z ? n_owned : n_total) + 16) * 4);
  if (out) {
    out->partial = partial; out->dwpath = dwpath; out->G = G; out->G_max = G_max;
    out->node_exp[0] = exps[0]; out->node_exp[1] = exps[1];
  }
  return used;
}

// Reverse pass of the message sum.  The sums of the forward pass over the outgoing edges, with da in the place of the features (a
// message is linear in its source, and the transpose of D_lo^T P D_li is D_li^T P^T D_lo), and the transposed weights -> dx;
// the destinations' part uses the forward pass's sums of harmonics.  The same sums against the features -> gradient of the path
// weights and, from that, of W and W_e.  c from so2n_backward_carve, its maxima and t_max zero on entry.
int so2n_message_sum_backward(egnn_ctx* ctx, const egnn_graph* g, const int32_t* col_ptr, const int32_t* perm, const float* rhat_d,
                              const float* x, const float* W_e, const float* W, const float* da, float scale, float* dx,
                              float* dW_e, float* dW, const So2nCall& c, hipStream_t st) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  int rc;
  if ((rc = so2n_launch_sums(ctx, g, rhat_d, nullptr, ctx->desc.n_rbf, false, c, st))) return rc;
  So2nPack q = {};
  q.x = da; q.n_rows = g->n_owned; q.out = c.packed; q.row_exp = c.row_exp;
  q.X_max = c.G_max; q.ptr = g->row_ptr; q.n_ptr = g->n_owned; q.node_exp = c.node_exp[1]; q.used = c.maxima + 5;
  if ((rc = so2n_launch_pack(ctx, q, st))) return rc;
  So2nArgs p = {};
  p.ptr = col_ptr; p.perm = perm; p.index = g->dst; p.rhat_d = reinterpret_cast<const float4*>(rhat_d);
  p.packed = c.packed; p.row_exp = c.row_exp; p.packed_bytes = (unsigned)so2n_packed_bytes(ctx, g->n_owned); p.x_self = da;
  p.T = c.T; p.t_max = c.t_max; p.g = c.g;
  p.j_begin = 0; p.j_end = g->n_total; p.n_self = g->n_owned; p.self_ptr = g->row_ptr; p.form = SO2N_PLAIN;
  if ((rc = so2n_launch_gather<false>(ctx, p, st))) return rc;
  q.x = x; q.n_rows = g->n_total; q.out = nullptr; q.row_exp = nullptr;
  q.X_max = c.t_max; q.col_ptr = col_ptr; q.node_exp = c.node_exp[0]; q.used = c.maxima + 4;
  if ((rc = so2n_launch_pack(ctx, q, st))) return rc;
  So2nW s;
  So2nSteps steps;
  so2n_w_layout(lmax, E, SO2N_GRAD, &s, &steps);
  So2nWgrad w;
  so2n_wgrad_plan(ctx, g->n_total, g->n_owned, &w);
  w.T = c.T; w.x = x; w.G = c.G; w.da = da; w.partial = c.partial; w.used = c.maxima + 4;
  w.node_exp[0] = c.node_exp[0]; w.node_exp[1] = c.node_exp[1];
  hipLaunchKernelGGL(so2n_wgrad_kernel, dim3((w.unit0[5] + 3) / 4), dim3(256), 0, st, w);
  EGNN_LAUNCH_CHECK(ctx, "so2n_wgrad_kernel");
  const long n_wp = (long)s.k_first[lmax + 1] * E;
  hipLaunchKernelGGL(so2n_wgrad_sum_kernel, dim3((unsigned)((n_wp + 255) / 256)), dim3(256), 0, st, w, s, lmax, scale, c.dwpath);
  EGNN_LAUNCH_CHECK(ctx, "so2n_wgrad_sum_kernel");
  const long un_blocks = ((long)s.off[5] + 255) / 256 + ((long)E * ctx->desc.n_rbf + 3) / 4;
  hipLaunchKernelGGL(so2n_unpack_wgrad_kernel, dim3((unsigned)un_blocks), dim3(256), 0, st, c.dwpath, s, lmax, E,
                     ctx->desc.n_rbf, W, W_e, dW, dW_e);
  EGNN_LAUNCH_CHECK(ctx, "so2n_unpack_wgrad_kernel");
  if ((rc = so2n_pack_weights(ctx, W, nullptr, SO2N_PLAIN, true, c, st))) return rc;
  return so2n_launch_mix(ctx, c, SO2N_PLAIN, g->n_total, scale, dx, st);
}

// a[j] for the owned nodes; rhat_d and c carved by the caller, c.maxima and c.t_max zero on entry
int so2n_message_sum(egnn_ctx* ctx, const egnn_graph* g, const float* rhat_d, const float* x, const float* W_e, const float* W,
                     float scale, float* a, const So2nCall& c, hipStream_t st) {
  int rc;
  if ((rc = so2n_pack_features(ctx, x, g->n_total, c, st))) return rc;
  if ((rc = so2n_pack_weights(ctx, W, W_e, SO2N_GAUSS, false, c, st))) return rc;
  So2nArgs p = {};
  p.ptr = g->row_ptr; p.index = g->src; p.rhat_d = reinterpret_cast<const float4*>(rhat_d);
  p.packed = c.packed; p.row_exp = c.row_exp; p.packed_bytes = (unsigned)so2n_packed_bytes(ctx, g->n_total); p.x_self = x;
  p.T = c.T; p.t_max = c.t_max; p.g = c.g;
  p.j_begin = 0; p.j_end = g->n_owned; p.n_self = g->n_owned; p.self_ptr = g->row_ptr; p.form = SO2N_GAUSS;
  if ((rc = so2n_launch_sums(ctx, g, rhat_d, nullptr, ctx->desc.n_rbf, true, c, st))) return rc;
  if ((rc = so2n_launch_gather<false>(ctx, p, st))) return rc;
  return so2n_launch_mix(ctx, c, SO2N_GAUSS, g->n_owned, scale, a, st);
}

// Node block: scores, their softmax, then the sums over the incoming edges weighted with it: source and destination as in the
// message sum, the edges' own rows by a second gathering launch into the third group.
int so2n_node_block(egnn_ctx* ctx, const egnn_graph* g, const float* rhat_d, const float* x, const float* T_edge, const float* W,
                    const float* w_att, float* alpha, float* a, const So2nCall& c, hipStream_t st) {
  const int lmax = ctx->desc.lmax, E = ctx->desc.channels;
  int rc;
  if ((rc = so2n_pack_features(ctx, x, g->n_total, c, st))) return rc;
  if ((rc = so2n_pack_weights(ctx, W, nullptr, SO2N_EDGES, false, c, st))) return rc;
  const size_t lds = std::max<size_t>(32 * (size_t)((lmax + 1) * E + 4) * 4, 16384);
  const dim3 grid((unsigned)((g->n_edges + 31) / 32));
  const unsigned x_bytes = (unsigned)((size_t)g->n_total * (lmax + 1) * (lmax + 1) * E * 4);   // (32 bits: the caller's rule)
#define SO2N_SCORE(L)                                                                                                         \
  do {                                                                                                                        \
    if (lds > 48 * 1024) {                                                                                                    \
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(so2n_score_kernel<L>),                                 \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                               \
      if (e != hipSuccess) return egnn_check_hip(ctx, e, "hipFuncSetAttribute(so2n_score_kernel)");                           \
    }                                                                                                                         \
    hipLaunchKernelGGL(so2n_score_kernel<L>, grid, dim3(256), lds, st, g->src, g->dst, reinterpret_cast<const float4*>(rhat_d), \
                       x, x_bytes, T_edge, W, w_att, alpha, (long)g->n_edges, ctx->log2_channels, c.maxima + 3);              \
  } while (0)
  switch (lmax) {
    case 0: SO2N_SCORE(0); break;
    case 1: SO2N_SCORE(1); break;
    case 2: SO2N_SCORE(2); break;
    case 3: SO2N_SCORE(3); break;
    default: SO2N_SCORE(4); break;
  }
#undef SO2N_SCORE
  EGNN_LAUNCH_CHECK(ctx, "so2n_score_kernel");
  hipLaunchKernelGGL(so2n_softmax_kernel, dim3((g->n_owned + 3) / 4), dim3(256), 0, st, g->row_ptr, alpha, g->n_owned);
  EGNN_LAUNCH_CHECK(ctx, "so2n_softmax_kernel");
  So2nArgs p = {};
  p.ptr = g->row_ptr; p.index = g->src; p.rhat_d = reinterpret_cast<const float4*>(rhat_d); p.alpha = alpha;
  p.packed = c.packed; p.row_exp = c.row_exp; p.packed_bytes = (unsigned)so2n_packed_bytes(ctx, g->n_total); p.x_self = x;
  p.T = c.T; p.t_max = c.t_max; p.g = c.g; p.form = SO2N_EDGES;
  p.j_begin = 0; p.j_end = g->n_owned; p.n_self = g->n_owned; p.self_ptr = g->row_ptr;
  if ((rc = so2n_launch_sums(ctx, g, rhat_d, alpha, 0, false, c, st))) return rc;
  if ((rc = so2n_launch_gather<false>(ctx, p, st))) return rc;
  p.rows = T_edge; p.rows_max = c.maxima + 3; p.x_self = nullptr;
  if ((rc = so2n_launch_gather<true>(ctx, p, st))) return rc;
  return so2n_launch_mix(ctx, c, SO2N_EDGES, g->n_owned, 1.0f, a, st);
}
