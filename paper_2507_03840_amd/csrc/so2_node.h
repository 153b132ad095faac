// Node-wise form of the SO(2) message sums (so2_node.hip): shapes shared by its kernels and the host code that calls them.
#pragma once
#include "egnn_internal.h"

#define SO2N_AUX 32   // columns of the Gaussian basis, padded

// Coupling paths into degree lo: (li, L) with |lo - li| <= L <= lo + li, li-major, all parities.
__host__ __device__ constexpr int so2n_path_base(int lo, int li) {
  int n = 0;
  for (int q = 0; q < li; ++q) n += 2 * (q < lo ? q : lo) + 1;
  return n;
}
__host__ __device__ constexpr int so2n_paths(int lmax, int lo) { return so2n_path_base(lo, lmax + 1); }

// The coupled sums T: per node (lmax+1)^2 rows (lo, mo) of so2n_ld(lo) floats, columns (group, path, channel) with group
// 0 = neighbours, 1 = the node itself, 2 = the edges' own rows; then, in the message sum, a column per channel of the initial
// edge embedding.  The gradient of the path weights has rows of the same order, with those of the Gaussian basis itself instead.
enum So2nForm { SO2N_PLAIN = 0, SO2N_GAUSS = 1, SO2N_EDGES = 2, SO2N_GRAD = 3 };   // two groups; message sum; three groups; gradient
__host__ __device__ constexpr int so2n_groups(int form) { return form == SO2N_EDGES ? 3 : 2; }
__host__ __device__ constexpr int so2n_ld(int lmax, int E, int lo, int form) {
  return so2n_groups(form) * so2n_paths(lmax, lo) * E + (form == SO2N_GAUSS ? E : form == SO2N_GRAD ? SO2N_AUX : 0);
}
// first float of degree lo within a node; lo = lmax + 1: floats of a node
__host__ __device__ constexpr int so2n_node_off(int lmax, int E, int lo, int form) {
  int n = 0;
  for (int q = 0; q < lo; ++q) n += (2 * q + 1) * so2n_ld(lmax, E, q, form);
  return n;
}

struct So2nCall {
  float* T;              // [n_t] nodes
  float* partial;        // reverse pass: partial gradients of the path weights
  float* dwpath;         // and their sum
  float* G;              // and [n_owned][(lmax + 1)^2][SO2N_AUX] sums of harmonics times Gaussian basis
  uint32_t* packed;      // feature rows as half-precision pieces (low piece in the high half)
  int* row_exp;          // and the exponent each was scaled with
  float* g;              // [n_owned][(2 lmax + 1)^2] weighted sums of the harmonics over the incoming edges
  float* wpath;          // path weights, fp32
  uint4* wpack;          // the same cut into pieces in operand order
  unsigned* maxima;      // bit patterns: 1 path weights, 3 edge rows; 4, 5 scales of the weight gradient
  unsigned* t_max;       // largest |T| of every one of the n_t nodes
  unsigned* G_max;       // reverse pass: largest |G| of every owned node, and the exponents that T and G are scaled with
  int* node_exp[2];
};
// words from maxima on that start at zero
inline long so2n_zero_words(int32_t n_t) { return 64 + (long)n_t; }

// base = NULL: bytes only.  n_rows feature rows, T for n_t nodes.
size_t so2n_carve(const egnn_ctx*, int32_t n_owned, int32_t n_rows, int32_t n_t, int form, char* base, So2nCall* out);
int so2n_message_sum(egnn_ctx*, const egnn_graph*, const float* rhat_d, const float* x, const float* W_e, const float* W,
                     float scale, float* a, const So2nCall&, hipStream_t);
int so2n_node_block(egnn_ctx*, const egnn_graph*, const float* rhat_d, const float* x, const float* T_edge, const float* W,
                    const float* w_att, float* alpha, float* a, const So2nCall&, hipStream_t);
size_t so2n_backward_carve(const egnn_ctx*, int32_t n_owned, int32_t n_total, char* base, So2nCall* out);
int so2n_message_sum_backward(egnn_ctx*, const egnn_graph*, const int32_t* col_ptr, const int32_t* perm, const float* rhat_d,
                              const float* x, const float* W_e, const float* W, const float* da, float scale, float* dx,
                              float* dW_e, float* dW, const So2nCall&, hipStream_t);
