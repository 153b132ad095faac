// Edge block in one kernel (so2_edge.hip): host entry points for so2_message.hip.
#pragma once
#include "egnn_internal.h"

// largest magnitude of all weights -> *w_max, as bits, if it is larger than what is there (so2_message.hip)
int so2_launch_wmax(egnn_ctx*, const float* W, unsigned* w_max, hipStream_t);
// bytes of the weights in operand order
size_t so2e_weight_bytes(const egnn_ctx*);
// T_out = T_in + f_c (transformed message); w_max (zero on entry) and wpack are scratch.  T_out may be T_in up to 32 channels.
int so2e_edge_block(egnn_ctx*, const egnn_graph*, const float* rhat_d, const float* x, const float* T_in, const float* W,
                    float* T_out, unsigned* w_max, uint4* wpack, hipStream_t);
