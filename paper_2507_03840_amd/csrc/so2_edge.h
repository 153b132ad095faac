// Edge block in one kernel (so2_edge.hip): host entry points for so2_message.hip.
#pragma once
#include "egnn_internal.h"

// bytes of the weights in operand order
size_t so2e_weight_bytes(const egnn_ctx*);
// T_out = T_in + f_c (transformed message); w_max (zero on entry) and wpack are scratch.  T_out may be T_in up to 32 channels.
int so2e_edge_block(egnn_ctx*, const egnn_graph*, const float* rhat_d, const float* x, const float* T_in, const float* W,
                    float* T_out, unsigned* w_max, uint4* wpack, hipStream_t);
