// Internal: S3 + S4 in one kernel (edge_fused.hip).
#pragma once
#include "egnn_internal.h"
#define EF_WG_PER_CU 2   // workgroups of four wavefronts: two wavefronts a SIMD, 256 registers each
#define EF_CGX 2         // channel groups that share an XCD
bool egnn_edge_fused_fits(const egnn_ctx*, const egnn_graph*);
// the steps one by one (scratch: as large as a weight tensor in fp32, one row per edge) ...
int egnn_launch_edge_fused_first(egnn_ctx*, const egnn_graph*, const float* pos, const float box[3], const float* W_r1,
                                 const float* W_r2, void* scratch, hipStream_t);
int egnn_launch_edge_fused_second(egnn_ctx*, const egnn_graph*, const float* W_r1, const float* W_r2, void* scratch,
                                  hipStream_t);
int egnn_launch_edge_fused_features(egnn_ctx*, const egnn_graph*, const float* x_in, const float* W_pre, void* scratch,
                                    hipStream_t);
int egnn_launch_edge_fused_sum(egnn_ctx*, const egnn_graph*, void* scratch, float* a, bool half, hipStream_t);
// ... and all of them: a = the summed messages
int egnn_launch_edge_fused(egnn_ctx*, const egnn_graph*, const float* pos, const float box[3], const float* x_in,
                           const float* W_pre, const float* W_r1, const float* W_r2, void* scratch, float* a, hipStream_t);
