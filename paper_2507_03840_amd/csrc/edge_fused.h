// Internal: S3 + S4 in one kernel (edge_fused.hip), S3 + S6 in one kernel (readout_fused.hip).
#pragma once
#include "egnn_internal.h"
#define EF_WG_PER_CU 2   // workgroups of four wavefronts: two wavefronts a SIMD, 256 registers each
#define EF_CGX 2         // channel groups that share an XCD

typedef _Float16 ef_h8 __attribute__((ext_vector_type(8)));
typedef float ef_f4 __attribute__((ext_vector_type(4)));

// The compiler does not know which LDS words a load from memory to LDS writes, nor when: both waits are spelled out, and the
// fences (no instructions at this scope) keep the LDS reads on their side of them.
__device__ __forceinline__ void ef_wait_arrived() {         // the loads to LDS issued so far have arrived
  __builtin_amdgcn_s_waitcnt(0x0F70);                       // vmcnt(0)
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ void ef_wait_read() {            // the LDS reads issued so far have returned
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_s_waitcnt(0xC07F);                       // lgkmcnt(0)
}

static inline size_t ef_align(size_t b) { return (b + 255) & ~(size_t)255; }

// scratch: scales and their parts (256 bytes), A, frames, lengths, records, h in groups of four channels
struct EfScratch {
  float* scales;
  uint4* A;
  float4* frame;
  float2* length;       // and cutoff envelope of a row
  uint4* rec;
  float *h4, *t4;       // (t4: the readout's features of the destinations)
  size_t bytes;
};
static inline int ef_tiles(const egnn_ctx* ctx, int which) { return (ctx->n_paths[which] + 3) / 4; }
static inline int ef_quads(const egnn_ctx* ctx) { return ((ctx->desc.lmax + 1) * (ctx->desc.lmax + 1) + 3) / 4; }
static inline EfScratch egnn_ef_carve(const egnn_ctx* ctx, const egnn_graph* g, int which, void* base) {
  const size_t G = ctx->desc.channels / 4, n_rows = g->n_edges;
  const size_t a = 256, f = a + ef_align(G * ef_tiles(ctx, which) * 256 * sizeof(uint4)), l = f + ef_align((size_t)g->n_edges * 16),
               r = l + ef_align(n_rows * 8), h = r + ef_align(n_rows * 256),
               t = h + ef_align((size_t)g->n_total * G * ef_quads(ctx) * 64),
               end = t + (which ? ef_align((size_t)g->n_total * G * ef_quads(ctx) * 64) : 0);
  char* p = (char*)base;
  return {reinterpret_cast<float*>(p), reinterpret_cast<uint4*>(p + a), reinterpret_cast<float4*>(p + f),
          reinterpret_cast<float2*>(p + l), reinterpret_cast<uint4*>(p + r), reinterpret_cast<float*>(p + h),
          reinterpret_cast<float*>(p + t), end};
}

bool egnn_edge_fused_fits(const egnn_ctx*, const egnn_graph*);
// the steps one by one (scratch: as large as a weight tensor in fp32, one row per edge).
// For a call that needs a weight tensor as well, the steps leave what S3 and the reverse pass read, so that nothing is prepared twice:
// rhat_d (as egnn_launch_geometry writes it), w2s (for egnn_launch_radial_prepared, with rec), h in rows; each may be NULL.
int egnn_launch_edge_fused_first(egnn_ctx*, const egnn_graph*, int which, const float* pos, const float box[3],
                                 const float* W_r1, const float* W_r2, void* scratch, hipStream_t, float* rhat_d = nullptr);
int egnn_launch_edge_fused_second(egnn_ctx*, const egnn_graph*, int which, const float* W_r1, const float* W_r2, void* scratch,
                                  hipStream_t, void* w2s = nullptr);
int egnn_launch_edge_fused_features(egnn_ctx*, const egnn_graph*, const float* x_in, const float* W_pre, void* scratch,
                                    hipStream_t, float* h = nullptr);
int egnn_launch_edge_fused_sum(egnn_ctx*, const egnn_graph*, void* scratch, float* a, bool half, hipStream_t);

// S3 + S6 in one kernel (readout_fused.hip), from the same preparation with which = 1
bool egnn_readout_fused_fits(const egnn_ctx*, const egnn_graph*);
int egnn_launch_readout_fused(egnn_ctx*, const egnn_graph*, void* scratch, const float* V, float* H, bool half, hipStream_t);
