// S1: radius graph (Sec. 3 "Initialization": edges i -> j within r_cut; Sec. 4.4: periodic structures).
//
// Output: all ordered pairs (src i, dst j), i != j, j owned, inside the cutoff (fp64 minimum-image predicate on
// the fp32 data, strict '<'), sorted by (dst, src), with the CSR index over destinations.
//
// Two search strategies feed the same compaction:
//   * cell list (when the caller supplies a workspace): atoms are binned into cells of edge >= r_cut; one wavefront
//     per destination atom visits the atoms of the <= 27 neighbouring cells, lists the candidates, evaluates the predicate and
//     sets a bit per accepted source in an LDS bitmap.  The bits before a source's own (popcounts, wave prefix
//     sum) say where it stands in ascending order, whatever order the cells delivered it in, so no sort
//     pass is needed and the order inside a cell (filled with integer atomics) does not matter.
//   * full sweep (no workspace, or more atoms than the bitmap holds): the wavefront sweeps all sources in index
//     order, 64 per step; a ballot collects the outcomes and its prefix popcount places the accepted ones.
// Each runs twice: a counting pass (row lengths -> exclusive scan -> row_ptr) and a filling pass, which finds most of the search's work done.
#include <algorithm>
#include "egnn_internal.h"

#define NL_MAX_CELLS_AXIS 64
#define NL_MAX_BITMAP_ATOMS 262144   // 8192 words = 32 KB of LDS per wavefront
#define NL_LIST 1024                 // candidates that the exact predicate is asked of at a time
#define NL_KEEP 256                  // sources kept per atom, halo atoms included (what those do not need the others share) ...
#define NL_KEEP_MOST (16 << 20)      // ... and the most of them in all

struct NlistGeom {
  double box[3];
  double rc2;
  int pbc[3];
};

__device__ __forceinline__ bool pair_inside(const double pj[3], const float* __restrict__ pos, int i,
                                            const NlistGeom& g, int sh[3]) {
  double d2 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double d = (double)pos[3 * i + a] - pj[a];
    sh[a] = 0;
    if (g.pbc[a] && __any(!(fabs(d) < 0.4999 * g.box[a]))) {   // (below that the image is the atom itself)
      const double n = rint(d / g.box[a]);
      d -= n * g.box[a];
      sh[a] = -(int)n;
    }
    d2 += d * d;
  }
  return d2 < g.rc2;
}

// ------------------------------------------------------------------------------------------------ full sweep
template <bool FILL>
__global__ __launch_bounds__(256) void nlist_sweep_kernel(const float* __restrict__ pos, int n_owned, int n_total,
                                                          NlistGeom g, int* __restrict__ row_ptr,
                                                          int* __restrict__ src, int* __restrict__ dst,
                                                          int8_t* __restrict__ shift) {
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= n_owned) return;
  const double pj[3] = {(double)pos[3 * j], (double)pos[3 * j + 1], (double)pos[3 * j + 2]};
  const long base = FILL ? row_ptr[j] : 0;
  const long row_end = FILL ? row_ptr[j + 1] : 0;   // the fill pass never writes past the row the count pass sized
  int count = 0;
  for (int i0 = 0; i0 < n_total; i0 += 64) {
    const int i = i0 + lane;
    int sh[3] = {0, 0, 0};
    const bool inside = (i < n_total) && (i != j) && pair_inside(pj, pos, i, g, sh);
    const unsigned long long mask = __ballot(inside);
    const long at = base + count + __popcll(mask & ((1ull << lane) - 1ull));
    if (FILL && inside && at < row_end) {
      src[at] = i;
      dst[at] = j;
      if (shift) {
        shift[3 * at + 0] = (int8_t)sh[0];
        shift[3 * at + 1] = (int8_t)sh[1];
        shift[3 * at + 2] = (int8_t)sh[2];
      }
    }
    count += __popcll(mask);
  }
  if (!FILL && lane == 0) row_ptr[j + 1] = count;
}

// ------------------------------------------------------------------------------------------------ cell list
// bounding box of all atoms: one workgroup, result as 6 floats (min xyz, max xyz)
__global__ __launch_bounds__(1024) void bbox_kernel(const float* __restrict__ pos, int n_total, float* __restrict__ out) {
  __shared__ float smin[3][1024], smax[3][1024];
  const int tid = threadIdx.x;
  float mn[3] = {3.0e38f, 3.0e38f, 3.0e38f}, mx[3] = {-3.0e38f, -3.0e38f, -3.0e38f};
  for (int i = tid; i < n_total; i += 1024)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float v = pos[3 * i + a];
      mn[a] = fminf(mn[a], v);
      mx[a] = fmaxf(mx[a], v);
    }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    smin[a][tid] = mn[a];
    smax[a][tid] = mx[a];
  }
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if (tid < off)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        smin[a][tid] = fminf(smin[a][tid], smin[a][tid + off]);
        smax[a][tid] = fmaxf(smax[a][tid], smax[a][tid + off]);
      }
    __syncthreads();
  }
  if (tid < 3) {
    out[tid] = smin[tid][0];
    out[3 + tid] = smax[tid][0];
  }
}

__device__ __forceinline__ int cell_coord(double x, int a, const CellGrid& cg) {
  double u = x - cg.lo[a];
  if (cg.pbc[a] && !(u >= 0.0 && u < cg.box[a])) u -= floor(u / cg.box[a]) * cg.box[a];
  int ci = (int)floor(u * cg.inv_cell[a]);
  return ci < 0 ? 0 : (ci >= cg.n[a] ? cg.n[a] - 1 : ci);
}

__device__ __forceinline__ int cell_index(float x, float y, float z, const CellGrid& cg) {
  const int cx = cell_coord((double)x, 0, cg), cy = cell_coord((double)y, 1, cg), cz = cell_coord((double)z, 2, cg);
  return (cx * cg.n[1] + cy) * cg.n[2] + cz;
}

__global__ void cell_count_kernel(const float* __restrict__ pos, int n_total, CellGrid cg, CellGrid* __restrict__ grid,
                                  int* __restrict__ cell_of, int* __restrict__ cell_ptr) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *grid = cg;
  if (i >= n_total) return;
  const int cell = cell_index(pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], cg);
  cell_of[i] = cell;
  atomicAdd(&cell_ptr[cell + 1], 1);   // integer count: independent of order
}

// The atoms in the order of the cells (order inside a cell is irrelevant: bitmap): position and index, or the index alone where the
// workspace has no room for more.
struct CellAtoms {
  float4* at;
  int* index;
  template <bool PLACED>
  __device__ __forceinline__ void put(int place, const float* __restrict__ pos, int i) const {
    if (PLACED) at[place] = make_float4(pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], __int_as_float(i));
    else index[place] = i;
  }
  template <bool PLACED>
  __device__ __forceinline__ float4 get(int place, const float* __restrict__ pos, int n_total) const {
    if (PLACED) return at[place];
    const int i = index[place], r = min(max(i, 0), n_total - 1);
    return make_float4(pos[3 * r], pos[3 * r + 1], pos[3 * r + 2], __int_as_float(i));
  }
};

template <bool PLACED>
__global__ void cell_fill_kernel(const float* __restrict__ pos, int n_total, const int* __restrict__ cell_of,
                                 const int* __restrict__ cell_ptr, int* __restrict__ cursor, CellAtoms cell_atoms) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_total) return;
  const int cell = cell_of[i];
  cell_atoms.put<PLACED>(cell_ptr[cell] + atomicAdd(&cursor[cell], 1), pos, i);
}

// The grid: periodic axes span the box, open axes the bounding box of the atoms (bb: min xyz, max xyz); cell edge >= r_cut (1 + 1e-6), at
// most `most` cells in all (coarser ones are cells too).
__host__ __device__ inline void cell_grid(const NlistGeom& g, const float* bb, double rc_pad, int most, CellGrid& cg) {
  double extent[3];
  cg.n_cells = 1;
  for (int a = 0; a < 3; ++a) {
    cg.pbc[a] = g.pbc[a];
    cg.box[a] = g.box[a];
    cg.lo[a] = g.pbc[a] ? 0.0 : (double)bb[a];
    extent[a] = g.pbc[a] ? g.box[a] : (double)bb[3 + a] - (double)bb[a];
    if (!(extent[a] > 0.0)) extent[a] = rc_pad;
    const double n = floor(extent[a] / rc_pad);
    cg.n[a] = n >= 1.0 ? (n < (double)NL_MAX_CELLS_AXIS ? (int)n : NL_MAX_CELLS_AXIS) : 1;
    cg.n_cells *= cg.n[a];
  }
  while (cg.n_cells > most) {
    const int a = cg.n[0] >= cg.n[1] && cg.n[0] >= cg.n[2] ? 0 : cg.n[1] >= cg.n[2] ? 1 : 2;
    cg.n_cells = cg.n_cells / cg.n[a] * (cg.n[a] / 2);
    cg.n[a] /= 2;
  }
  for (int a = 0; a < 3; ++a) cg.inv_cell[a] = (double)cg.n[a] / extent[a];
}

// The cells of a structure of up to NL_BUILD_ATOMS atoms by one workgroup, counters in LDS.  Bound by latency: 20 atoms a thread at 20,000.
// As kernels of their own (bounding box, its read-back for the host to lay out the grid, two fills, counts and places by atomics in
// memory, scan) it took 52 us of kernels and a read-back at 20,000 atoms, now 26.
#define NL_BUILD_ATOMS 32768
#define NL_BUILD_CELLS 8192
template <bool PLACED>
__global__ __launch_bounds__(1024) void cells_build_kernel(const float* __restrict__ pos, int n_total, NlistGeom g, double rc_pad,
                                                           CellGrid* __restrict__ grid, int* __restrict__ cell_of,
                                                           int* __restrict__ cell_ptr, CellAtoms cell_atoms) {
  __shared__ int s_count[NL_BUILD_CELLS];
  __shared__ float s_box[6][16];
  __shared__ int s_wave[16];
  __shared__ CellGrid s_grid;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (!(g.pbc[0] && g.pbc[1] && g.pbc[2])) {
    float b[6] = {3.0e38f, 3.0e38f, 3.0e38f, -3.0e38f, -3.0e38f, -3.0e38f};
#pragma unroll 4
    for (int i = tid; i < n_total; i += 1024)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float v = pos[3 * i + a];
        b[a] = fminf(b[a], v);
        b[3 + a] = fmaxf(b[3 + a], v);
      }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        b[a] = fminf(b[a], __shfl_xor(b[a], off));
        b[3 + a] = fmaxf(b[3 + a], __shfl_xor(b[3 + a], off));
      }
    if (lane == 0)
#pragma unroll
      for (int a = 0; a < 6; ++a) s_box[a][wave] = b[a];
  }
  for (int c = tid; c < NL_BUILD_CELLS; c += 1024) s_count[c] = 0;
  __syncthreads();
  if (tid == 0) {
    float bb[6];
    for (int a = 0; a < 6; ++a) {
      bb[a] = s_box[a][0];
      for (int w = 1; w < 16; ++w) bb[a] = a < 3 ? fminf(bb[a], s_box[a][w]) : fmaxf(bb[a], s_box[a][w]);
    }
    cell_grid(g, bb, rc_pad, NL_BUILD_CELLS, s_grid);
    *grid = s_grid;
  }
  __syncthreads();
  const CellGrid cg = s_grid;
#pragma unroll 4
  for (int i = tid; i < n_total; i += 1024) {
    const int cell = cell_index(pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], cg);
    cell_of[i] = cell;
    atomicAdd(&s_count[cell], 1);
  }
  __syncthreads();
  // exclusive scan: eight cells a thread
  int v[8], own = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    v[q] = s_count[tid * 8 + q];
    own += v[q];
  }
  int incl = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int add = __shfl_up(incl, off);
    if (lane >= off) incl += add;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  int run = incl - own;
  for (int w = 0; w < wave; ++w) run += s_wave[w];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int c = tid * 8 + q;
    if (c <= cg.n_cells) cell_ptr[c] = run;
    s_count[c] = run;
    run += v[q];
  }
  if (tid == 1023 && cg.n_cells == NL_BUILD_CELLS) cell_ptr[NL_BUILD_CELLS] = run;
  __syncthreads();
#pragma unroll 4
  for (int i = tid; i < n_total; i += 1024)
    cell_atoms.put<PLACED>(atomicAdd(&s_count[cell_of[i]], 1), pos, i);
}
static_assert(NL_BUILD_CELLS == 8 * 1024, "eight cells a thread");

// neighbour cell coordinates along one axis (without duplicates): returns the count, fills out[3]
__device__ __forceinline__ int axis_neighbours(int c, int a, const CellGrid& cg, int out[3]) {
  const int n = cg.n[a];
  if (n == 1) { out[0] = 0; return 1; }
  if (n == 2) { out[0] = 0; out[1] = 1; return 2; }
  int k = 0;
  for (int d = -1; d <= 1; ++d) {
    int v = c + d;
    if (cg.pbc[a]) v = (v + n) % n;
    else if (v < 0 || v >= n) continue;
    out[k++] = v;
  }
  return k;
}

// Candidates are told from the rest in fp32 with room for its rounding (a candidate too many is harmless, see below), the exact
// predicate is asked of those alone, 64 at a time.  With fp64 divisions for every atom of the cells, in both passes, and the
// accepted sources written by the lane that held their word, the two passes took 87 + 139 us for 12,000 + 8,000 atoms and
// 2.35 million edges; now 52 + 18, bound by the instructions of the search.  What the counting pass finds it keeps where the workspace has room
// (NlistKeep::row sources an atom); the filling pass searches again for a longer row only.
struct NlistKeep {
  int* list;       // [n_owned][row]
  int row;
};
template <bool FILL, bool PLACED>
__global__ __launch_bounds__(256) void nlist_cells_kernel(const float* __restrict__ pos, int n_owned, int n_total,
                                                          NlistGeom g, const CellGrid* __restrict__ grid,
                                                          const int* __restrict__ cell_of, const int* __restrict__ cell_ptr,
                                                          CellAtoms cell_atoms, int* __restrict__ row_ptr,
                                                          int* __restrict__ src, int* __restrict__ dst,
                                                          int8_t* __restrict__ shift, NlistKeep keep, int words) {
  extern __shared__ unsigned int lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = blockIdx.x * (blockDim.x >> 6) + wave;
  if (j >= n_owned) return;
  const double pj[3] = {(double)pos[3 * j], (double)pos[3 * j + 1], (double)pos[3 * j + 2]};
  const long base = FILL ? row_ptr[j] : 0;
  const long row_end = FILL ? row_ptr[j + 1] : 0;   // the fill pass never writes past the row the count pass sized
  int* const kept = keep.list + (size_t)j * keep.row;
  auto write = [&](long at, int i, const int sh[3]) {
    src[at] = i;
    dst[at] = j;
    if (shift) {
      shift[3 * at + 0] = (int8_t)sh[0];
      shift[3 * at + 1] = (int8_t)sh[1];
      shift[3 * at + 2] = (int8_t)sh[2];
    }
  };
  // indices read back from the workspace are clamped: a workspace overwritten between the count and the fill call
  // then gives a wrong list, never an access outside the buffers
  if (FILL && row_end - base <= keep.row) {
    for (long at = base + lane; at < row_end; at += 64) {
      const int i = min(max(kept[at - base], 0), n_total - 1);
      int sh[3];
      pair_inside(pj, pos, i, g, sh);
      write(at, i, sh);
    }
    return;
  }
  unsigned int* bitmap = lds + (size_t)wave * (2 * words + NL_LIST);     // accepted sources
  int* first = reinterpret_cast<int*>(bitmap + words);                   // how many of them lie before a word
  int* list = first + words;                                             // candidates
  for (int wi = lane; wi < words; wi += 64) bitmap[wi] = 0u;
  auto lds_order = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  };
  lds_order();
  int n_list = 0;
  bool all_listed = true;
  // the exact predicate for the candidates listed so far: those that pass are set in the bitmap, the others leave the list
  auto decide = [&]() {
    lds_order();
    for (int b = 0; b < n_list; b += 64) {
      const int i = list[min(b + lane, n_list - 1)];
      int sh[3];
      const bool inside = pair_inside(pj, pos, i, g, sh);
      if (b + lane < n_list) {
        if (inside) atomicOr(&bitmap[i >> 5], 1u << (i & 31));
        else list[b + lane] = -1;
      }
    }
    lds_order();
  };

  // The cells next to the atom's own, as runs of the cell order: up to nine columns along z, each one run, or two where it goes
  // round the box.  A lane each looks one up.
  CellGrid cg = *grid;
#pragma unroll
  for (int a = 0; a < 3; ++a) cg.n[a] = min(max(cg.n[a], 1), NL_MAX_CELLS_AXIS);
  cg.n_cells = cg.n[0] * cg.n[1] * cg.n[2];
  const int cj = min(max(cell_of[j], 0), cg.n_cells - 1);
  const int cz = cj % cg.n[2], cy = (cj / cg.n[2]) % cg.n[1], cx = cj / (cg.n[2] * cg.n[1]);
  int nx[3], ny[3];
  const int kx = axis_neighbours(cx, 0, cg, nx), ky = axis_neighbours(cy, 1, cg, ny);
  const int nz = cg.n[2];
  int lo = max(cz - 1, 0), hi = min(cz + 1, nz - 1), lo2 = 0, hi2 = -1;      // (two cells or one: all of them)
  if (nz > 2 && cg.pbc[2]) {
    if (cz == 0) lo2 = hi2 = nz - 1;
    if (cz == nz - 1) lo2 = hi2 = 0;
  }
  if (nz <= 2) { lo = 0; hi = nz - 1; }
  int a0 = 0, a1 = 0;
  {
    const int column = lane % 9, ix = column / 3, iy = column % 3, run = lane / 9;
    const int z0 = run ? lo2 : lo, z1 = run ? hi2 : hi;
    if (run < 2 && ix < kx && iy < ky && z1 >= z0) {
      const int x = ix == 0 ? nx[0] : ix == 1 ? nx[1] : nx[2], y = iy == 0 ? ny[0] : iy == 1 ? ny[1] : ny[2];
      const int cell = (x * cg.n[1] + y) * nz;
      a0 = max(cell_ptr[cell + z0], 0);
      a1 = min(cell_ptr[cell + z1 + 1], n_total);
    }
  }
  // fp32: the difference of two coordinates is rounded once (2^-24 of it), the image's multiple of the box is subtracted in one
  // rounding, and where the two precisions disagree about the image the vector is half a box long in both, off by at most 2^-22 of the
  // difference; 2^-20 of the sum of the differences covers the three axes.  A square is then off by 2 r_cut times that.
  const float rc2 = (float)g.rc2 * 1.000004f, slack = 4.0f * sqrtf((float)g.rc2) * 9.5367431640625e-7f;
  const float bx = (float)g.box[0], by = (float)g.box[1], bz = (float)g.box[2];
  const float vx = g.pbc[0] ? 1.0f / bx : 0.0f, vy = g.pbc[1] ? 1.0f / by : 0.0f, vz = g.pbc[2] ? 1.0f / bz : 0.0f;
  const float fx = pos[3 * j], fy = pos[3 * j + 1], fz = pos[3 * j + 2];
  for (int run = 0; run < 18; ++run) {
    const int r0 = __builtin_amdgcn_readlane(a0, run), r1 = __builtin_amdgcn_readlane(a1, run);
    for (int b = r0; b < r1; b += 64) {
      const float4 p = cell_atoms.get<PLACED>(min(b + lane, r1 - 1), pos, n_total);
      const int i = __float_as_int(p.w);
      const float ex = p.x - fx, ey = p.y - fy, ez = p.z - fz;
      const float dx = __builtin_fmaf(-rintf(ex * vx), bx, ex), dy = __builtin_fmaf(-rintf(ey * vy), by, ey),
                  dz = __builtin_fmaf(-rintf(ez * vz), bz, ez);
      const float d2 = dx * dx + dy * dy + dz * dz, most = rc2 + slack * (fabsf(ex) + fabsf(ey) + fabsf(ez));
      const bool near = !(d2 > most) && (unsigned)i < (unsigned)n_total && i != j && b + lane < r1;
      const unsigned long long mask = __ballot(near);
      if (near) list[n_list + __popcll(mask & ((1ull << lane) - 1ull))] = i;
      n_list += __popcll(mask);
      if (n_list > NL_LIST - 64) {           // (room for 64 more at any time)
        decide();
        n_list = 0;
        all_listed = false;
      }
    }
  }
  decide();

  // ascending order: an accepted source stands where the bits before its own say
  const int per = (words + 63) / 64, w0 = min(lane * per, words), w1 = min(w0 + per, words);
  int mine = 0;
  for (int wi = w0; wi < w1; ++wi) mine += __popc(bitmap[wi]);
  int incl = mine;   // inclusive prefix sum over the wave
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int up = __shfl_up(incl, off);
    if (lane >= off) incl += up;
  }
  const int count = __shfl(incl, 63);
  auto put = [&](int at, int i) {
    if (!FILL) {
      if (at < keep.row) kept[at] = i;
    } else if (base + at < row_end) {
      int sh[3];
      pair_inside(pj, pos, i, g, sh);
      write(base + at, i, sh);
    }
  };
  int at = incl - mine;
  if (all_listed) {
    for (int wi = w0; wi < w1; ++wi) {
      first[wi] = at;
      at += __popc(bitmap[wi]);
    }
    lds_order();
    for (int b = lane; b < n_list; b += 64) {
      const int i = list[b];
      if (i >= 0) put(first[i >> 5] + __popc(bitmap[i >> 5] & ((1u << (i & 31)) - 1u)), i);
    }
  } else {
    for (int wi = w0; wi < w1; ++wi)
      for (unsigned int bits = bitmap[wi]; bits; bits &= bits - 1, ++at) put(at, wi * 32 + __ffs(bits) - 1);
  }
  if (!FILL && lane == 0) row_ptr[j + 1] = count;
}

// ------------------------------------------------------------------------------------------------ row scan
// In-place inclusive scan of row_ptr[1..n] (row lengths) by one workgroup; row_ptr[0] = 0.
// If the total does not fit in int32 the last entry is set to -1.
// Bound by latency, and by the cache's lines per access: four consecutive counts per thread in 16 bytes, up to eight blocks of 4,096 that
// are all asked for at once, sums by shuffles, two barriers.  (Eight per thread as single words, 8,192 a round of three barriers:
// 11.5 us on average for the scans of a graph of 20,000 nodes, this 6.7; 32 single words a thread at once 20.)
#define SCAN_BLOCKS 8
struct __attribute__((packed, aligned(4))) ScanQuad { int v[4]; };     // (row_ptr + 1: not on a 16-byte boundary)
__global__ __launch_bounds__(1024) void row_scan_kernel(int* __restrict__ row_ptr, int n) {
  __shared__ long s_wave[SCAN_BLOCKS * 16];        // sums of the wavefronts, then of what lies before them
  __shared__ long s_all;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) row_ptr[0] = 0;
  long carry = 0;
  for (long base = 0; base < n; base += 4096 * SCAN_BLOCKS) {
    const int blocks = (int)min((n - base + 4095) / 4096, (long)SCAN_BLOCKS);
    ScanQuad x[SCAN_BLOCKS];
    long own[SCAN_BLOCKS], incl[SCAN_BLOCKS];
#pragma unroll
    for (int b = 0; b < SCAN_BLOCKS; ++b) {
      const long at = base + b * 4096 + tid * 4;
      if (at + 4 <= n) {
        x[b] = *reinterpret_cast<const ScanQuad*>(row_ptr + at + 1);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) x[b].v[q] = at + q < n ? row_ptr[at + q + 1] : 0;
      }
    }
#pragma unroll
    for (int b = 0; b < SCAN_BLOCKS; ++b) {
      if (b >= blocks) continue;
      own[b] = ((long)x[b].v[0] + x[b].v[1]) + ((long)x[b].v[2] + x[b].v[3]);
      incl[b] = own[b];
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const long add = __shfl_up(incl[b], off);
        if (lane >= off) incl[b] += add;
      }
      if (lane == 63) s_wave[b * 16 + wave] = incl[b];
    }
    __syncthreads();
    if (wave == 0) {                               // two sums a lane, in the order of the rows
      const long one = 2 * lane < 16 * blocks ? s_wave[2 * lane] : 0, two = 2 * lane < 16 * blocks ? s_wave[2 * lane + 1] : 0;
      long up_to = one + two;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const long add = __shfl_up(up_to, off);
        if (lane >= off) up_to += add;
      }
      s_wave[2 * lane] = up_to - one - two;
      s_wave[2 * lane + 1] = up_to - two;
      if (lane == 63) s_all = up_to;
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < SCAN_BLOCKS; ++b) {
      if (b >= blocks) continue;
      const long at = base + b * 4096 + tid * 4;
      long run = carry + s_wave[b * 16 + wave] + incl[b] - own[b];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        run += x[b].v[q];
        x[b].v[q] = run > 2147483647L ? -1 : (int)run;
      }
      if (at + 4 <= n) {
        *reinterpret_cast<ScanQuad*>(row_ptr + at + 1) = x[b];
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (at + q < n) row_ptr[at + q + 1] = x[b].v[q];
      }
    }
    carry += s_all;
    __syncthreads();
  }
}
static_assert(SCAN_BLOCKS * 16 == 128, "one wavefront adds up the wavefronts, two a lane");

int egnn_launch_row_scan(egnn_ctx* ctx, int* row_ptr, int n, hipStream_t st) {
  hipLaunchKernelGGL(row_scan_kernel, dim3(1), dim3(1024), 0, st, row_ptr, n);
  EGNN_LAUNCH_CHECK(ctx, "row_scan_kernel");
  return EGNN_OK;
}

// ------------------------------------------------------------------------------------------------ host side
static size_t a256(size_t n) { return (n + 255) & ~(size_t)255; }
static const int kMaxCells = NL_MAX_CELLS_AXIS * NL_MAX_CELLS_AXIS * NL_MAX_CELLS_AXIS;

struct CellWs {
  float* bbox;       // [6]
  CellGrid* grid;
  int* cell_of;      // [n_total]
  int* cell_ptr;     // [max cells + 1]
  int* cursor;       // [max cells]
  CellAtoms atoms;   // [n_total]
  int* kept;         // [kept_n] sources that the counting pass found
  size_t kept_n;
  size_t need, need_kept;   // bytes up to the atoms' end, up to the end of what is kept
};

// With room for the indices of the atoms alone (as much as has always been accepted) their positions are gathered, and what lies beyond
// the positions is for the sources that are kept, down to none.
static size_t least_cell_bytes(int n_total) {
  return 256 + 2 * a256((size_t)n_total * sizeof(int)) + a256(((size_t)kMaxCells + 1) * sizeof(int)) + a256((size_t)kMaxCells * sizeof(int));
}
static size_t most_cell_bytes(int n_total) {
  return least_cell_bytes(n_total) - a256((size_t)n_total * sizeof(int)) + a256((size_t)n_total * sizeof(float4)) +
         a256(std::min<size_t>((size_t)n_total * NL_KEEP, NL_KEEP_MOST) * sizeof(int));
}
static CellWs carve_cells(void* ws, size_t ws_bytes, int n_total) {
  CellWs w = {};
  size_t used = 0;
  auto take = [&](size_t bytes) { char* p = (char*)ws + used; used += a256(bytes); return p; };
  static_assert(128 + sizeof(CellGrid) <= 256, "bounding box and grid share 256 bytes");
  w.bbox = (float*)take(256);
  w.grid = (CellGrid*)((char*)w.bbox + 128);
  w.cell_of = (int*)take((size_t)n_total * sizeof(int));
  w.cell_ptr = (int*)take(((size_t)kMaxCells + 1) * sizeof(int));
  w.cursor = (int*)take((size_t)kMaxCells * sizeof(int));
  if (ws_bytes >= used + a256((size_t)n_total * sizeof(float4)))
    w.atoms.at = (float4*)take((size_t)n_total * sizeof(float4));
  else
    w.atoms.index = (int*)take((size_t)n_total * sizeof(int));
  w.need = used;
  w.kept_n = std::min({(size_t)n_total * NL_KEEP, (size_t)NL_KEEP_MOST, (ws_bytes - used) / sizeof(int)});
  w.kept = (int*)take(w.kept_n * sizeof(int));
  w.need_kept = (size_t)((char*)(w.kept + w.kept_n) - (char*)ws);
  return w;
}

extern "C" int egnn_nlist_workspace_bytes(const egnn_ctx* ctx, int32_t n_total, size_t* bytes) {
  if (!ctx || !bytes || n_total < 0) return EGNN_EINVAL;
  *bytes = most_cell_bytes(n_total);
  return EGNN_OK;
}

static int nlist_geom(egnn_ctx* ctx, const float* pos, int32_t n_owned, int32_t n_total, const float box[3],
                      const uint8_t pbc[3], NlistGeom* g) {
  if (!pos || !box || !pbc || n_owned < 0 || n_total < n_owned)
    return egnn_fail(ctx, EGNN_EINVAL, "nlist: null pointer or n_owned/n_total out of range");
  const double rc = (double)ctx->desc.r_cut;
  for (int a = 0; a < 3; ++a) {
    g->box[a] = (double)box[a];
    g->pbc[a] = pbc[a] ? 1 : 0;
    if (pbc[a] && !((double)box[a] >= 2.0 * rc))
      return egnn_fail(ctx, EGNN_EBOX, "nlist: periodic box edge shorter than 2*r_cut");
  }
  g->rc2 = rc * rc;
  return EGNN_OK;
}

static bool use_cells(const void* ws, size_t ws_bytes, int n_total) {
  return ws && n_total > 0 && n_total <= NL_MAX_BITMAP_ATOMS && ws_bytes >= least_cell_bytes(n_total);
}

// sources kept per atom
static int keep_row(const CellWs& w, int n_owned, int n_total) { return (int)std::min<size_t>(w.kept_n / n_owned, n_total); }

template <bool FILL>
static int launch_cells(egnn_ctx* ctx, const float* pos, int n_owned, int n_total, const NlistGeom& g,
                        const CellWs& w, int keep_row, int* row_ptr, int* src, int* dst, int8_t* shift, hipStream_t st) {
  const int words = (n_total + 31) / 32;
  const int waves = words <= 1024 ? 4 : 1;
  const size_t shmem = (size_t)waves * (2 * words + NL_LIST) * sizeof(unsigned int);
  const auto kernel = w.atoms.at ? nlist_cells_kernel<FILL, true> : nlist_cells_kernel<FILL, false>;
  if (shmem > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess) return egnn_check_hip(ctx, e, "hipFuncSetAttribute(nlist_cells_kernel)");
  }
  const NlistKeep keep = {w.kept, keep_row};
  hipLaunchKernelGGL(kernel, dim3((n_owned + waves - 1) / waves), dim3(64 * waves), shmem, st, pos, n_owned,
                     n_total, g, w.grid, w.cell_of, w.cell_ptr, w.atoms, row_ptr, src, dst, shift, keep, words);
  EGNN_LAUNCH_CHECK(ctx, "nlist_cells_kernel");
  return EGNN_OK;
}

extern "C" int egnn_nlist_count(egnn_ctx* ctx, const float* pos, int32_t n_owned, int32_t n_total,
                                const float box[3], const uint8_t pbc[3], int32_t* row_ptr, int64_t* n_edges,
                                void* ws, size_t ws_bytes, void* stream) {
  if (!ctx) return EGNN_EINVAL;
  NlistGeom g;
  int rc = nlist_geom(ctx, pos, n_owned, n_total, box, pbc, &g);
  if (rc) return rc;
  if (!row_ptr || !n_edges) return egnn_fail(ctx, EGNN_EINVAL, "nlist_count: null output pointer");
  if (ws && ((uintptr_t)ws & 255) != 0) return egnn_fail(ctx, EGNN_EINVAL, "nlist_count: workspace not 256-byte aligned");
  hipStream_t st = (hipStream_t)stream;
  if (n_owned > 0 && use_cells(ws, ws_bytes, n_total)) {
    const CellWs w = carve_cells(ws, ws_bytes, n_total);
    const double rc_pad = (double)ctx->desc.r_cut * (1.0 + 1e-6);
    ctx->nl_grid_atoms = n_total;   // egnn_nlist_fill walks the same cells
    ctx->nl_grid_owned = n_owned;
    ctx->nl_grid_ws = ws;
    ctx->nl_grid_ws_bytes = ws_bytes;
    ctx->nl_grid_pos = pos;
    if (n_total <= NL_BUILD_ATOMS) {
      hipLaunchKernelGGL(w.atoms.at ? cells_build_kernel<true> : cells_build_kernel<false>, dim3(1), dim3(1024), 0, st, pos, n_total, g, rc_pad, w.grid, w.cell_of, w.cell_ptr,
                         w.atoms);
      EGNN_LAUNCH_CHECK(ctx, "cells_build_kernel");
    } else {
      float bb[6] = {};
      if (!(g.pbc[0] && g.pbc[1] && g.pbc[2])) {
        hipLaunchKernelGGL(bbox_kernel, dim3(1), dim3(1024), 0, st, pos, n_total, w.bbox);
        EGNN_LAUNCH_CHECK(ctx, "bbox_kernel");
        EGNN_HIP(ctx, hipMemcpyAsync(bb, w.bbox, sizeof(bb), hipMemcpyDeviceToHost, st));
        EGNN_HIP(ctx, hipStreamSynchronize(st));
      }
      CellGrid cg;
      cell_grid(g, bb, rc_pad, kMaxCells, cg);
      if ((rc = egnn_launch_fill_int(ctx, w.cell_ptr, (long)cg.n_cells + 1, 0, st))) return rc;
      if ((rc = egnn_launch_fill_int(ctx, w.cursor, cg.n_cells, 0, st))) return rc;
      const dim3 ga((n_total + 255) / 256), b(256);
      hipLaunchKernelGGL(cell_count_kernel, ga, b, 0, st, pos, n_total, cg, w.grid, w.cell_of, w.cell_ptr);
      EGNN_LAUNCH_CHECK(ctx, "cell_count_kernel");
      if ((rc = egnn_launch_row_scan(ctx, w.cell_ptr, cg.n_cells, st))) return rc;
      hipLaunchKernelGGL(w.atoms.at ? cell_fill_kernel<true> : cell_fill_kernel<false>, ga, b, 0, st, pos, n_total, w.cell_of, w.cell_ptr, w.cursor, w.atoms);
      EGNN_LAUNCH_CHECK(ctx, "cell_fill_kernel");
    }
    if ((rc = launch_cells<false>(ctx, pos, n_owned, n_total, g, w, keep_row(w, n_owned, n_total), row_ptr, nullptr, nullptr, nullptr, st)))
      return rc;
  } else if (n_owned > 0) {
    hipLaunchKernelGGL(nlist_sweep_kernel<false>, dim3((n_owned + 3) / 4), dim3(256), 0, st, pos, n_owned, n_total,
                       g, row_ptr, (int*)nullptr, (int*)nullptr, (int8_t*)nullptr);
    EGNN_LAUNCH_CHECK(ctx, "nlist_sweep_kernel<count>");
  }
  if ((rc = egnn_launch_row_scan(ctx, row_ptr, n_owned, st))) return rc;
  int32_t total = 0;
  EGNN_HIP(ctx, hipMemcpyAsync(&total, row_ptr + n_owned, sizeof(int32_t), hipMemcpyDeviceToHost, st));
  EGNN_HIP(ctx, hipStreamSynchronize(st));
  if (total < 0) return egnn_fail(ctx, EGNN_EINVAL, "nlist_count: more than 2^31-1 edges");
  *n_edges = total;
  return EGNN_OK;
}

extern "C" int egnn_nlist_fill(egnn_ctx* ctx, const float* pos, int32_t n_owned, int32_t n_total,
                               const float box[3], const uint8_t pbc[3], const int32_t* row_ptr, int64_t n_edges,
                               int32_t* src, int32_t* dst, int8_t* shift, void* ws, size_t ws_bytes, void* stream) {
  if (!ctx) return EGNN_EINVAL;
  NlistGeom g;
  int rc = nlist_geom(ctx, pos, n_owned, n_total, box, pbc, &g);
  if (rc) return rc;
  if (!row_ptr || n_edges < 0 || (n_edges > 0 && (!src || !dst)))
    return egnn_fail(ctx, EGNN_EINVAL, "nlist_fill: null pointer");
  if (ws && ((uintptr_t)ws & 255) != 0) return egnn_fail(ctx, EGNN_EINVAL, "nlist_fill: workspace not 256-byte aligned");
  if (n_owned == 0 || n_edges == 0) return EGNN_OK;
  hipStream_t st = (hipStream_t)stream;
  if (use_cells(ws, ws_bytes, n_total)) {
    // the cells built by egnn_nlist_count, their grid and the sources it found are still in the workspace, laid out for the size it had
    if (ctx->nl_grid_atoms != n_total || ctx->nl_grid_ws != ws || ctx->nl_grid_pos != pos)
      return egnn_fail(ctx, EGNN_EINVAL, "nlist_fill: call egnn_nlist_count with the same atoms and workspace first");
    const CellWs w = carve_cells(ws, ctx->nl_grid_ws_bytes, n_total);
    // (rows of sources lie as the counting pass laid them out: for another number of rows, or where the workspace is now shorter,
    // there are none)
    const int row = ctx->nl_grid_owned == n_owned && ws_bytes >= w.need_kept ? keep_row(w, n_owned, n_total) : 0;
    if (ws_bytes >= w.need) return launch_cells<true>(ctx, pos, n_owned, n_total, g, w, row, const_cast<int*>(row_ptr), src, dst, shift, st);
  }
  hipLaunchKernelGGL(nlist_sweep_kernel<true>, dim3((n_owned + 3) / 4), dim3(256), 0, st, pos, n_owned, n_total, g,
                     const_cast<int*>(row_ptr), src, dst, shift);
  EGNN_LAUNCH_CHECK(ctx, "nlist_sweep_kernel<fill>");
  return EGNN_OK;
}
