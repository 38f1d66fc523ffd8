// Cell-shape diagnostics for gfx950: the Taylor deformation parameter from
// the discretised inertia tensor (Sec. "Taylor deformation parameter", eqs.
// inertia-tensor-discretized, inertia-tensor-ellipsoid-semiaxes and
// taylor-deformation-parameter-definition) and the cell strain (eq.
// cell-strain).
//
//   tile_moments          one wavefront per tile: the current signed volume
//                         V of every tetrahedron and its centroid r, summed
//                         as V, V r and V r r^T (float64) about a per-cell
//                         origin (the cell's first node), one record per tile,
//                         and the tile's count of tetrahedra with V not > 0;
//   cell_search           one workgroup per cell: the largest distance d_max of
//                         two nodes;
//   shape_pass_kernel     both of these, neither of which needs the other;
//   shape_cell_kernel     one wavefront per cell: the tile records summed in a
//                         fixed order, the inertia tensor about the centre of
//                         mass, its eigenvalues by cyclic Jacobi rotations,
//                         semi-axes, D, and the strain; beside them the rest of
//                         the search of cells that left it to more workgroups.
// The farthest two nodes are convex-hull vertices, and a node whose faces are
// all shared by two tetrahedra on opposite sides lies inside the image of its
// star while those keep their orientation (their solid angles at the node sum
// to a positive multiple of 4 pi, so no direction has the node strictly beyond
// all its neighbours): only the other nodes, the candidates, are searched, and
// all nodes of a cell with an inverted tetrahedron.
// Batches with a cell of more than kCellNodes candidates (meshes of some 25,000
// nodes), which the LDS of a workgroup does not hold, are searched block by block over many
// workgroups instead (shape_extreme_kernel, shape_bbox_kernel,
// pair_max_kernel, pair_all_kernel, shape_finalize_kernel, behind
// shape_moments_kernel):
//   shape_extreme_kernel  per cell, the nodes extreme along the three axes and
//                         the four body diagonals; the largest distance among
//                         these pairs is a lower bound L of d_max (the
//                         distance of two actual nodes) and starts the maximum;
//                         and the cell's count of inverted tetrahedra;
//   shape_bbox_kernel     the bounding box of every candidate block of 256
//                         nodes, the nodes of a cell taken candidates
//                         first, each part in Morton order of the reference
//                         positions;
//   pair_max_kernel       the largest squared distance between two candidate
//                         nodes of a cell, over 256 x 256 blocks of node pairs
//                         (float64 differences of the float32 positions are
//                         exact; the maximum of non-negative doubles is an
//                         order-free integer maximum of their bit patterns); a
//                         block pair whose bounding boxes are closer than the
//                         current maximum cannot hold a larger distance and is
//                         skipped (the result is the same, only the work
//                         changes);
//   pair_all_kernel       cells with an inverted tetrahedron: all node pairs;
//   shape_finalize_kernel per cell (one wavefront) the sums and eigenvalues.
// Readings: the tensor is taken about the centre of mass; V is the current
// volume with the reference orientation (negative when inverted); the
// paper's semi-axis formula gives squared semi-axes of a solid ellipsoid, so
// a_i is its square root (0 for a negative radicand); d_ref is the caller's.
#include <hip/hip_runtime.h>

#include <cmath>

#include "device_util.h"
#include "shape.h"

namespace cm {
namespace {

constexpr int kMom = 10;  // V, V r (3), V r r^T (xx yy zz xy xz yz)

struct MomArgs {
  DeviceTables T;
  const int64_t* node_off;
  const float* y;
  double* mom;        // kMom per tile
  int32_t* tile_inv;  // per tile: tetrahedra whose current volume is not > 0
  const uint64_t* chunk_neg;  // per chunk: lanes of negative reference orientation
  int32_t per_block;          // wavefronts (tiles) of a workgroup that have LDS
};

// One tile's record, by one wavefront with ys for the tile's nodes.  Of the
// chunks only the indices are read (8 of every 16 bytes of one row, a third
// of the chunk), two chunks ahead of their use.
constexpr int kMomWaves = 8;  // of the records alone

__device__ __forceinline__ void tile_moments(const MomArgs& a, int t, int lane, float4* ys) {
  const TileDesc d = a.T.tiles[t];
  const int64_t N = a.T.n_nodes;
  const TetChunk* ch = a.T.chunks + d.chunk_begin;
  const uint2 none = make_uint2(kEmptyLane, kEmptyLane);
  uint2 q0 = none, q1 = none;
  if (0 < d.n_chunks) q0 = *reinterpret_cast<const uint2*>(ch[0].a[lane]);
  if (1 < d.n_chunks) q1 = *reinterpret_cast<const uint2*>(ch[1].a[lane]);
  const int64_t o = a.node_off[d.cell];
  for (int l = lane; l < d.n_own + d.n_shr; l += 64) {
    const int64_t g = l < d.n_own ? (int64_t)d.own_begin + l
                                  : (int64_t)a.T.slot_node[d.shr_begin + l - d.n_own];
    ys[l] = make_float4(a.y[g], a.y[N + g], a.y[2 * N + g], 0.f);
  }
  const double ox = a.y[o], oy = a.y[N + o], oz = a.y[2 * N + o];
  wave_sync();
  double m[kMom];
#pragma unroll
  for (int j = 0; j < kMom; ++j) m[j] = 0.0;
  int ninv = 0;
  for (int k = 0; k < d.n_chunks; ++k) {
    const uint64_t neg = a.chunk_neg[d.chunk_begin + k];  // wave-uniform
    const uint2 c = q0;
    q0 = q1;
    if (k + 2 < d.n_chunks) q1 = *reinterpret_cast<const uint2*>(ch[k + 2].a[lane]);
    if (c.x == kEmptyLane) continue;
    const float4 p[4] = {ys[c.x & 0xffff], ys[c.x >> 16], ys[c.y & 0xffff],
                         ys[c.y >> 16]};
    double e[3][3];
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      e[v][0] = (double)p[v].x - (double)p[3].x;
      e[v][1] = (double)p[v].y - (double)p[3].y;
      e[v][2] = (double)p[v].z - (double)p[3].z;
    }
    const double det_s = e[0][0] * (e[1][1] * e[2][2] - e[1][2] * e[2][1]) -
                         e[0][1] * (e[1][0] * e[2][2] - e[1][2] * e[2][0]) +
                         e[0][2] * (e[1][0] * e[2][1] - e[1][1] * e[2][0]);
    // current volume with the orientation of the reference vertex order (the
    // sign of the reference edges' determinant for the stored vertex order)
    const double V = (((neg >> lane) & 1ull) ? -det_s : det_s) * (1.0 / 6.0);
    ninv += V > 0.0 ? 0 : 1;
    const double rx = 0.25 * (((double)p[0].x + (double)p[1].x) +
                              ((double)p[2].x + (double)p[3].x)) - ox;
    const double ry = 0.25 * (((double)p[0].y + (double)p[1].y) +
                              ((double)p[2].y + (double)p[3].y)) - oy;
    const double rz = 0.25 * (((double)p[0].z + (double)p[1].z) +
                              ((double)p[2].z + (double)p[3].z)) - oz;
    m[0] += V;
    m[1] += V * rx; m[2] += V * ry; m[3] += V * rz;
    m[4] += V * rx * rx; m[5] += V * ry * ry; m[6] += V * rz * rz;
    m[7] += V * rx * ry; m[8] += V * rx * rz; m[9] += V * ry * rz;
  }
#pragma unroll
  for (int j = 0; j < kMom; ++j) m[j] = wave_sum(m[j]);
  ninv = wave_sum(ninv);
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < kMom; ++j) a.mom[(int64_t)kMom * t + j] = m[j];
    a.tile_inv[t] = ninv;
  }
}

__global__ __launch_bounds__(64 * kMomWaves) void shape_moments_kernel(MomArgs a) {
  extern __shared__ float4 ys[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t t = (int64_t)blockIdx.x * a.per_block + wave;
  if (wave < a.per_block && t < a.T.n_tiles)
    tile_moments(a, (int)t, lane, ys + (size_t)wave * a.T.nloc);
}

struct PairArgs {
  const int4* blocks;  // (cell, row block, column block, first node block of the cell)
  const int64_t* node_off;
  const int32_t* order;  // per cell, node ids in spatial (Morton) order
  const float* y;
  int64_t N;
  const double* bbox;         // per node block: min x y z, max x y z
  unsigned long long* d2max;  // per cell, bits of a non-negative double
};

struct AllArgs {
  const int64_t* node_off;
  const float* y;
  int64_t N;
  const int32_t* cell_inv;
  unsigned long long* d2max;
};

// Largest squared distance over all node pairs of [n0, n1), this thread's part
// of a workgroup's 256.
__device__ __forceinline__ double all_pairs(const float* y, int64_t N, int64_t n0,
                                            int64_t n1) {
  double best = 0.0;
  for (int64_t p = n0 + threadIdx.x; p < n1; p += 256) {
    const double xp = y[p], yp = y[N + p], zp = y[2 * N + p];
    for (int64_t q = p + 1; q < n1; ++q) {
      const double dx = xp - y[q], dy = yp - y[N + q], dz = zp - y[2 * N + q];
      best = fmax(best, dx * dx + dy * dy + dz * dz);
    }
  }
  return best;
}

// Cells with an inverted (or degenerate) tetrahedron, which the candidate
// search does not cover: one workgroup per such cell takes the largest
// squared distance over all its node pairs (other cells return at once).
__global__ __launch_bounds__(256) void pair_all_kernel(AllArgs a) {
  __shared__ double red[4];
  const int c = blockIdx.x, tid = threadIdx.x;
  if (a.cell_inv[c] == 0) return;  // uniform over the workgroup
  const double best = wave_max(all_pairs(a.y, a.N, a.node_off[c], a.node_off[c + 1]));
  if ((tid & 63) == 0) red[tid >> 6] = best;
  __syncthreads();
  if (tid == 0) {
    const double m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    atomicMax(&a.d2max[c], (unsigned long long)__double_as_longlong(m));
  }
}

// Directions of the extreme-node search: the axes and the body diagonals.
__constant__ float kDirs[7][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}, {1, 1, 1},
                                  {1, 1, -1}, {1, -1, 1}, {-1, 1, 1}};

struct ExtArgs {
  DeviceTables T;
  const int64_t* node_off;
  const float* y;
  int64_t N;
  unsigned long long* d2max;
  const int32_t* tile_inv;
  int32_t* cell_inv;  // per cell: tetrahedra whose current volume is not > 0
};

// Per cell: for every direction the node of smallest and of largest
// projection (ties to the smaller index), then d2max = the largest squared
// distance among those pairs; and the cell's count of tetrahedra that are
// inverted (or degenerate) in the current positions.  One pass over the
// nodes: every thread keeps the 14 extremes of its nodes (a largest
// projection as the smallest negated one), then a (value, index)
// lexicographic minimum over the wavefront (butterfly) and the 4 wavefronts.
__global__ __launch_bounds__(256) void shape_extreme_kernel(ExtArgs a) {
  __shared__ double wv[4][14];
  __shared__ int wi[4][14];
  __shared__ int inv[4];
  const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t n0 = a.node_off[c], n1 = a.node_off[c + 1], N = a.N;
  {
    int s = 0;
    const int t0 = a.T.cell_tile_first[c], nt = a.T.cell_tile_count[c];
    for (int k = tid; k < nt; k += 256) s += a.tile_inv[t0 + (int64_t)k * a.T.tile_stride];
    s = wave_sum(s);
    if (lane == 0) inv[w] = s;
  }
  double best[14];
  int arg[14];
#pragma unroll
  for (int k = 0; k < 14; ++k) {
    best[k] = INFINITY;
    arg[k] = -1;
  }
  for (int64_t i = n0 + tid; i < n1; i += 256) {
    const double px = a.y[i], py = a.y[N + i], pz = a.y[2 * N + i];
    const int li = (int)(i - n0);
#pragma unroll
    for (int d = 0; d < 7; ++d) {
      const double pr = (double)kDirs[d][0] * px + (double)kDirs[d][1] * py +
                        (double)kDirs[d][2] * pz;
      // indices grow along a thread's nodes: strict < keeps the smaller one
      if (pr < best[2 * d]) { best[2 * d] = pr; arg[2 * d] = li; }
      if (-pr < best[2 * d + 1]) { best[2 * d + 1] = -pr; arg[2 * d + 1] = li; }
    }
  }
#pragma unroll
  for (int k = 0; k < 14; ++k) {
    double v = best[k];
    int ix = arg[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double v2 = __shfl_xor(v, off);
      const int i2 = __shfl_xor(ix, off);
      if (i2 >= 0 && (ix < 0 || v2 < v || (v2 == v && i2 < ix))) { v = v2; ix = i2; }
    }
    if (lane == 0) { wv[w][k] = v; wi[w][k] = ix; }
  }
  __syncthreads();
  if (tid == 0) {
    a.cell_inv[c] = inv[0] + inv[1] + inv[2] + inv[3];
    int ext[14];
    for (int k = 0; k < 14; ++k) {
      double v = wv[0][k];
      int ix = wi[0][k];
      for (int q = 1; q < 4; ++q) {
        const double v2 = wv[q][k];
        const int i2 = wi[q][k];
        if (i2 >= 0 && (ix < 0 || v2 < v || (v2 == v && i2 < ix))) { v = v2; ix = i2; }
      }
      ext[k] = ix;
    }
    double m = 0.0;
    for (int d = 0; d < 7; ++d) {
      if (ext[2 * d] < 0 || ext[2 * d + 1] < 0) continue;
      const int64_t p = n0 + ext[2 * d], q = n0 + ext[2 * d + 1];
      const double dx = (double)a.y[p] - a.y[q], dy = (double)a.y[N + p] - a.y[N + q],
                   dz = (double)a.y[2 * N + p] - a.y[2 * N + q];
      m = fmax(m, dx * dx + dy * dy + dz * dz);
    }
    a.d2max[c] = (unsigned long long)__double_as_longlong(m);
  }
}

struct BoxArgs {
  const int2* node_blocks;  // (cell, block of the cell)
  const int64_t* node_off;
  const int32_t* order;
  const float* y;
  int64_t N;
  double* bbox;
};

__global__ __launch_bounds__(256) void shape_bbox_kernel(BoxArgs a) {
  __shared__ double red[6][4];
  const int2 nb = a.node_blocks[blockIdx.x];
  const int64_t n1 = a.node_off[nb.x + 1];
  const int64_t i = a.node_off[nb.x] + (int64_t)nb.y * 256 + threadIdx.x;
  const bool in = i < n1;
  const int64_t g = in ? (int64_t)a.order[i] : 0;
  double v[6];
  for (int d = 0; d < 3; ++d) {
    const double q = in ? (double)a.y[d * a.N + g] : 0.0;
    v[d] = in ? q : INFINITY;
    v[3 + d] = in ? q : -INFINITY;
  }
  for (int off = 32; off > 0; off >>= 1)
    for (int d = 0; d < 3; ++d) {
      v[d] = fmin(v[d], __shfl_xor(v[d], off));
      v[3 + d] = fmax(v[3 + d], __shfl_xor(v[3 + d], off));
    }
  if ((threadIdx.x & 63) == 0)
    for (int k = 0; k < 6; ++k) red[k][threadIdx.x >> 6] = v[k];
  __syncthreads();
  if (threadIdx.x < 6) {
    const int k = threadIdx.x;
    const double r = k < 3 ? fmin(fmin(red[k][0], red[k][1]), fmin(red[k][2], red[k][3]))
                           : fmax(fmax(red[k][0], red[k][1]), fmax(red[k][2], red[k][3]));
    a.bbox[6 * (int64_t)blockIdx.x + k] = r;
  }
}

__global__ __launch_bounds__(256) void pair_max_kernel(PairArgs a) {
  __shared__ double cx[256], cy[256], cz[256];
  __shared__ double red[4];
  __shared__ int skip;
  __shared__ double cur_d2;
  const int4 b = a.blocks[blockIdx.x];
  const int tid = threadIdx.x;
  if (tid == 0) {
    // farthest points of the two bounding boxes vs the current maximum
    const double* r = a.bbox + 6 * (int64_t)(b.w + b.y);
    const double* q = a.bbox + 6 * (int64_t)(b.w + b.z);
    double u = 0.0;
    for (int d = 0; d < 3; ++d) {
      const double e = fmax(r[3 + d] - q[d], q[3 + d] - r[d]);
      u += e * e;
    }
    const unsigned long long cur = __hip_atomic_load(&a.d2max[b.x], __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
    cur_d2 = __longlong_as_double((long long)cur);
    // (with a relative margin far above the rounding of the two sums)
    skip = u < cur_d2 * (1.0 - 1e-12);
  }
  __syncthreads();
  if (skip) return;  // uniform over the workgroup
  const int64_t n0 = a.node_off[b.x], n1 = a.node_off[b.x + 1];
  const int64_t j0 = n0 + (int64_t)b.z * 256;
  const int ncol = n1 - j0 < 256 ? (int)(n1 - j0) : 256;
  if (tid < ncol) {
    const int64_t g = a.order[j0 + tid];
    cx[tid] = a.y[g];
    cy[tid] = a.y[a.N + g];
    cz[tid] = a.y[2 * a.N + g];
  }
  __syncthreads();
  const int64_t i = n0 + (int64_t)b.y * 256 + tid;
  double best = 0.0;
  if (i < n1) {
    const int64_t g = a.order[i];
    const double xi = a.y[g], yi = a.y[a.N + g], zi = a.y[2 * a.N + g];
    // the column block's box cannot hold a node farther from this one than
    // the current maximum: nothing to find for this row
    const double* q = a.bbox + 6 * (int64_t)(b.w + b.z);
    const double ex = fmax(xi - q[0], q[3] - xi), ey = fmax(yi - q[1], q[4] - yi),
                 ez = fmax(zi - q[2], q[5] - zi);
    const int ncheck = ex * ex + ey * ey + ez * ez < cur_d2 * (1.0 - 1e-12) ? 0 : ncol;
    for (int k = 0; k < ncheck; ++k) {
      const double dx = xi - cx[k], dy = yi - cy[k], dz = zi - cz[k];
      best = fmax(best, dx * dx + dy * dy + dz * dz);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) best = fmax(best, __shfl_xor(best, off));
  if ((tid & 63) == 0) red[tid >> 6] = best;
  __syncthreads();
  if (tid == 0) {
    const double m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    atomicMax(&a.d2max[b.x], (unsigned long long)__double_as_longlong(m));
  }
}

// Eigenvalues of a symmetric 3x3 matrix (A00 A11 A22 A01 A02 A12) by cyclic
// Jacobi rotations; at most 32 sweeps (convergence is quadratic).
__device__ void sym3_eigenvalues(const double s[6], double ev[3]) {
  double A[3][3] = {{s[0], s[3], s[4]}, {s[3], s[1], s[5]}, {s[4], s[5], s[2]}};
  for (int sweep = 0; sweep < 32; ++sweep) {
    const double off = A[0][1] * A[0][1] + A[0][2] * A[0][2] + A[1][2] * A[1][2];
    const double dia = A[0][0] * A[0][0] + A[1][1] * A[1][1] + A[2][2] * A[2][2];
    if (off <= 1e-32 * dia || off == 0.0) break;
    for (int p = 0; p < 2; ++p)
      for (int q = p + 1; q < 3; ++q) {
        if (A[p][q] == 0.0) continue;
        const double tau = (A[q][q] - A[p][p]) / (2.0 * A[p][q]);
        const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
        const double c = 1.0 / sqrt(1.0 + tt * tt), sn = tt * c;
        for (int k = 0; k < 3; ++k) {  // A <- A G (columns p, q)
          const double akp = A[k][p], akq = A[k][q];
          A[k][p] = c * akp - sn * akq;
          A[k][q] = sn * akp + c * akq;
        }
        for (int k = 0; k < 3; ++k) {  // A <- G^T A (rows p, q)
          const double apk = A[p][k], aqk = A[q][k];
          A[p][k] = c * apk - sn * aqk;
          A[q][k] = sn * apk + c * aqk;
        }
        A[p][q] = A[q][p] = 0.0;
      }
  }
  ev[0] = A[0][0]; ev[1] = A[1][1]; ev[2] = A[2][2];
}

struct ShapeFinArgs {
  DeviceTables T;
  const int64_t* node_off;
  const float* y;
  const double* mom;
  const unsigned long long* d2max;
  const double* d_ref;  // nullable
  double* out;          // kShapeFields per cell
};

// The fields of cell c but d_max and the strain, on one wavefront: lane l sums
// the tile records l, l + 64, ..., then a fixed butterfly; lane 0 finishes the
// cell.
__device__ void shape_fields(const ShapeFinArgs& a, int c, int lane) {
  double m[kMom];
#pragma unroll
  for (int j = 0; j < kMom; ++j) m[j] = 0.0;
  const int t0 = a.T.cell_tile_first[c], nt = a.T.cell_tile_count[c];
  for (int k = lane; k < nt; k += 64) {
    const int64_t t = t0 + (int64_t)k * a.T.tile_stride;
#pragma unroll
    for (int j = 0; j < kMom; ++j) m[j] += a.mom[kMom * t + j];
  }
#pragma unroll
  for (int j = 0; j < kMom; ++j) m[j] = wave_sum(m[j]);
  if (lane != 0) return;
  const int64_t N = a.T.n_nodes, o = a.node_off[c];
  const double M = m[0];
  const double cx = m[1] / M, cy = m[2] / M, cz = m[3] / M;
  // second moments about the centre of mass, then the inertia tensor
  const double Sxx = m[4] - m[1] * cx, Syy = m[5] - m[2] * cy, Szz = m[6] - m[3] * cz;
  const double Sxy = m[7] - m[1] * cy, Sxz = m[8] - m[1] * cz, Syz = m[9] - m[2] * cz;
  const double tr = Sxx + Syy + Szz;
  const double I[6] = {tr - Sxx, tr - Syy, tr - Szz, -Sxy, -Sxz, -Syz};
  double th[3];
  sym3_eigenvalues(I, th);
  // theta_1 >= theta_2 >= theta_3
  if (th[0] < th[1]) { const double s = th[0]; th[0] = th[1]; th[1] = s; }
  if (th[1] < th[2]) { const double s = th[1]; th[1] = th[2]; th[2] = s; }
  if (th[0] < th[1]) { const double s = th[0]; th[0] = th[1]; th[1] = s; }
  const double f = 5.0 / (2.0 * M);
  const double a1 = sqrt(fmax(f * (-th[0] + th[1] + th[2]), 0.0));
  const double a2 = sqrt(fmax(f * (th[0] - th[1] + th[2]), 0.0));
  const double a3 = sqrt(fmax(f * (th[0] + th[1] - th[2]), 0.0));
  double* r = a.out + (int64_t)kShapeFields * c;
  r[0] = M;
  r[1] = (double)a.y[o] + cx;
  r[2] = (double)a.y[N + o] + cy;
  r[3] = (double)a.y[2 * N + o] + cz;
  r[4] = a1; r[5] = a2; r[6] = a3;
  r[7] = (a3 - a1) / (a3 + a1);
}

__device__ __forceinline__ void shape_distance(const ShapeFinArgs& a, int c, double d2) {
  const double dmax = sqrt(d2);
  double* r = a.out + (int64_t)kShapeFields * c;
  r[8] = dmax;
  r[9] = a.d_ref ? (dmax - a.d_ref[c]) / a.d_ref[c] : __builtin_nan("");
}

__global__ __launch_bounds__(256) void shape_finalize_kernel(ShapeFinArgs a) {
  const int c = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (c >= a.T.n_cells) return;  // uniform per wavefront
  shape_fields(a, c, lane);
  if (lane == 0) shape_distance(a, c, __longlong_as_double((long long)a.d2max[c]));
}

// ------------------------------------------------- one workgroup per cell
__device__ __forceinline__ double dist2(double dx, double dy, double dz) {
  return dx * dx + dy * dy + dz * dz;
}

constexpr int kGroup = 16;  // nodes that share a bounding box

struct CellArgs {
  MomArgs mom;
  const int32_t* order;       // per cell, node ids, candidates first
  const int32_t* candidates;  // per cell: how many of them are candidates
  unsigned long long* d2max;
  int32_t cap;                // nodes that the LDS holds (multiple of 64)
  const int32_t* helpers;     // these as in ShapeTables
  const int2* helper;
  SearchRest* rest;           // null: no helpers
};

// Largest value over the workgroup (v >= 0) on every thread, and one of the
// places it was found at.
template <int W>
__device__ __forceinline__ void cell_argmax(double& v, int& i, double* rv, int* ri) {
  const double m = wave_max(v);
  const int first = __ffsll((long long)__ballot(v == m)) - 1;
  i = __shfl(i, first);
  if ((threadIdx.x & 63) == 0) { rv[threadIdx.x >> 6] = m; ri[threadIdx.x >> 6] = i; }
  __syncthreads();
  v = rv[0];
  i = ri[0];
#pragma unroll
  for (int w = 1; w < W; ++w)
    if (rv[w] > v) { v = rv[w]; i = ri[w]; }
  __syncthreads();  // rv, ri are used again
}

struct Min { __device__ float operator()(float a, float b) const { return fminf(a, b); } };
struct Max { __device__ float operator()(float a, float b) const { return fmaxf(a, b); } };

// The largest squared distance of two candidates of a cell.  The candidates'
// positions are kept in LDS.  From the node farthest from the centre of their box
// (at distance R), three steps to the node farthest from the last one give a pair
// whose distance L is a lower bound of d_max, mostly d_max itself.  A node nearer
// to the centre than L - R has no partner at L or more: the others, in order, are
// what remains (a few at the tips of an elongated cell, a ring of a flat one, all
// of a sphere).  They are compact in groups of 16 (Morton order), each with its
// bounding box: a wavefront takes 64 of them, one per lane, and goes over a group
// only if the boxes, and then some lane's node and the box, could be farther
// apart than the largest distance so far.  All tests keep a relative margin of
// 1e-12 against the rounding of the sums, so the result is that of all pairs.

// The candidates of cell c into LDS (no barrier); this thread's part of their box.
template <int W>
__device__ __forceinline__ void load_candidates(const CellArgs& a, int c, float* sx,
                                                float (&lo)[3], float (&hi)[3]) {
  const float* y = a.mom.y;
  const int tid = threadIdx.x;
  const int64_t n0 = a.mom.node_off[c], N = a.mom.T.n_nodes;
  const int ns = a.candidates[c];
  float *sy = sx + a.cap, *sz = sy + a.cap;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lo[d] = INFINITY;
    hi[d] = -INFINITY;
  }
  for (int b = 0; b < ns; b += 4 * 64 * W) {  // four gathers in flight
    int64_t g[4];
    float p[4][3];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      g[u] = a.order[n0 + min(b + u * 64 * W + tid, ns - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      p[u][0] = y[g[u]];
      p[u][1] = y[N + g[u]];
      p[u][2] = y[2 * N + g[u]];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        lo[d] = fminf(lo[d], p[u][d]);
        hi[d] = fmaxf(hi[d], p[u][d]);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = b + u * 64 * W + tid;
      if (i < ns) { sx[i] = p[u][0]; sy[i] = p[u][1]; sz[i] = p[u][2]; }
    }
  }
}

// The nodes at least sqrt(least2) from (cx, cy, cz), in place and in order; how
// many they are.  ri: W ints of LDS.
template <int W>
__device__ __forceinline__ int keep_far_nodes(const CellArgs& a, int ns, float* sx, double cx,
                                              double cy, double cz, double least2, int* ri) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float *sy = sx + a.cap, *sz = sy + a.cap;
  int kept = 0;
  for (int b = 0; b < ns; b += 64 * W) {
    const int k = b + tid;
    float x = 0.f, yk = 0.f, z = 0.f;
    bool keep = false;
    if (k < ns) {
      x = sx[k]; yk = sy[k]; z = sz[k];
      keep = !(dist2(x - cx, yk - cy, z - cz) < least2);
    }
    const unsigned long long m = __ballot(keep);
    if (lane == 0) ri[wave] = __popcll(m);
    __syncthreads();  // (all positions of this round are in registers)
    int at = kept;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      if (w < wave) at += ri[w];
      kept += ri[w];
    }
    if (keep) {
      at += __popcll(m & ((1ull << lane) - 1));
      sx[at] = x; sy[at] = yk; sz[at] = z;
    }
    __syncthreads();  // ri is used again
  }
  return kept;
}

// The largest squared distance of two of the `kept` nodes into *best_bits (LDS),
// from L2 on: of the blocks of 64 rows against 16 column groups, every `stride`-th
// from first + wave on.  Called by all threads; ends with a barrier.
template <int W>
__device__ __forceinline__ void search_pairs(const CellArgs& a, float* sx, int kept, double L2,
                                             int first, int stride,
                                             unsigned long long* best_bits) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float *sy = sx + a.cap, *sz = sy + a.cap, *box = sz + a.cap;
  // the last 64 are filled up with the last node, then the boxes
  const int blocks = (kept + 63) / 64;
  for (int b = wave; b < blocks; b += W) {
    const int k = 64 * b + lane, from = min(k, kept - 1);
    const float v[3] = {sx[from], sy[from], sz[from]};
    wave_sync();
    if (k >= kept) { sx[k] = v[0]; sy[k] = v[1]; sz[k] = v[2]; }
    float* to = box + 6 * (k / kGroup);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const float lo = row_reduce(v[d], Min()), hi = row_reduce(v[d], Max());
      if ((lane & 15) == 0) { to[d] = lo; to[3 + d] = hi; }
    }
  }
  if (tid == 0) *best_bits = (unsigned long long)__double_as_longlong(L2);
  __syncthreads();
  double best = L2;  // per lane
  constexpr int kRows = 64 / kGroup;  // groups of a block's rows
  const int groups = blocks * kRows;
  int turn = 0;
  for (int g = 0; g < blocks; ++g)
    for (int h0 = g * kRows; h0 < groups; h0 += kGroup) {
      const bool mine = turn == first + wave;
      turn = turn + 1 == stride ? 0 : turn + 1;
      if (!mine) continue;
      const double best0 = __longlong_as_double((long long)__hip_atomic_load(
          best_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
      best = fmax(best, best0);
      // a lane per pair of a row group and a column group
      bool near = false;
      if (h0 + (lane & 15) < groups) {
        const float* r = box + 6 * (g * kRows + (lane >> 4));
        const float* q = box + 6 * (h0 + (lane & 15));
        const double ex = fmax((double)r[3] - q[0], (double)q[3] - r[0]),
                     ey = fmax((double)r[4] - q[1], (double)q[4] - r[1]),
                     ez = fmax((double)r[5] - q[2], (double)q[5] - r[2]);
        near = !(dist2(ex, ey, ez) < best0 * (1.0 - 1e-12));
      }
      const unsigned long long m = __ballot(near);
      const double x = sx[64 * g + lane], yk = sy[64 * g + lane], z = sz[64 * g + lane];
      for (uint32_t todo = (uint32_t)(m | m >> 16 | m >> 32 | m >> 48) & 0xffffu; todo != 0;
           todo &= todo - 1) {
        const int h = h0 + __ffs((int)todo) - 1;
        const float* q = box + 6 * h;
        const double ex = fmax(x - q[0], q[3] - x), ey = fmax(yk - q[1], q[4] - yk),
                     ez = fmax(z - q[2], q[5] - z);
        if (__ballot(!(dist2(ex, ey, ez) < best * (1.0 - 1e-12))) == 0) continue;
        const float4* vx = reinterpret_cast<const float4*>(sx + kGroup * h);
        const float4* vy = reinterpret_cast<const float4*>(sy + kGroup * h);
        const float4* vz = reinterpret_cast<const float4*>(sz + kGroup * h);
#pragma unroll
        for (int j = 0; j < kGroup / 4; ++j) {
          const float4 u = vx[j], v = vy[j], w = vz[j];
          best = fmax(best, dist2(x - u.x, yk - v.x, z - w.x));
          best = fmax(best, dist2(x - u.y, yk - v.y, z - w.y));
          best = fmax(best, dist2(x - u.z, yk - v.z, z - w.z));
          best = fmax(best, dist2(x - u.w, yk - v.w, z - w.w));
        }
      }
      // the maximum of non-negative doubles is that of their bit patterns
      if (__ballot(best > best0) != 0) {
        best = wave_max(best);
        if (lane == 0)
          atomicMax(best_bits, (unsigned long long)__double_as_longlong(best));
      }
    }
  __syncthreads();
}

// The search of cell c by one workgroup; where too many nodes remain for it
// (search_helpers, shape.h), only up to them: a.rest is for the helpers.
template <int W>
__device__ __forceinline__ void cell_search(const CellArgs& a, int c, float* sx) {
  __shared__ double rv[W];
  __shared__ int ri[W];
  __shared__ float rb[W][6];
  __shared__ unsigned long long best_bits;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ns = a.candidates[c];
  float *sy = sx + a.cap, *sz = sy + a.cap;
  float lo[3], hi[3];
  load_candidates<W>(a, c, sx, lo, hi);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float l = wave_reduce(lo[d], Min()), h = wave_reduce(hi[d], Max());
    if (lane == 0) { rb[wave][d] = l; rb[wave][3 + d] = h; }
  }
  __syncthreads();
  double ctr[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    float l = rb[0][d], h = rb[0][3 + d];
#pragma unroll
    for (int w = 1; w < W; ++w) {
      l = fminf(l, rb[w][d]);
      h = fmaxf(h, rb[w][3 + d]);
    }
    ctr[d] = 0.5 * ((double)l + (double)h);
  }
  // farthest from the centre, then from the node found last
  const double cx = ctr[0], cy = ctr[1], cz = ctr[2];
  double px = cx, py = cy, pz = cz, R2 = 0.0, L2 = 0.0;
  for (int step = 0; step < 4; ++step) {
    double v = 0.0;
    int i = 0;
    for (int k = tid; k < ns; k += 64 * W) {
      const double d2 = dist2(px - sx[k], py - sy[k], pz - sz[k]);
      if (d2 > v) { v = d2; i = k; }
    }
    cell_argmax<W>(v, i, rv, ri);
    if (step == 0) {
      R2 = v;
    } else {
      if (!(v > L2)) break;  // uniform: the last pair is mutually farthest
      L2 = v;
    }
    px = sx[i]; py = sy[i]; pz = sz[i];
  }
  // the nodes that remain, in place and in order (all of them if L - R is not
  // positive, or no number)
  const double gap = sqrt(L2) * (1.0 - 1e-12) - sqrt(R2) * (1.0 + 1e-12);
  const double least2 = gap > 0.0 ? gap * gap * (1.0 - 1e-12) : 0.0;
  const int kept = keep_far_nodes<W>(a, ns, sx, cx, cy, cz, least2, ri);
  if (a.rest) {
    const int helpers = a.helpers[c];
    if (helpers > 0 && kept > max(kSearchNodes, ns / 8)) {
      if (tid == 0) {
        a.rest[c] = SearchRest{{cx, cy, cz}, least2, helpers, 0};
        a.d2max[c] = (unsigned long long)__double_as_longlong(L2);
      }
      return;
    }
  }
  search_pairs<W>(a, sx, kept, L2, 0, W, &best_bits);
  if (tid == 0) {
    a.d2max[c] = best_bits;
    if (a.rest) a.rest[c].left = 0;
  }
}

// The searches, one workgroup per cell, and behind them in the same launch the
// tile records, a wavefront per tile.  Both are bound by their chains of
// dependent loads, which overlap here; six launches in a row before (records,
// extreme nodes, boxes, pairs of blocks of 256, all pairs of inverted cells,
// fields).  512 cells of 1,000 to 9,000 nodes, 5 M tets: 131 -> 38 us for
// cm_shape, of which 29 here and 9 in shape_cell_kernel (its eigenvalues are a
// chain of divisions and square roots); 64 cells of 20,000 nodes 200 -> 42, one
// of 1,000 nodes 43 -> 13; 1,024 equal spheres of 2,000 nodes, where every
// candidate remains, 189 -> 123.
template <int W>
__global__ __launch_bounds__(64 * W) void shape_pass_kernel(CellArgs a) {
  extern __shared__ float4 lds[];
  const int nc = a.mom.T.n_cells;
  if ((int)blockIdx.x < nc) {
    cell_search<W>(a, blockIdx.x, reinterpret_cast<float*>(lds));
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t t = (int64_t)((int)blockIdx.x - nc) * a.mom.per_block + wave;
  if (wave < a.mom.per_block && t < a.mom.T.n_tiles)
    tile_moments(a.mom, (int)t, lane, lds + (size_t)wave * a.mom.T.nloc);
}

constexpr int kFieldWaves = 4;

// Whether a tetrahedron of cell c is not positively oriented: this thread's part.
__device__ __forceinline__ int cell_inverted(const ShapeFinArgs& f, const int32_t* tile_inv,
                                             int c, int tid) {
  int inv = 0;
  const int t0 = f.T.cell_tile_first[c], nt = f.T.cell_tile_count[c];
  for (int k = tid; k < nt; k += 64 * kFieldWaves)
    inv |= tile_inv[t0 + (int64_t)k * f.T.tile_stride];
  return inv;
}

// A helper of cell c: it loads the candidates again, keeps the same nodes and takes
// its share of their pairs; with LAST, the last of the cell's helpers to arrive
// writes the distance.

template <bool LAST>
__device__ __forceinline__ void help_search(const ShapeFinArgs& f, const CellArgs& a, int c,
                                            int helper, float* sx) {
  __shared__ int ri[kFieldWaves], flag;
  __shared__ unsigned long long best_bits, start_bits;
  const SearchRest r = a.rest[c];  // (but its counter)
  if (r.left == 0) return;
  const int tid = threadIdx.x;
  if (tid == 0) start_bits = device_load(a.d2max + c);  // the others raise it
  float lo[3], hi[3];
  load_candidates<kFieldWaves>(a, c, sx, lo, hi);
  __syncthreads();
  const int kept = keep_far_nodes<kFieldWaves>(a, a.candidates[c], sx, r.centre[0], r.centre[1],
                                               r.centre[2], r.least2, ri);
  const unsigned long long start = start_bits;
  search_pairs<kFieldWaves>(a, sx, kept, __longlong_as_double((long long)start),
                            kFieldWaves * helper, kFieldWaves * r.left, &best_bits);
  if (tid == 0 && best_bits > start) atomicMax(a.d2max + c, best_bits);
  if constexpr (LAST) {
    if (!last_arrival(&a.rest[c].done, r.left - 1, tid, &flag)) return;
    // (a cell with an inverted tetrahedron: all its pairs were compared elsewhere)
    if (!__syncthreads_or(cell_inverted(f, a.mom.tile_inv, c, tid)) && tid == 0)
      shape_distance(f, c, __longlong_as_double((long long)device_load(a.d2max + c)));
  }
}

// The helpers in a launch of their own.
__global__ __launch_bounds__(64 * kFieldWaves) void shape_help_kernel(ShapeFinArgs f,
                                                                      CellArgs a) {
  extern __shared__ float4 lds[];
  const int2 w = a.helper[blockIdx.x];
  help_search<false>(f, a, w.x, w.y, reinterpret_cast<float*>(lds));
}

// The cell's fields, by one wavefront; all four search all node pairs first if
// the cell has a tetrahedron that is not positively oriented, which the
// candidates do not cover.  HELP: behind the cells' workgroups, the helpers of
// each, which write the distance of a cell whose search was left to them, unless
// all its pairs are compared here.
template <bool HELP>
__global__ __launch_bounds__(64 * kFieldWaves) void shape_cell_kernel(ShapeFinArgs f,
                                                                      const int32_t* tile_inv,
                                                                      CellArgs a) {
  extern __shared__ float4 lds[];
  __shared__ double rv[kFieldWaves];
  const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  if (!HELP || c < f.T.n_cells) {
    const int inv = cell_inverted(f, tile_inv, c, tid);
    // (the helpers raise d2max meanwhile)
    const bool left = HELP && a.rest[c].left != 0;
    double d2 = left ? 0.0 : __longlong_as_double((long long)f.d2max[c]);
    const bool all = __syncthreads_or(inv != 0);
    if (all) {
      const double m = wave_max(all_pairs(f.y, f.T.n_nodes, f.node_off[c], f.node_off[c + 1]));
      if (lane == 0) rv[tid >> 6] = m;
      __syncthreads();
      d2 = fmax(fmax(d2, fmax(rv[0], rv[1])), fmax(rv[2], rv[3]));
    }
    if (tid >= 64) return;
    shape_fields(f, c, lane);
    if (lane == 0 && (!left || all)) shape_distance(f, c, d2);
    return;
  }
  if constexpr (HELP) {
    const int2 w = a.helper[c - f.T.n_cells];
    help_search<true>(f, a, w.x, w.y, reinterpret_cast<float*>(lds));
  }
}

}  // namespace

size_t shape_lds(int nloc) { return (size_t)16 * nloc; }

// LDS of the search of one workgroup per cell, for cap nodes: positions, boxes.
static size_t cell_lds(int cap) { return (size_t)12 * cap + (size_t)24 * (cap / kGroup); }

hipError_t launch_shape(const DeviceTables& T, const int64_t* node_off,
                        const ShapeTables& S, const float* y, const double* d_ref,
                        double* out, hipStream_t st) {
  const int nc = T.n_cells;
  hipError_t e;
  // Wavefronts of a workgroup: four unless the search takes more than 32 KB of
  // LDS (2,300 candidates), which the records' workgroups beside it are given
  // too; then eight fill a CU better.  Eight -> four: 512 uneven cells of up to
  // 2,140 candidates 40.7 -> 38.2 us, 1,024 cells of 2,000 nodes 61.5 -> 54.6; 64
  // cells of 3,670 candidates 41.5 -> 47.0.
  const int waves = S.cell_nodes > 0 && cell_lds(S.cell_nodes) <= 32768 ? 4 : kMomWaves;
  // (the caller checks that one tile fits 64 KB; a workgroup takes as many tiles
  // as do)
  const int per =
      std::min(waves, std::max(1, (int)(65536 / std::max<size_t>(shape_lds(T.nloc), 1))));
  const MomArgs m{T, node_off, y, S.mom, S.tile_inv, S.chunk_neg, per};
  const unsigned mom_blocks = (unsigned)((T.n_tiles + per - 1) / per);
  const size_t mom_lds = per * shape_lds(T.nloc);
  const ShapeFinArgs f{T, node_off, y, S.mom, S.d2max, d_ref, out};
  if (S.cell_nodes > 0) {
    const CellArgs a{m, S.order, S.candidates, S.d2max, S.cell_nodes, S.helpers,
                     S.helper, S.rest};
    const size_t lds = std::max(mom_lds, cell_lds(S.cell_nodes));
    if (waves == 4)
      hipLaunchKernelGGL(shape_pass_kernel<4>, dim3(nc + mom_blocks), dim3(256), lds, st, a);
    else
      hipLaunchKernelGGL(shape_pass_kernel<kMomWaves>, dim3(nc + mom_blocks),
                         dim3(64 * kMomWaves), lds, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // The helpers beside the cells' workgroups cost no launch (1.5 to 2 us), but give
    // all of those the LDS of the search: only if they fit the chip with it at once.
    const int help = S.n_helpers;
    const size_t search = cell_lds(S.cell_nodes);
    if (help > 0 && nc <= 256 * (int)(163840 / (search + 512))) {
      hipLaunchKernelGGL(shape_cell_kernel<true>, dim3(nc + help), dim3(64 * kFieldWaves),
                         search, st, f, (const int32_t*)S.tile_inv, a);
      return hipGetLastError();
    }
    if (help > 0) {
      hipLaunchKernelGGL(shape_help_kernel, dim3(help), dim3(64 * kFieldWaves), search, st,
                         f, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(shape_cell_kernel<false>, dim3(nc), dim3(64 * kFieldWaves), 0, st, f,
                       (const int32_t*)S.tile_inv, a);
    return hipGetLastError();
  }
  if (mom_blocks > 0) {
    hipLaunchKernelGGL(shape_moments_kernel, dim3(mom_blocks), dim3(64 * kMomWaves),
                       mom_lds, st, m);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  ExtArgs x{T, node_off, y, T.n_nodes, S.d2max, S.tile_inv, S.cell_inv};
  hipLaunchKernelGGL(shape_extreme_kernel, dim3(nc), dim3(256), 0, st, x);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (S.n_node_blocks > 0) {
    BoxArgs bx{S.node_blocks, node_off, S.order, y, T.n_nodes, S.bbox};
    hipLaunchKernelGGL(shape_bbox_kernel, dim3((unsigned)S.n_node_blocks), dim3(256), 0,
                       st, bx);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (S.n_cand_blocks > 0) {
    PairArgs p{S.cand_blocks, node_off, S.order, y, T.n_nodes, S.bbox, S.d2max};
    hipLaunchKernelGGL(pair_max_kernel, dim3((unsigned)S.n_cand_blocks), dim3(256), 0,
                       st, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  AllArgs al{node_off, y, T.n_nodes, S.cell_inv, S.d2max};
  hipLaunchKernelGGL(pair_all_kernel, dim3(nc), dim3(256), 0, st, al);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(shape_finalize_kernel, dim3((nc + 3) / 4), dim3(256), 0, st, f);
  return hipGetLastError();
}

}  // namespace cm
