// Conjugate-gradient iteration of the quasi-static solver: parts that its own
// kernel (quasistatic.hip) and the Hessian-vector product that ends in it
// (tail.h) share.
#pragma once
#include <hip/hip_runtime.h>

#include "aux_kernels.h"
#include "finalize.h"

namespace cm {

constexpr int kThreads = 1024;

// Workgroup sum in a fixed order: a butterfly inside each wavefront (every
// lane ends with the same bits), then every thread adds the wavefront totals
// in wavefront order.  red: at least NT / 64 doubles of LDS.
template <int NT = kThreads>
__device__ __forceinline__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = red[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) r += red[w];
  __syncthreads();  // red is reused by the next reduction
  return r;
}

// K workgroup sums at once, each in the order of block_sum (bitwise its
// result): the wavefront totals of sum k are added up by thread k alone, so
// no thread holds all K NT / 64 totals at once.  red: at least K (NT / 64 +
// 1) doubles.
template <int K, int NT = kThreads>
__device__ __forceinline__ void block_sums(double (&v)[K], double* red) {
  constexpr int NW = NT / 64;
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) red[k * NW + (threadIdx.x >> 6)] = v[k];
  }
  __syncthreads();
  if ((int)threadIdx.x < K) {
    const int k = threadIdx.x;
    double r = red[k * NW];
    for (int w = 1; w < NW; ++w) r += red[k * NW + w];
    red[K * NW + k] = r;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = red[K * NW + k];
  __syncthreads();  // red is reused by the next reduction
}

// Sphere indenter (Indenter with R > 0): node (x, y, z) against the sphere
// of cell c whose lowest point is at height top.  g = max(0, R - d) is the
// penetration, d the distance to the centre, n the unit vector from the
// centre to the node (zero without contact).  The penalty potential is
// (k/3) g^3 as for the plates: force k g^2 n on the node, k g^2 (c_z - z) / d
// upward on the sphere, Hessian 2 k g n n^T - k (g^2 / d) (I - n n^T).
struct SphereHit {
  double g, d, n[3];
};

__device__ __forceinline__ SphereHit sphere_hit(const Indenter& ind, int c, double top,
                                                double x, double y, double z) {
  SphereHit h;
  const double rx = x - ind.axis[2 * c], ry = y - ind.axis[2 * c + 1];
  const double rz = z - (top + ind.R);
  h.d = sqrt(rx * rx + ry * ry + rz * rz);
  h.g = h.d > 0.0 ? fmax(ind.R - h.d, 0.0) : 0.0;
  const double inv = h.g > 0.0 ? 1.0 / h.d : 0.0;
  h.n[0] = rx * inv;
  h.n[1] = ry * inv;
  h.n[2] = rz * inv;
  return h;
}

// Hessian of the sphere's penalty potential times v.
__device__ __forceinline__ void sphere_hess(const SphereHit& h, double k, double vx,
                                            double vy, double vz, double out[3]) {
  if (!(h.g > 0.0)) {
    out[0] = out[1] = out[2] = 0.0;
    return;
  }
  const double nv = h.n[0] * vx + h.n[1] * vy + h.n[2] * vz;
  const double a = 2.0 * k * h.g * nv, b = k * h.g * h.g / h.d;
  out[0] = a * h.n[0] - b * (vx - nv * h.n[0]);
  out[1] = a * h.n[1] - b * (vy - nv * h.n[1]);
  out[2] = a * h.n[2] - b * (vz - nv * h.n[2]);
}

// Projection onto the complement of the modes the sphere setup removes
// (translations in x and y, which the held centroid takes, and the rotation
// about the vertical axis through the centroid (cx, cy), a symmetry): from
// the cell sums sx = sum v_x, sy = sum v_y, sr = sum (dx v_y - dy v_x), with
// inv_n = 1 / nodes and ww = sum (dx^2 + dy^2).
struct ModeFit {
  double tx, ty, om;
};

__device__ __forceinline__ ModeFit mode_fit(double sx, double sy, double sr,
                                           double inv_n, double ww) {
  return ModeFit{sx * inv_n, sy * inv_n, ww > 0.0 ? sr / ww : 0.0};
}

// z = M r for one symmetric 3x3 block m = (xx yy zz xy xz yz).
__device__ __forceinline__ void sym3_mul(const float* m, float rx, float ry, float rz,
                                         float& zx, float& zy, float& zz) {
  zx = m[0] * rx + m[3] * ry + m[4] * rz;
  zy = m[3] * rx + m[1] * ry + m[5] * rz;
  zz = m[4] * rx + m[5] * ry + m[2] * rz;
}

struct CgArgs {
  const int64_t* node_off;
  int64_t N;
  const float* y;
  const double* plate;
  double k, rel_tol;
  const float* ybar;  // (df/dy)^T p
  float *x, *r, *p, *Ap;
  double* st;
  const float* minv;  // preconditioner blocks (6 n_nodes), nullable
  // With part set, ybar holds the owned nodes only (a backward tile pass
  // without its finalize) and the shared nodes' values are the sums of
  // their slot partials, formed here in the finalize's order.
  const float* part;
  const int4* shared_rec;
  const int4* shared_rec4;
  const int32_t* shared_more;
  const int32_t* cell_shared_off;
  const int32_t* cell_shared_first;  // first shared node of every cell
  Indenter ind;
};

inline CgArgs cg_args(const int64_t* node_off, int64_t N, const float* y, const double* plate,
                      double k, double rel_tol, const float* ybar, float* x, float* r,
                      float* p, float* Ap, double* st, const float* minv,
                      const DeviceTables* slots, const Indenter& ind) {
  return CgArgs{node_off, N, y, plate, k, rel_tol, ybar, x, r, p, Ap, st, minv,
                slots ? slots->part : nullptr,
                slots ? slots->shared_rec : nullptr,
                slots ? slots->shared_rec4 : nullptr,
                slots ? slots->shared_more : nullptr,
                slots ? slots->cell_shared_off : nullptr,
                slots ? slots->cell_shared_first : nullptr, ind};
}

// The shared nodes of a cell are the contiguous ids [sh0, sh0 + ns) (owned
// nodes first, see layout.h); s0 is the cell's first shared-node entry.
struct ShrRange {
  int64_t sh0, sh1;
  int s0;
};

__device__ __forceinline__ ShrRange shared_range(const CgArgs& a, int c, int64_t n1) {
  ShrRange r{n1, n1, 0};
  if (a.part) {
    r.s0 = a.cell_shared_off[c];
    const int ns = a.cell_shared_off[c + 1] - r.s0;
    if (ns > 0) {
      r.sh0 = a.cell_shared_first[c];
      r.sh1 = r.sh0 + ns;
    }
  }
  return r;
}

// ybar of node i: stored, or for a shared node the sum of its slot partials
// in slot order (the order of backward_finalize_kernel: bitwise its result).
__device__ __forceinline__ void ybar_of(const CgArgs& a, const ShrRange& sr, int64_t i,
                                        float& bx, float& by, float& bz) {
  if (i >= sr.sh0 && i < sr.sh1) {
    const int s = sr.s0 + (int)(i - sr.sh0);
    const float* const part[1] = {a.part};
    float v[1][3];
    shared_sums(shared_slots(a.shared_rec[s], a.shared_rec4), a.shared_more, part, v);
    bx = v[0][0]; by = v[0][1]; bz = v[0][2];
  } else {
    bx = a.ybar[i]; by = a.ybar[a.N + i]; bz = a.ybar[2 * a.N + i];
  }
}

// Nodes per thread up to which a cell's CG iteration keeps every operand in
// registers (cells of at most kRegNodes * kThreads nodes; cells of at most
// kThreads * 2 nodes take a 2-node variant that needs fewer registers).
constexpr int kRegNodes = 4;

__device__ __forceinline__ void cg_finish(const CgArgs& a, double* s, double rn,
                                          double rzn) {
  if (threadIdx.x == 0) {
    s[0] = rzn;
    const double tol = fmax(a.rel_tol, s[14]);
    if (rn <= tol * tol * s[1]) s[2] = 0.0;
  }
}


// The iteration of qs_cg_kernel for a cell of at most R * kThreads nodes: p,
// r, x, Hess(Pi) p and the preconditioner block of every node are loaded
// once and kept in registers through the three phases (Ap is not stored).
// The loads come in two waves, each issued whole before any of its results
// is used: the node values with the slot records of the shared nodes, then
// those slots' partials, summed in slot order as the finalize does.  Same
// operations in the same order as the streaming version (which fused
// multiply-adds the compiler forms may differ between the two, a last-bit
// difference).  DEVICE: ybar and the partials were written in this launch
// (tail.h).
template <int R, bool SPH, bool DEVICE = false>
__device__ __forceinline__ void cg_step_regs(const CgArgs& a, double* s, int c, int64_t n0,
                                             int64_t n1, double top, double bot,
                                             double* red, const ShrRange& sr) {
  constexpr int kRegNodes = R;
  const int64_t N = a.N;
  float p[kRegNodes][3], r[kRegNodes][3], ap[kRegNodes][3], x[kRegNodes][3];
  float m[kRegNodes][6], b[kRegNodes][3];
  double h[kRegNodes];        // plates: penalty Hessian on zz
  float yv[kRegNodes][3];     // sphere: positions
  int4 rec[kRegNodes];        // a shared node's slots (node < 0: an owned node)
#pragma unroll
  for (int u = 0; u < kRegNodes; ++u) {
    const int64_t i = n0 + threadIdx.x + (int64_t)u * kThreads;
    rec[u] = make_int4(-1, -1, -1, -1);
    if (i < n1) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        p[u][d] = a.p[d * N + i];
        r[u][d] = a.r[d * N + i];
        x[u][d] = a.x[d * N + i];
      }
      if (a.minv) {
#pragma unroll
        for (int q = 0; q < 6; ++q) m[u][q] = a.minv[q * N + i];
      }
      if constexpr (SPH) {
#pragma unroll
        for (int d = 0; d < 3; ++d) yv[u][d] = a.y[d * N + i];
      } else {
        const double z = a.y[2 * N + i];
        h[u] = 2.0 * a.k * (fmax(z - top, 0.0) + fmax(bot - z, 0.0));
      }
      if (i >= sr.sh0 && i < sr.sh1) {
        rec[u] = a.shared_rec[sr.s0 + (int)(i - sr.sh0)];
      } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) b[u][d] = load_as<DEVICE>(a.ybar + d * N + i);
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kRegNodes; ++u) {
    if (rec[u].x >= 0) {
      const float* const part[1] = {a.part};
      float v[1][3];
      shared_sums<1, DEVICE>(shared_slots(rec[u], a.shared_rec4), a.shared_more, part, v);
#pragma unroll
      for (int c = 0; c < 3; ++c) b[u][c] = v[0][c];
    }
  }
  // sphere: centroid and sum (dx^2 + dy^2) of the Newton step's positions
  double gcx = 0.0, gcy = 0.0, gww = 0.0;
  if constexpr (SPH) {
    gcx = a.ind.geo[3 * c];
    gcy = a.ind.geo[3 * c + 1];
    gww = a.ind.geo[3 * c + 2];
  }
  const double inv_n = 1.0 / (double)(n1 - n0);
  double pap = 0.0, sa[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < kRegNodes; ++u) {
    const int64_t i = n0 + threadIdx.x + (int64_t)u * kThreads;
    if (i < n1) {
      if constexpr (SPH) {
        const SphereHit hh = sphere_hit(a.ind, c, top, yv[u][0], yv[u][1], yv[u][2]);
        double hp[3];
        sphere_hess(hh, a.k, p[u][0], p[u][1], p[u][2], hp);
        hp[2] += 2.0 * a.k * fmax(bot - (double)yv[u][2], 0.0) * (double)p[u][2];
#pragma unroll
        for (int d = 0; d < 3; ++d) ap[u][d] = (float)(-(double)b[u][d] + hp[d]);
        const double dx = yv[u][0] - gcx, dy = yv[u][1] - gcy;
        sa[0] += ap[u][0];
        sa[1] += ap[u][1];
        sa[2] += dx * ap[u][1] - dy * ap[u][0];
      } else {
        ap[u][0] = -b[u][0];
        ap[u][1] = -b[u][1];
        ap[u][2] = (float)(-(double)b[u][2] + h[u] * (double)p[u][2]);
      }
      pap += (double)p[u][0] * ap[u][0] + (double)p[u][1] * ap[u][1] +
             (double)p[u][2] * ap[u][2];
    }
  }
  ModeFit ma{0.0, 0.0, 0.0};
  if constexpr (SPH) {
    double v[4] = {pap, sa[0], sa[1], sa[2]};
    block_sums(v, red);
    pap = v[0];
    ma = mode_fit(v[1], v[2], v[3], inv_n, gww);
  } else {
    pap = block_sum(pap, red);
  }
  const double rs = s[0];
  if (!(pap > 0.0)) {
    if (threadIdx.x == 0) s[2] = 0.0;
    return;
  }
  const float alpha = (float)(rs / pap);
  double rn = 0.0, rzn = 0.0, sz[3] = {0.0, 0.0, 0.0};
  float zv[kRegNodes][3];
#pragma unroll
  for (int u = 0; u < kRegNodes; ++u) {
    const int64_t i = n0 + threadIdx.x + (int64_t)u * kThreads;
    if (i < n1) {
      if constexpr (SPH) {
        // Ap projected: the held centroid and the symmetry take its mode part
        const double dx = yv[u][0] - gcx, dy = yv[u][1] - gcy;
        ap[u][0] = (float)((double)ap[u][0] - ma.tx + ma.om * dy);
        ap[u][1] = (float)((double)ap[u][1] - ma.ty - ma.om * dx);
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int64_t q = d * N + i;
        a.x[q] = x[u][d] + alpha * p[u][d];
        r[u][d] = r[u][d] - alpha * ap[u][d];
        a.r[q] = r[u][d];
        rn += (double)r[u][d] * r[u][d];
      }
      zv[u][0] = r[u][0];
      zv[u][1] = r[u][1];
      zv[u][2] = r[u][2];
      if (a.minv) sym3_mul(m[u], r[u][0], r[u][1], r[u][2], zv[u][0], zv[u][1], zv[u][2]);
      rzn += (double)r[u][0] * zv[u][0] + (double)r[u][1] * zv[u][1] +
             (double)r[u][2] * zv[u][2];
      if constexpr (SPH) {
        const double dx = yv[u][0] - gcx, dy = yv[u][1] - gcy;
        sz[0] += zv[u][0];
        sz[1] += zv[u][1];
        sz[2] += dx * zv[u][1] - dy * zv[u][0];
      }
    }
  }
  ModeFit mz{0.0, 0.0, 0.0};
  if constexpr (SPH) {
    double v[5] = {rn, rzn, sz[0], sz[1], sz[2]};
    block_sums(v, red);
    rn = v[0];
    rzn = v[1];
    mz = mode_fit(v[2], v[3], v[4], inv_n, gww);
  } else {
    double sums[2] = {rn, rzn};
    block_sums(sums, red);
    rn = sums[0];
    rzn = sums[1];
  }
  const float beta = (float)(rzn / rs);
#pragma unroll
  for (int u = 0; u < kRegNodes; ++u) {
    const int64_t i = n0 + threadIdx.x + (int64_t)u * kThreads;
    if (i < n1) {
      if constexpr (SPH) {
        const double dx = yv[u][0] - gcx, dy = yv[u][1] - gcy;
        zv[u][0] = (float)((double)zv[u][0] - mz.tx + mz.om * dy);
        zv[u][1] = (float)((double)zv[u][1] - mz.ty - mz.om * dx);
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) a.p[d * N + i] = zv[u][d] + beta * p[u][d];
    }
  }
  cg_finish(a, s, rn, rzn);
}

}  // namespace cm
