// Parts that the tile passes with several wavefronts per tile share (wide.hip,
// lists.hip): arguments, node gather, the evaluation of one tetrahedron, the
// output of one node.
#pragma once
#include <hip/hip_runtime.h>

#include "cg.h"
#include "device_util.h"
#include "kernels.h"
#include "mr_tet.h"
#include "plate.h"

namespace cm {

// What the pass reads before its first tetrahedron comes first: the kernel
// loads it with the arguments' first two cache lines.
struct WideArgs {
  const TileDesc* tiles;
  const TetChunk* chunks;
  const int32_t* ids;      // slot_node, or slot_node_first for a plate step
  const int32_t* tile_mat;
  const double* params;
  const float* y;
  const float* fbar;       // y where there is none (then has_fbar is 0)
  const double* flags;     // per cell: CellMask (nullable)
  int64_t flag_stride, N;
  int32_t tile_begin, n_tiles, nloc, n_mat, last_slot, has_fbar;
  int32_t check;           // count tets with a non-finite energy or force
  const double* ebar;      // nullable
  float* f;
  float* ybar;
  float* part;             // the forward's scratch
  double* tile_acc;
  double* tile_plate;
  int32_t* tile_ninv;
  int32_t* tile_nonfin;
  float* part_b;           // the backward's
  double* tile_acc_b;
  ListTables lists;        // lists.hip
  int32_t copies;          // tiles per list block (copies of a shared mesh)
  PlateFwd pf;             // used when PL and FWD
  PlateBwd pb;             // used when PL and BWD
  CellOut out;             // tail.h, with T
  DeviceTables T;
  CgArgs cg;               // tail.h: the iteration that a Hessian product ends in
};

inline WideArgs wide_args(const DeviceTables& T, const Range& r, const float* y,
                          const int32_t* ids, const CellOut& out = CellOut{}) {
  WideArgs a{};
  a.tiles = T.tiles;
  a.chunks = T.chunks;
  a.ids = ids;
  a.tile_mat = T.tile_mat;
  a.params = T.params;
  a.y = y;
  a.fbar = y;
  a.flag_stride = 1;
  a.N = T.n_nodes;
  a.tile_begin = r.tile_begin;
  a.n_tiles = r.tile_end - r.tile_begin;
  a.nloc = T.nloc;
  a.n_mat = T.n_mat;
  a.lists = T.lists;
  a.copies = T.tile_stride;
  a.last_slot = T.n_slots > 0 ? (int32_t)T.n_slots - 1 : 0;
  a.out = out;
  a.T = T;
  return a;
}

inline WideArgs forward_args(const DeviceTables& T, const Range& r, const float* y, float* f,
                             const PlateFwd& pl, bool check,
                             const CellOut& out = CellOut{}) {
  WideArgs a = wide_args(T, r, y, pl.plate ? T.slot_node_first : T.slot_node, out);
  a.f = f;
  a.part = T.part;
  a.tile_acc = T.tile_acc;
  a.tile_plate = T.tile_plate;
  a.tile_ninv = T.tile_ninv;
  a.tile_nonfin = T.tile_nonfin;
  a.check = check ? 1 : 0;
  a.pf = pl;
  return a;
}

inline WideArgs backward_args(const DeviceTables& T, const Range& r, const float* y,
                              const float* fbar, const double* ebar, float* ybar,
                              const CellMask& mask, const PlateBwd& pl,
                              const CellOut& out = CellOut{}) {
  WideArgs a = wide_args(T, r, y, T.slot_node, out);
  if (fbar) a.fbar = fbar;
  a.has_fbar = fbar ? 1 : 0;
  a.ebar = ebar;
  a.ybar = ybar;
  a.part_b = T.part;
  a.tile_acc_b = T.tile_acc;
  a.flags = mask.flags;
  a.flag_stride = mask.stride;
  a.pb = pl;
  return a;
}

inline WideArgs forward_backward_args(const DeviceTables& T, const DeviceTables& Tb,
                                      const Range& r, const float* y, float* f,
                                      const float* fbar, const double* ebar, float* ybar,
                                      const CellOut& out = CellOut{}) {
  WideArgs a = wide_args(T, r, y, T.slot_node, out);
  a.f = f;
  a.part = T.part;
  a.tile_acc = T.tile_acc;
  a.tile_ninv = T.tile_ninv;
  if (fbar) a.fbar = fbar;
  a.has_fbar = fbar ? 1 : 0;
  a.ebar = ebar;
  a.ybar = ybar;
  a.part_b = Tb.part;
  a.tile_acc_b = Tb.tile_acc;
  return a;
}

// Loads grouped by data flow: each of these empty statements makes all of its
// values available at once, so that the compiler issues their loads together
// instead of each where its value is first used, one more round trip to
// memory for every step.
__device__ __forceinline__ void together(int32_t (&)[1]) {}
__device__ __forceinline__ void together(float (&v)[1][3]) {
  asm("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]));
}
__device__ __forceinline__ void together(float (&v)[1][3], float (&w)[1][3]) {
  asm("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(w[0][0]), "+v"(w[0][1]),
           "+v"(w[0][2]));
}
__device__ __forceinline__ void together(int32_t (&v)[2]) {
  asm("" : "+v"(v[0]), "+v"(v[1]));
}
__device__ __forceinline__ void together(int32_t (&v)[3]) {
  asm("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]));
}
__device__ __forceinline__ void together(float (&v)[2][3]) {
  asm("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(v[1][0]), "+v"(v[1][1]),
           "+v"(v[1][2]));
}
__device__ __forceinline__ void together(float (&v)[3][3]) {
  asm("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(v[1][0]), "+v"(v[1][1]),
           "+v"(v[1][2]), "+v"(v[2][0]), "+v"(v[2][1]), "+v"(v[2][2]));
}
__device__ __forceinline__ void together(float (&v)[2][3], float (&w)[2][3]) {
  asm("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(v[1][0]), "+v"(v[1][1]),
           "+v"(v[1][2]), "+v"(w[0][0]), "+v"(w[0][1]), "+v"(w[0][2]), "+v"(w[1][0]),
           "+v"(w[1][1]), "+v"(w[1][2]));
}
__device__ __forceinline__ void together(float (&v)[3][3], float (&w)[3][3]) {
  asm("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(v[1][0]), "+v"(v[1][1]),
           "+v"(v[1][2]), "+v"(v[2][0]), "+v"(v[2][1]), "+v"(v[2][2]), "+v"(w[0][0]),
           "+v"(w[0][1]), "+v"(w[0][2]), "+v"(w[1][0]), "+v"(w[1][1]), "+v"(w[1][2]),
           "+v"(w[2][0]), "+v"(w[2][1]), "+v"(w[2][2]));
}

// Node gather of L threads: the ids of U nodes per thread, then their
// positions and cotangents, each step's loads issued together (a loop over
// single nodes waits for both steps every time, and a tile of 283 nodes makes
// two or three rounds of 64 K threads).  Threads past the last node load a
// valid one again.  mu, kappa and w arrive with the ids.
template <int L, int U, bool FWD, bool BWD, bool PL>
__device__ __forceinline__ void gather_nodes(const WideArgs& a, TileDesc& d, int nl, int tid,
                                             float4* ys, float2* vs, double& mu,
                                             double& kappa, double& w) {
  const int64_t N = a.N;
  for (int b = 0; b < nl; b += U * L) {
    const int l0 = b + tid;
    int32_t v[U];
    float yv[U][3], fv[U][3];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = a.ids[min(d.shr_begin + max(min(l0 + u * L, nl - 1) - d.n_own, 0),
                       a.last_slot)];
    together(v);
    // (the material has arrived when the first addresses are formed)
    asm("" : "+s"(mu), "+s"(kappa), "+s"(w), "+s"(d.own_begin));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int l = min(l0 + u * L, nl - 1);
      if (l < d.n_own) v[u] = (PL && FWD ? INT32_MIN : 0) | (d.own_begin + l);
      const int64_t g = v[u] & 0x7fffffff;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        yv[u][c] = a.y[c * N + g];
        if constexpr (BWD) fv[u][c] = a.fbar[c * N + g];
      }
    }
    if constexpr (BWD)
      together(yv, fv);
    else
      together(yv);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int l = l0 + u * L;
      if (l < nl) {
        float f0 = PL && FWD && v[u] < 0 ? 1.f : 0.f;
        if constexpr (BWD) {
          f0 = a.has_fbar ? fv[u][0] : 0.f;
          vs[l] = a.has_fbar ? make_float2(fv[u][1], fv[u][2]) : make_float2(0.f, 0.f);
        }
        ys[l] = make_float4(yv[u][0], yv[u][1], yv[u][2], f0);
      }
    }
  }
}

// One lane's tetrahedron: contributions to the forces (h) and to ybar (hb) of
// vertices 0..2 (vertex 3 takes the negative sum), energy, parameter-gradient
// terms; as tet_forward and tet_backward.
struct TetOut {
  float h[3][3], hb[3][3];
  double vU, gp[3], ge[3], vol;
  bool inv, bad;
};

template <bool FWD, bool BWD, bool GRAD>
__device__ __forceinline__ void eval_tet(const TetRegs& cur, const float4* ys,
                                         const float2* vs, const Material& mat, double eb,
                                         bool check, TetOut& o) {
  const int i0 = cur.q.x & 0xffff, i1 = cur.q.x >> 16;
  const int i2 = cur.q.y & 0xffff, i3 = cur.q.y >> 16;
  const float4 p0 = ys[i0], p1 = ys[i1], p2 = ys[i2], p3 = ys[i3];
  double Fd[3][3];
  float F[3][3], Cf[6];
  deformation_gradient(p0, p1, p2, p3, cur.B, Fd, F);
  Scalars sc;
  invariants(Fd, Cf, sc);
  if constexpr (FWD) {
    stress_forces(F, Cf, sc, cur.B, cur.V0, mat, o.h, o.vU);
    o.inv = !(sc.J > 0.0);
    if (!BWD && check) {
      float sum = 0.f;
#pragma unroll
      for (int c = 0; c < 3; ++c) sum += o.h[c][0] + o.h[c][1] + o.h[c][2];
      o.bad = !(isfinite(o.vU) && isfinite(sum));
    }
    // the forward half's temporaries are dead before the adjoint half's are
    // formed
    if constexpr (BWD) __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (BWD) {
    const float2 w0 = vs[i0], w1 = vs[i1], w2 = vs[i2], w3 = vs[i3];
    const float4 v0 = make_float4(p0.w, w0.x, w0.y, 0.f);
    const float4 v1 = make_float4(p1.w, w1.x, w1.y, 0.f);
    const float4 v2 = make_float4(p2.w, w2.x, w2.y, 0.f);
    const float4 v3 = make_float4(p3.w, w3.x, w3.y, 0.f);
    float dF[3][3], Kc[3][3];
    cofactor(F, Kc);
    direction_gradient(v0, v1, v2, v3, cur.B, dF);
    adjoint_terms<GRAD>(F, dF, Cf, Kc, sc, cur.B, cur.V0, mat, eb, o.hb, o.gp, o.ge);
    o.vol = (double)cur.V0;
  }
}

// Output of tile node l with force sum fv and ybar sum gv: an owned node's
// values (or its plate step), a shared node's slot partials.
template <bool FWD, bool BWD, bool PL, bool TAIL = false, bool CG = false>
__device__ __forceinline__ void store_node(const WideArgs& a, const TileDesc& d, int l,
                                           const float fv[3], const float gv[3],
                                           const float4* ys, const float2* vs, float top,
                                           float bot, float gw) {
  const int64_t N = a.N;
  if (l < d.n_own) {
    const int64_t g = (int64_t)d.own_begin + l;
    if constexpr (PL) {
      const float4 p = ys[l];
      if constexpr (FWD) {
        plate_node_step(p.x, p.y, p.z, fv[0], fv[1], fv[2], top, bot, a.pf.k,
                        a.pf.m, a.pf.y_next, N, g);
      } else {
        const float2 v = vs[l];
        plate_node_adjoint(p.z, p.w, v.x, v.y, gv[0], gv[1], gv[2], top, bot,
                           a.pb.k, a.pb.m, gw, a.pb.lam, N, g);
      }
    } else {
      if constexpr (FWD) {
        a.f[g] = fv[0]; a.f[N + g] = fv[1]; a.f[2 * N + g] = fv[2];
      }
      if constexpr (BWD) {
#pragma unroll
        for (int c = 0; c < 3; ++c) store_as<CG>(a.ybar + c * N + g, gv[c]);
      }
    }
  } else {
    const int slot = d.shr_begin + l - d.n_own;
    const int64_t s = 3 * (int64_t)slot;
    if constexpr (TAIL) {
      if constexpr (FWD) device_store3(a.part, slot, fv);
      if constexpr (BWD) device_store3(a.part_b, slot, gv);
      return;
    }
    if constexpr (FWD) {
      a.part[s] = fv[0]; a.part[s + 1] = fv[1]; a.part[s + 2] = fv[2];
    }
    if constexpr (BWD) {
      a.part_b[s] = gv[0]; a.part_b[s + 1] = gv[1]; a.part_b[s + 2] = gv[2];
    }
  }
}

// The tile's share of the top-plate force, on one wavefront: its owned nodes
// and the shared nodes whose first slot it holds.
__device__ __forceinline__ double plate_share(const TileDesc& d, const float4* ys, int lane,
                                              float top, float k) {
  double fp = 0.0;
  for (int i = lane; i < d.n_own; i += 64) fp += plate_top_term(ys[i].z, top, k);
  for (int j = lane; j < d.n_shr; j += 64) {
    const float4 p = ys[d.n_own + j];
    if (p.w != 0.f) fp += plate_top_term(p.z, top, k);
  }
  return wave_sum(fp);
}

}  // namespace cm
