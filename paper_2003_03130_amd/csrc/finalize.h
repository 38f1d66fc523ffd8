// Sums of the finalize kernels, each in a fixed order (deterministic):
// per cell the tile energies and inverted counts, per material slot the
// parameter-gradient sums, per shared node its slot partials.
#pragma once
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "kernels.h"
#include "plate.h"

namespace cm {

// Here and below, DEVICE: in the launch that wrote the terms (tail.h).
// Energy, inverted count and (with nonfin) non-finite count of cell c over
// its tiles, on every lane of the wave: lane l takes tiles l, l + 64, ...,
// then a fixed butterfly (the cells' long chains of loads run in parallel).
struct CellSums {
  double e;
  int ni, nf;
};
template <bool DEVICE = false>
__device__ __forceinline__ CellSums cell_sums(const DeviceTables& T, int c, int lane,
                                              bool nonfin) {
  CellSums s{0.0, 0, 0};
  const int t0 = T.cell_tile_first[c], nt = T.cell_tile_count[c];
  for (int k = lane; k < nt; k += 64) {
    const int64_t t = t0 + (int64_t)k * T.tile_stride;
    s.e += load_as<DEVICE>(T.tile_acc + t);
    s.ni += load_as<DEVICE>(T.tile_ninv + t);
    if (nonfin) s.nf += load_as<DEVICE>(T.tile_nonfin + t);
  }
  s.e = wave_sum(s.e);
  s.ni = wave_sum(s.ni);
  if (nonfin) s.nf = wave_sum(s.nf);
  return s;
}

// Top-plate force of cell c: the tile shares, then the nodes of no
// tetrahedron, on every lane.
template <bool DEVICE = false>
__device__ __forceinline__ double cell_plate_force(const DeviceTables& T, int c, int lane,
                                                   const float* y, float top, float k) {
  const int t0 = T.cell_tile_first[c], nt = T.cell_tile_count[c];
  double fp = 0.0;
  for (int i = lane; i < nt; i += 64)
    fp += load_as<DEVICE>(T.tile_plate + t0 + (int64_t)i * T.tile_stride);
  for (int o = T.orphan_off[c] + lane; o < T.orphan_off[c + 1]; o += 64)
    fp += plate_top_term(y[2 * T.n_nodes + T.orphan_node[o]], top, k);
  return wave_sum(fp);
}

// dL/d(mu, kappa, w) of material slot mt, on every lane of the wave:
//   dL/dmu = w g_I + (1 - w) g_K, dL/dkappa = g_J, dL/dw = mu (g_I - g_K)
// from its tiles' sums (tile_acc, three per tile) of dL/d(mu1, mu2, kappa)
// with mu1 = w mu, mu2 = (1 - w) mu; lane l takes tiles l, l + 64, ...,
// then a fixed butterfly.
template <bool DEVICE = false>
__device__ __forceinline__ void slot_theta(const DeviceTables& T, const double* tile_acc,
                                           int mt, int lane, double t3[3]) {
  double gI = 0.0, gK = 0.0, gJ = 0.0;
  const int t0 = T.mat_tile_first[mt], nt = T.mat_tile_count[mt];
  for (int k = lane; k < nt; k += 64) {
    const int64_t t = t0 + (int64_t)k * T.tile_stride;
    gI += load_as<DEVICE>(tile_acc + 3 * t);
    gK += load_as<DEVICE>(tile_acc + 3 * t + 1);
    gJ += load_as<DEVICE>(tile_acc + 3 * t + 2);
  }
  gI = wave_sum(gI);
  gK = wave_sum(gK);
  gJ = wave_sum(gJ);
  const int nm = T.n_mat;
  const double mu = T.params[mt], w = T.params[2 * nm + mt];
  t3[0] = w * gI + (1.0 - w) * gK;
  t3[1] = gJ;
  t3[2] = mu * (gI - gK);
}

// The slots of one shared node.  Its record (shared_rec, 16 bytes) holds the
// node and its first three slots, -1 for none; a node with more slots has
// -2 - k in place of the third, and the record shared_rec4[k] holds its third
// to sixth, the sixth being -2 - m for a node with more than six, whose sixth
// slot on follows in shared_more[m + 1 ...], their number in shared_more[m].
// One load thus gives most nodes' slots and a second the others', and all of
// a node's partials are loaded at once: the finalize kernels are bound by
// this chain of loads.  Before (an offset, then slot after slot its id and its
// partial) -> now: forward 8 cells 4.9 -> 3.7 us, 1,024 uneven cells 15.8 ->
// 13.0; plate step of 32 cells 5.7 -> 4.4; both passes 4,096 cells 77 -> 69;
// the CG kernel, which forms the same sums, 7.9 -> 7.3.
struct SharedSlots {
  int64_t node;
  int slot[6];  // -1: none
  int more;     // >= 0: further slots in shared_more
};

__device__ __forceinline__ SharedSlots shared_slots(const int4& r, const int4* rec4) {
  SharedSlots o{r.x, {r.y, r.z, r.w, -1, -1, -1}, -1};
  if (r.w < -1) {
    const int4 q = rec4[-2 - r.w];
    o.slot[2] = q.x;
    o.slot[3] = q.y;
    o.slot[4] = q.z;
    o.slot[5] = q.w;
    if (q.w < -1) {
      o.slot[5] = -1;
      o.more = -2 - q.w;
    }
  }
  return o;
}

template <bool DEVICE>
__device__ __forceinline__ void load3_as(const float* part, int slot, float (&v)[3]) {
  if constexpr (DEVICE) {
    device_load3(part, slot, v);
  } else {
    const float* p = part + 3 * (int64_t)slot;
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = p[c];
  }
}

// Sums of M arrays of slot partials (three floats per slot) over the node's
// slots, in tile order.
template <int M, bool DEVICE = false>
__device__ __forceinline__ void shared_sums(const SharedSlots& o, const int32_t* more,
                                            const float* const (&part)[M], float (&sum)[M][3]) {
  float v[6][M][3];
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    if (j < 3 || o.slot[3] >= 0) {
      const int s = max(o.slot[j], 0);
#pragma unroll
      for (int m = 0; m < M; ++m) load3_as<DEVICE>(part[m], s, v[j][m]);
    }
  }
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int c = 0; c < 3; ++c) sum[m][c] = 0.f;
#pragma unroll
  for (int j = 0; j < 6; ++j)
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        sum[m][c] = o.slot[j] >= 0 ? sum[m][c] + v[j][m][c] : sum[m][c];
  if (o.more >= 0) {
    const int n = more[o.more];
    for (int k = 1; k <= n; ++k) {
      const int s = more[o.more + k];
#pragma unroll
      for (int m = 0; m < M; ++m) {
        float w[3];
        load3_as<DEVICE>(part[m], s, w);
#pragma unroll
        for (int c = 0; c < 3; ++c) sum[m][c] += w[c];
      }
    }
  }
}

__device__ __forceinline__ float3 shared_sum(const DeviceTables& T, const float* part,
                                             const SharedSlots& o) {
  const float* const p[1] = {part};
  float s[1][3];
  shared_sums(o, T.shared_more, p, s);
  return make_float3(s[0][0], s[0][1], s[0][2]);
}

}  // namespace cm
