// A cell's sums formed by the tile pass itself: the workgroup of the cell's tile
// that arrives last adds up its shared nodes, energies and parameter gradients
// in place of a second launch, in that launch's order (finalize.h): bitwise its
// results.
//
// What one tile's workgroup hands to another goes past the caches of its XCD:
// the slot partials and tile sums are stored and loaded with device scope, and
// every wavefront waits until its stores have arrived before the workgroup
// counts itself in.  (Fences of device scope write back and invalidate whole
// caches: forward of 16 cells 46 us instead of 9.)  The counter wraps to zero
// with the cell's last tile; only that one goes on, so nothing waits for another
// workgroup.
//
// Against the finalize launch behind the pass this saves a launch and its chain
// of loads, but one workgroup now forms all of a cell's sums; it is bound by the
// requests of those loads (12 bytes each; as three of 4 bytes 10.3 us where it
// is 8.9).  Calls with the finalize -> with the tail: forward, adjoint,
// Hessian-vector product of 8 cells of 2,054 nodes 10.9, 11.5, 11.0 -> 8.6, 9.8,
// 9.0 us; of 30 cells of 900 11.0, 11.4, 11.0 -> 8.3, 9.5, 8.6; backpropagation
// through 40 plate steps of 8 cells 1,440 -> 1,205.
#pragma once
#include "cg.h"
#include "wide.h"

namespace cm {

// Whether a tile pass goes on to its cells' sums, or (a Hessian-vector product of
// the search direction) to their conjugate-gradient iteration.
enum Tail { kNoTail, kCellSums, kCgPlates, kCgSphere };

template <int L, bool FWD, bool BWD, bool PL, bool GRAD>
__device__ __forceinline__ void cell_tail(const WideArgs& a, int c, int tid, int* flag) {
  constexpr int W = L / 64;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t N = a.N;
  const int s0 = a.T.cell_shared_off[c], s1 = a.T.cell_shared_off[c + 1];
  const uint32_t last = (uint32_t)a.T.cell_tile_count[c] - 1;
  // the slots of the thread's first node, while the stores are on their way
  SharedSlots sl{};
  if (s0 + tid < s1) sl = shared_slots(a.T.shared_rec[s0 + tid], a.T.shared_rec4);
  if (!last_arrival(a.out.done + (int64_t)kDoneStride * c, last, tid, flag)) return;

  float top = 0.f, bot = 0.f, gw = 0.f;
  if constexpr (PL) {
    const double* plate = FWD ? a.pf.plate : a.pb.plate;
    top = (float)plate[2 * c];
    bot = (float)plate[2 * c + 1];
    if constexpr (BWD) gw = plate_loss_weight(a.pb.F_meas, a.pb.F_target, a.pb.scale, c);
  }
  constexpr int M = (FWD ? 1 : 0) + (BWD ? 1 : 0);
  const float* part[M];
  if constexpr (FWD) part[0] = a.part;
  if constexpr (BWD) part[M - 1] = a.part_b;
  for (int i = s0 + tid; i < s1; i += L) {
    if (i >= s0 + L) sl = shared_slots(a.T.shared_rec[i], a.T.shared_rec4);
    const int64_t g = sl.node;
    float p[3], v[3], s[M][3];
    if constexpr (PL) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        p[d] = a.y[d * N + g];
        if constexpr (BWD) v[d] = a.fbar[d * N + g];
      }
    }
    shared_sums<M, true>(sl, a.T.shared_more, part, s);
    if constexpr (PL && FWD) {
      plate_node_step(p[0], p[1], p[2], s[0][0], s[0][1], s[0][2], top, bot, a.pf.k, a.pf.m,
                      a.pf.y_next, N, g);
    } else if constexpr (PL) {
      plate_node_adjoint(p[2], v[0], v[1], v[2], s[0][0], s[0][1], s[0][2], top, bot, a.pb.k,
                         a.pb.m, gw, a.pb.lam, N, g);
    } else {
      if constexpr (FWD) {
        a.f[g] = s[0][0]; a.f[N + g] = s[0][1]; a.f[2 * N + g] = s[0][2];
      }
      if constexpr (BWD) {
        const float* z = s[M - 1];
        a.ybar[g] = z[0]; a.ybar[N + g] = z[1]; a.ybar[2 * N + g] = z[2];
      }
    }
  }
  // the sums on the last wavefronts, which mostly have no node left
  if constexpr (FWD) {
    if (wave == W - 1) {
      const CellSums cs = cell_sums<true>(a.T, c, lane, a.out.nonfin != nullptr);
      if (lane == 0) {
        if (a.out.energy) a.out.energy[c] = cs.e;
        if (a.out.ninv) a.out.ninv[c] = cs.ni;
        if (a.out.nonfin) a.out.nonfin[c] = cs.nf;
      }
    }
    if constexpr (PL) {
      if (wave == W - 2 && a.pf.force) {
        const double fp = cell_plate_force<true>(a.T, c, lane, a.y, top, a.pf.k);
        if (lane == 0) a.pf.force[c] = fp;
      }
    }
  }
  if constexpr (GRAD) {
    double* const tb = PL ? a.pb.thetabar_acc : a.out.thetabar;
    if (tb) {
      const int R = a.T.n_regions;
      for (int r = W - 1 - wave - (FWD ? 1 : 0); r < R; r += W) {
        if (r < 0) continue;
        const int mt = c * R + r;
        double t3[3];
        slot_theta<true>(a.T, a.tile_acc_b, mt, lane, t3);
        if (lane == 0) {
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            if constexpr (PL)
              tb[3 * (int64_t)mt + q] += a.pb.m64 * t3[q];
            else
              tb[3 * (int64_t)mt + q] = t3[q];
          }
        }
      }
    }
  }
}

// One conjugate-gradient iteration of cell c (at most 2 kThreads nodes) by the
// workgroup of its last tile; red: 1 KB of LDS that the tile no longer uses.  An
// iteration was two launches, each a chain of loads on a few CUs: force curves of
// 16 cells of 1,900 nodes 48.5 -> 44.4 ms.
template <bool SPH>
__device__ __forceinline__ void cg_tail(const WideArgs& a, int c, int tid, int* flag,
                                        double* red) {
  const uint32_t last = (uint32_t)a.T.cell_tile_count[c] - 1;
  const CgArgs& g = a.cg;
  const int64_t n0 = g.node_off[c], n1 = g.node_off[c + 1];
  const double top = g.plate[2 * c], bot = g.plate[2 * c + 1];
  const ShrRange sr = shared_range(g, c, n1);
  if (!last_arrival(a.out.done + (int64_t)kDoneStride * c, last, tid, flag)) return;
  cg_step_regs<2, SPH, true>(g, g.st + kQsState * c, c, n0, n1, top, bot, red, sr);
}

}  // namespace cm
