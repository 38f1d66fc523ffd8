// Launch interface of the per-cell auxiliary kernels (host side): plate
// compression steps and their adjoint, quasi-static compression, shape
// diagnostics.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "kernels.h"

namespace cm {

// Shape diagnostics (Taylor deformation, cell strain): kShapeFields float64
// per cell = volume, centre of mass (3), semi-axes a1 <= a2 <= a3, D, d_max,
// strain.
constexpr int kShapeFields = 10;
// Most candidates of a cell for the search by one workgroup, which keeps them in
// LDS (with their boxes 55 KB).
constexpr int kCellNodes = 4096;
// The workgroup that searches a cell compares alone the pairs of up to kSearchNodes
// remaining nodes, or of an eighth of the candidates if that is more; those of more
// (near-spherical cells, where all remain) it leaves to helpers, up to 32 further
// workgroups of the cell: of 1,024 its share by the square of its candidates, none
// if that is below four (many cells of one size, whose searches fill the chip, and
// the small ones beside large ones).
// Equal spheres, alone -> with helpers, and by the block search: 1 cell of 2,000
// nodes 47 -> 22 us (46), of 9,000 185 -> 41 (54), of 20,000 334 -> 64 (68); 64 cells
// of 2,000 48 -> 25 (58), of 20,000 343 -> 158 (222); 256 of 9,000 197 -> 173 (259).
// Ellipsoids, of which a few nodes remain, pay 0.1 to 0.5 us of 14 to 37.  The line:
// noisy spheres with 250 to 500 nodes left, 64 cells of 2,000 nodes 43 alone, 26
// shared; but with 293 of 3,670 candidates left, which every helper loads again, 64
// cells of 20,000 nodes 41 alone, 60 shared.
constexpr int kSearchNodes = 256;
// Helpers of every cell and, a pair for each of them, the cell and the helper's
// number.
inline void search_helpers(const std::vector<int32_t>& candidates,
                           std::vector<int32_t>* helpers, std::vector<int2>* list) {
  double all = 0.0;
  for (int32_t n : candidates) all += (double)n * n;
  helpers->assign(candidates.size(), 0);
  for (size_t c = 0; c < candidates.size(); ++c) {
    const double n = candidates[c];
    const int share = (int)std::min(32.0, 1024.0 * n * n / all);
    if (candidates[c] <= kSearchNodes || share < 4) continue;
    (*helpers)[c] = share;
  }
  // one of each cell after the other: those of a cell are then mostly on one XCD,
  // whose L2 has its candidates (64 cells of 2,000 nodes 39 -> 25 us)
  for (int i = 0; i < 32; ++i)
    for (size_t c = 0; c < candidates.size(); ++c)
      if (i < (*helpers)[c]) list->push_back(make_int2((int)c, i));
}
// What such a search leaves: the nodes at least sqrt(least2) from the centre.
struct alignas(64) SearchRest {
  double centre[3], least2;
  int32_t left;   // to how many helpers (0: the search is done)
  uint32_t done;  // workgroups of the cell that have arrived
};
// Tables and scratch of a handle's shape diagnostics.  cell_nodes: the
// room of the search of one workgroup per cell, or 0 where some cell has more
// than kCellNodes candidates; then the block search's tables are there: node
// blocks (cell, block) of 256 nodes, with a bounding box (6 float64) each, and
// cand_blocks (cell, row block, column block, first node block of the cell)
// over the candidate blocks of every cell with row <= column.
struct ShapeTables {
  int32_t cell_nodes = 0;
  const int32_t* order = nullptr;       // per cell, node ids, candidates first,
                                        // each part in Morton order
  const int32_t* candidates = nullptr;  // per cell (all its nodes if it has none)
  const uint64_t* chunk_neg = nullptr;  // per chunk: lanes of negative orientation
  const int4* cand_blocks = nullptr;
  int64_t n_cand_blocks = 0;
  const int2* node_blocks = nullptr;
  int64_t n_node_blocks = 0;
  double* mom = nullptr;                // 10 per tile
  int32_t* tile_inv = nullptr;          // per tile
  int32_t* cell_inv = nullptr;          // per cell (block search)
  double* bbox = nullptr;
  unsigned long long* d2max = nullptr;  // per cell
  const int32_t* helpers = nullptr;     // search_helpers of the handle
  const int2* helper = nullptr;
  int32_t n_helpers = 0;
  SearchRest* rest = nullptr;           // per cell (with helpers)
};
size_t shape_lds(int nloc);
hipError_t launch_shape(const DeviceTables& T, const int64_t* node_off,
                        const ShapeTables& S, const float* y, const double* d_ref,
                        double* out, hipStream_t st);

// Quasi-static plate compression (one workgroup per cell): Newton residual,
// one conjugate-gradient iteration, bounded Newton update, plate predictor.
// Per-cell state: kQsState float64 = 0 CG r . z (|r|^2 without
// preconditioner), 1 CG |r_0|^2, 2 CG active,
// 3 Newton |r_N|^2, 4 accepted step scale, 5 |penalty|^2, 6 largest node move
// of the last step, 7 float32 floor of the residual, 8 Pi(y), 9 line-search
// scale, 10 slope r_N . x, 11 not in equilibrium, 12 line search pending,
// 13 max |x|, 14 CG forcing term eta of the Newton step, 15 |r_N|^2 of the
// last residual (for the next forcing term).
constexpr int kQsState = 16;
hipError_t launch_qs_residual(const int64_t* node_off, int64_t N, int32_t n_cells,
                              const float* y, const float* f, const double* energy,
                              const double* plate, double k, double abs_tol,
                              double rel_tol, double step_tol, double floor_factor,
                              double eta_max, int restart, float* r, float* p,
                              float* x, float* rn, double* st, double* force,
                              const float* kel, float* minv, hipStream_t s,
                              const Indenter& ind = Indenter{});
hipError_t launch_qs_ls_start(const int64_t* node_off, int64_t N, int32_t n_cells,
                              float* x, const float* rn, double cap,
                              const float* y, float* yt, double* st, hipStream_t s);
hipError_t launch_qs_ls_accept(const int64_t* node_off, int64_t N, int32_t n_cells,
                               const float* x, const double* plate, double k,
                               const double* energy_t, double armijo,
                               double min_move, float* y, float* yt, double* st,
                               const int32_t* ninv_t, int32_t* ninv, hipStream_t s,
                               const Indenter& ind = Indenter{});
hipError_t launch_qs_noise(const int64_t* node_off, int64_t N, int32_t n_cells,
                           const float* y, float* e, hipStream_t s);
hipError_t launch_qs_floor(const int64_t* node_off, int64_t N, int32_t n_cells,
                           const float* y, const double* plate, double k,
                           const float* e, const float* ybar, double* st,
                           hipStream_t s, const Indenter& ind = Indenter{});
// Start of the adjoint CG solve Hess(Pi) lam = weight_c dF_top/dy (under the
// sphere, of the projected system).
hipError_t launch_qs_adjoint_rhs(const int64_t* node_off, int64_t N, int32_t n_cells,
                                 const float* y, const double* plate, double k,
                                 const double* weight, float* r, float* p, float* x,
                                 double* st, const float* minv, hipStream_t s,
                                 const Indenter& ind = Indenter{});
// With slots set, ybar holds the owned nodes only (a backward tile pass
// without its finalize) and the shared nodes' values are summed from the
// slot partials of those tables (bitwise the finalize's sums).
hipError_t launch_qs_cg(const int64_t* node_off, int64_t N, int32_t n_cells,
                        const float* y, const double* plate, double k,
                        double rel_tol, const float* ybar, float* x, float* r,
                        float* p, float* Ap, double* st, const float* minv,
                        hipStream_t s, const DeviceTables* slots = nullptr,
                        const Indenter& ind = Indenter{});
// Small-strain stiffness blocks (the Newton preconditioner), 6 n_nodes
// floats SoA: xx yy zz xy xz yz; uses the forward scratch.
hipError_t launch_qs_stiffness(const DeviceTables& T, const Range& r, float* kel,
                               hipStream_t s);
hipError_t launch_qs_update(const int64_t* node_off, int64_t N, int32_t n_cells,
                            const float* x, double cap, float* y, double* st,
                            hipStream_t s);
hipError_t launch_qs_any(int32_t n_cells, const double* column, int32_t* flag, hipStream_t s);
hipError_t launch_qs_predict(const int64_t* node_off, int64_t N, int32_t n_cells,
                             const double* plate_old, const double* plate_new,
                             float* y, hipStream_t s);

// Plate compression step and its adjoint (one workgroup per cell).
hipError_t launch_plate_step(const int64_t* node_off, int64_t N, int32_t n_cells,
                             const float* y, const float* f, const double* plate,
                             double k, double m, float* y_next, double* force,
                             hipStream_t st);
hipError_t launch_plate_adjoint(const int64_t* node_off, int64_t N,
                                int32_t n_cells, const float* y,
                                const float* lam_next, const float* ybar_el,
                                const double* plate, double k, double m,
                                const double* F_meas, const double* F_target,
                                double scale, const double* thetabar_el,
                                double* thetabar_acc, int n_regions, float* lam,
                                hipStream_t st);

}  // namespace cm
