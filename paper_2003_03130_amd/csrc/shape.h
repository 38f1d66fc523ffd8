// Shape diagnostics: tables, scratch and launch (shape.hip).
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

// The workgroup that searches a cell of up to kSearchAlone candidates compares the
// remaining nodes' pairs alone: so it takes no longer than the block search did even
// for a sphere, of which all remain (1 cell of 2,000 nodes 45 us, 46 by that).  In
// larger cells it does so for up to kSearchNodes remaining nodes, or an eighth of the
// candidates if that is more, and leaves the pairs of more of them to helpers, up to 32
// further workgroups of the cell: of 1,024 its share by the square of its candidates,
// none if that is below four (many cells of one size, whose searches fill the chip,
// and the small ones beside large ones).
// Equal spheres, alone -> with helpers, and by the block search: 1 cell of 3,800 nodes
// 87 -> 26 us (49), of 9,000 185 -> 41 (54), of 20,000 334 -> 63 (68); 64 cells of 9,000
// 190 -> 72 (110), of 20,000 343 -> 156 (222); 256 of 9,000 197 -> 173 (259).
// Ellipsoids, of which a few nodes remain, pay 0.1 to 0.4 us of 15 to 53.  The line of
// kSearchNodes: noisy spheres with 250 to 500 nodes left, 64 cells of 2,000 nodes 43
// alone, 26 shared; but with 293 of 3,670 candidates left, which every helper loads
// again, 64 cells of 20,000 nodes 41 alone, 60 shared.
constexpr int kSearchAlone = 768;
constexpr int kSearchNodes = 256;

// Helpers of every cell and, a pair for each of them, the cell and the helper's
// number.
inline void search_helpers(const std::vector<int32_t>& candidates,
                           std::vector<int32_t>* helpers, std::vector<int2>* list) {
  double all = 0.0;
  for (int32_t n : candidates) all += (double)n * n;
  helpers->assign(candidates.size(), 0);
  std::vector<int32_t> cells;
  for (size_t c = 0; c < candidates.size(); ++c) {
    const double n = candidates[c];
    const int share = (int)std::min(32.0, 1024.0 * n * n / all);
    if (candidates[c] <= kSearchAlone || share < 4) continue;
    (*helpers)[c] = share;
    cells.push_back((int32_t)c);
  }
  // one of each cell after the other: those of a cell are then mostly on one XCD,
  // whose L2 has its candidates (64 cells of 2,000 nodes 39 -> 25 us)
  for (int i = 0; i < 32; ++i)
    for (int32_t c : cells)
      if (i < (*helpers)[c]) list->push_back(make_int2(c, i));
}

// What such a search leaves: the nodes at least sqrt(least2) from the centre.
struct alignas(64) SearchRest {
  double centre[3], least2;
  int32_t left;   // to how many helpers (0: the search is done)
  uint32_t done;  // helpers of the cell that have arrived
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

}  // namespace cm
