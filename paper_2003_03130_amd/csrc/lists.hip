// Tile passes with a wavefront per chunk, for launches of about one tile per
// CU or fewer.
//
// With several wavefronts per tile (wide.hip) a small launch is bound by the
// chain of turns in which they add their chunks to the tile's sums (12 turns
// of 830 cycles, 1,200 in the fused pass, two thirds of the kernel).  Here no
// wavefront waits for another's chunk: every one writes its tetrahedra's
// contributions to LDS (48 bytes per tetrahedron and output), and after one
// barrier a thread per tile node adds up the node's contributions from a list
// in (chunk, vertex slot) order (list_tables in prep.h).  That is the order in
// which the other passes add them, and the per-tile sums are likewise added
// chunk by chunk on the lane that forms them there: results are bitwise the
// same.  What remains is the evaluation at the issue rate of one CU and the
// loads before it: at 156 tiles (2,054-node cells, a call with its finalize)
// forward 11.4 -> 10.1 us, adjoint 12.0 -> 10.5, Hessian-vector product 11.2 ->
// 9.9, both passes 14.8 -> 12.1; with the cells' sums formed in the pass (tail.h)
// forward 8.6, adjoint 9.9, product 9.1.  The lists cost 8 bytes per tetrahedron and the LDS holds
// one tile per CU in the passes with a parameter gradient, so launches that
// fill the chip keep the other passes.
#include <hip/hip_runtime.h>

#include "tail.h"

namespace cm {
namespace {

// LDS of a workgroup, in the order of the kernel's carve-up (every part a
// multiple of 16 bytes: nloc is a multiple of 4); C: most chunks of a tile.
size_t list_lds(int nloc, const ListTables& lt, bool fwd, bool bwd, bool grad) {
  const size_t L = 64 * (size_t)lt.chunks;
  size_t b = (size_t)16 * nloc + (size_t)16 * lt.stride16;
  if (fwd) b += L * 8 + L * 48 + 16;
  if (bwd) b += L * 48 + 16 + (size_t)8 * nloc;
  if (grad) b += L * 48 + L * 4;
  return b + 128;
}

// The four vertex contributions of one tetrahedron (vertex slot 3 takes the
// negative sum of the others).
__device__ __forceinline__ void put_contributions(float* o, const float h[3][3]) {
  float4* p = reinterpret_cast<float4*>(o);
  p[0] = make_float4(h[0][0], h[0][1], h[0][2], h[1][0]);
  p[1] = make_float4(h[1][1], h[1][2], h[2][0], h[2][1]);
  p[2] = make_float4(h[2][2], -(h[0][0] + h[1][0] + h[2][0]),
                     -(h[0][1] + h[1][1] + h[2][1]), -(h[0][2] + h[1][2] + h[2][2]));
}

template <int K, bool FWD, bool BWD, bool PL, bool GRAD, Tail TAIL>
__global__ __launch_bounds__(64 * K) void list_kernel(WideArgs a) {
  extern __shared__ float4 lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nloc = a.nloc, nm = a.n_mat, L = 64 * a.lists.chunks, G = a.lists.groups;
  // the arguments of the prologue in one round trip
  asm("" : "+s"(a.tile_begin)
      : "s"(a.tiles), "s"(a.chunks), "s"(a.ids), "s"(a.tile_mat), "s"(a.params), "s"(a.y),
        "s"(a.N), "s"(a.last_slot), "s"(a.lists.blocks), "s"(a.lists.stride16));
  if constexpr (BWD) asm("" : "+s"(a.tile_begin) : "s"(a.fbar), "s"(a.flags));

  const int t = a.tile_begin + xcd_block(blockIdx.x, a.n_tiles);
  TileDesc d = a.tiles[t];
  int mt = a.tile_mat[t];
  // positions (and fbar.x, or the plate step's flag), the tile's lists, then
  // the contributions of all its chunks
  float4* ys = lds;
  uint4* blk = reinterpret_cast<uint4*>(ys + nloc);
  float4* at = reinterpret_cast<float4*>(blk + a.lists.stride16);
  double* el = nullptr;  // energies
  float* hf = nullptr;   // force contributions, then a zero one
  float* hb = nullptr;   // ybar contributions, then a zero one
  double* th = nullptr;  // parameter-gradient terms: gp (3), ge (3)
  float* vol = nullptr;
  float2* vs = nullptr;  // fbar.yz
  if constexpr (FWD) {
    el = reinterpret_cast<double*>(at);
    hf = reinterpret_cast<float*>(el + L);
    at = reinterpret_cast<float4*>(hf + 12 * L + 4);
  }
  if constexpr (BWD) {
    hb = reinterpret_cast<float*>(at);
    vs = reinterpret_cast<float2*>(hb + 12 * L + 4);
    at = reinterpret_cast<float4*>(vs + nloc);
  }
  if constexpr (GRAD) {
    th = reinterpret_cast<double*>(at);
    vol = reinterpret_cast<float*>(th + 6 * L);
    at = reinterpret_cast<float4*>(vol + L);
  }
  int* cnt = reinterpret_cast<int*>(at);  // per wave: inverted, non-finite

  {
    const uint4* src = a.lists.blocks + (int64_t)(t / a.copies) * a.lists.stride16;
    for (int i = tid; i < a.lists.stride16; i += 64 * K) blk[i] = src[i];
  }
  if (tid < 3) {
    if constexpr (FWD) hf[12 * L + tid] = 0.f;
    if constexpr (BWD) hb[12 * L + tid] = 0.f;
  }
  asm("" : "+s"(d.chunk_begin), "+s"(d.n_own), "+s"(mt));
  if (BWD && a.flags && a.flags[(int64_t)d.cell * a.flag_stride] == 0.0) return;

  TetRegs cur{};
  if (wave < d.n_chunks) load_tet(a.chunks + d.chunk_begin + wave, lane, cur);
  const int nl = d.n_own + d.n_shr;
  double mu = a.params[mt], kappa = a.params[nm + mt], w = a.params[2 * nm + mt];
  gather_nodes<64 * K, 1, FWD, BWD, PL>(a, d, nl, tid, ys, vs, mu, kappa, w);
  const Material mat{w * mu, (1.0 - w) * mu, kappa};
  const double eb = (GRAD && a.ebar) ? a.ebar[d.cell] : 0.0;
  float top = 0.f, bot = 0.f, gw = 0.f;
  if constexpr (PL) {
    const double* plate = FWD ? a.pf.plate : a.pb.plate;
    top = (float)plate[2 * d.cell];
    bot = (float)plate[2 * d.cell + 1];
    if constexpr (BWD) gw = plate_loss_weight(a.pb.F_meas, a.pb.F_target, a.pb.scale, d.cell);
  }
  __syncthreads();

  int ninv = 0, nonfin = 0;
  for (int k = wave; k < d.n_chunks; k += K) {
    TetOut r;
    r.vU = r.vol = 0.0;
    r.inv = r.bad = false;
#pragma unroll
    for (int c = 0; c < 3; ++c) r.gp[c] = r.ge[c] = 0.0;
    const int o = 64 * k + lane;
    if (cur.q.x != kEmptyLane) {
      eval_tet<FWD, BWD, GRAD>(cur, ys, vs, mat, eb, a.check, r);
      if constexpr (FWD) put_contributions(hf + 12 * o, r.h);
      if constexpr (BWD) put_contributions(hb + 12 * o, r.hb);
    }
    // (a lane without a tetrahedron: no list names it, its terms are zero)
    if constexpr (FWD) {
      el[o] = r.vU;
      ninv += __popcll(__ballot(r.inv));
      if (!BWD && a.check) nonfin += __popcll(__ballot(r.bad));
    }
    if constexpr (GRAD) {
      vol[o] = (float)r.vol;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        th[c * L + o] = r.gp[c];
        th[(3 + c) * L + o] = r.ge[c];
      }
    }
    if (k + K < d.n_chunks) load_tet(a.chunks + d.chunk_begin + k + K, lane, cur);
  }
  if constexpr (FWD) {
    if (lane == 0) {
      cnt[2 * wave] = ninv;
      cnt[2 * wave + 1] = nonfin;
    }
  }
  __syncthreads();

  const uint16_t* order = reinterpret_cast<const uint16_t*>(blk);
  const uint32_t* lists = reinterpret_cast<const uint32_t*>(order + 64 * G);
  const uint2* recs = reinterpret_cast<const uint2*>(blk + 8 * G + ((G + 3) >> 2));
  for (int g = wave; g < G; g += K) {
    const uint32_t fc = __builtin_amdgcn_readfirstlane(lists[g]);
    const int l = order[64 * g + lane];
    const uint2* p = recs + 64 * (fc & 0xffff) + lane;
    float fv[3] = {0.f, 0.f, 0.f}, gv[3] = {0.f, 0.f, 0.f};
    for (int n = fc >> 16; n > 0; --n, p += 64) {
      const uint2 rc = *p;
      const int i[4] = {3 * (int)(rc.x & 0xffff), 3 * (int)(rc.x >> 16),
                        3 * (int)(rc.y & 0xffff), 3 * (int)(rc.y >> 16)};
      float v[4][3], z[4][3];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if constexpr (FWD) v[j][c] = hf[i[j] + c];
          if constexpr (BWD) z[j][c] = hb[i[j] + c];
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if constexpr (FWD) fv[c] += v[j][c];
          if constexpr (BWD) gv[c] += z[j][c];
        }
      }
    }
    if (l < nl)
      store_node<FWD, BWD, PL, TAIL != kNoTail, (TAIL > kCellSums)>(a, d, l, fv, gv, ys, vs,
                                                                    top, bot, gw);
  }
  // per-tile sums on the last wavefronts, chunk by chunk on each lane
  if constexpr (FWD) {
    if (wave == K - 1) {
      double e = 0.0;
      for (int k = 0; k < d.n_chunks; ++k) e += el[64 * k + lane];
      e = wave_sum(e);
      if (lane == 0) {
        int ni = 0, nf = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          ni += cnt[2 * k];
          nf += cnt[2 * k + 1];
        }
        store_as<TAIL != kNoTail>(a.tile_acc + t, e);
        store_as<TAIL != kNoTail>(a.tile_ninv + t, ni);
        if (!BWD && a.check) store_as<TAIL != kNoTail>(a.tile_nonfin + t, nf);
      }
    }
    if constexpr (PL) {
      if (wave == K - 2) {
        const double fp = plate_share(d, ys, lane, top, a.pf.k);
        if (lane == 0) store_as<TAIL != kNoTail>(a.tile_plate + t, fp);
      }
    }
  }
  if constexpr (GRAD) {
    const int c = K - 2 - wave;
    if (c >= 0 && c < 3) {
      double p = 0.0, e = 0.0;
      for (int k = 0; k < d.n_chunks; ++k) {
        const double v = (double)vol[64 * k + lane];
        p = fma(v, th[c * L + 64 * k + lane], p);
        e = fma(v, th[(3 + c) * L + 64 * k + lane], e);
      }
      const double s = wave_sum(fma(0.5 * eb, e, -p));
      if (lane == 0) store_as<TAIL != kNoTail>(a.tile_acc_b + 3 * (int64_t)t + c, s);
    }
  }
  if constexpr (TAIL == kCellSums) cell_tail<64 * K, FWD, BWD, PL, GRAD>(a, d.cell, tid, cnt);
  if constexpr (TAIL > kCellSums) {
    static_assert(64 * K == kThreads, "threads of a conjugate-gradient iteration");
    cg_tail<TAIL == kCgSphere>(a, d.cell, tid, cnt, reinterpret_cast<double*>(lds));
  }
}

template <int K, bool FWD, bool BWD, bool PL, bool GRAD, Tail TAIL>
hipError_t list_go(const WideArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((list_kernel<K, FWD, BWD, PL, GRAD, TAIL>), dim3(a.n_tiles), dim3(64 * K),
                     list_lds(a.nloc, a.lists, FWD, BWD, GRAD), st, a);
  return hipGetLastError();
}

// 16 wavefronts: 12 or 8 were slower (both passes at 156 tiles 12.1, 12.2 and
// 13.0 us, adjoint 10.5, 11.4, 11.8).
template <bool FWD, bool BWD, bool PL, bool GRAD>
hipError_t list_run(const WideArgs& a, hipStream_t st) {
  if (a.out.done) return list_go<16, FWD, BWD, PL, GRAD, kCellSums>(a, st);
  return list_go<16, FWD, BWD, PL, GRAD, kNoTail>(a, st);
}

}  // namespace

// One tile per CU.  With turns -> with lists: 247 tiles 11.8 -> 10.1 us forward,
// 12.5 -> 10.9 adjoint, 15.0 -> 12.3 both; at 325 tiles, two on some CUs,
// 12.6 -> 13.1, 13.7 -> 15.8 and 16.2 -> 19.0.  Never slower below, down to one
// tile and to tiles of one chunk.
int64_t list_tiles() { return 256; }

bool use_lists(const DeviceTables& T, const Range& r, const LaunchCfg& cfg, bool fwd, bool bwd,
               bool grad) {
  return T.lists.blocks && cfg.waves == 1 && cfg.blocks == 0 &&
         r.tile_end - r.tile_begin <= list_tiles() &&
         list_lds(T.nloc, T.lists, fwd, bwd, grad) <= 163840;
}

// Most shared nodes of a cell whose sums one workgroup forms in place of a finalize
// launch, finalize -> tail: at 1,512 all single passes are faster, 11.1, 11.4, 11.3
// -> 8.9, 10.6, 9.4 us (forward, adjoint, Hessian-vector product); at 2,607 the
// adjoint and the product are slower, 11.3, 10.8 -> 12.1, 11.4; the forward, which
// has the same limit, still gains there, 11.0 -> 10.4, and loses at 4,820, 10.8 ->
// 14.6.  Both passes at once gain at 331, 12.5 -> 11.8, and lose at 1,040, 12.0 ->
// 12.6; nothing was measured between.  Passes with more than 256 tiles keep the
// finalize: several workgroups share a CU there, and the arrival of a tile's
// stores holds up the next tile (forward of 650 tiles 13.9 -> 18.4).
constexpr int kTailShared = 2048, kTailSharedBoth = 512;

bool use_tail(const DeviceTables& T, const Range& r, const LaunchCfg& cfg, bool fwd, bool bwd,
              bool grad) {
  return T.cell_done && r.tile_end > r.tile_begin && use_lists(T, r, cfg, fwd, bwd, grad) &&
         T.max_cell_shared <= (fwd && bwd ? kTailSharedBoth : kTailShared);
}

hipError_t launch_list_forward(const DeviceTables& T, const Range& r, const float* y, float* f,
                               hipStream_t st, const PlateFwd& pl, bool check,
                               const CellOut& out) {
  WideArgs a = forward_args(T, r, y, f, pl, check, out);
  return pl.plate ? list_run<true, false, true, false>(a, st)
                  : list_run<true, false, false, false>(a, st);
}

hipError_t launch_list_backward(const DeviceTables& T, const Range& r, const float* y,
                                const float* fbar, const double* ebar, float* ybar,
                                hipStream_t st, const CellMask& mask, const PlateBwd& pl,
                                bool grad, const CellOut& out) {
  WideArgs a = backward_args(T, r, y, fbar, ebar, ybar, mask, pl, out);
  if (pl.plate)
    return grad ? list_run<false, true, true, true>(a, st)
                : list_run<false, true, true, false>(a, st);
  return grad ? list_run<false, true, false, true>(a, st)
              : list_run<false, true, false, false>(a, st);
}

hipError_t launch_list_forward_backward(const DeviceTables& T, const DeviceTables& Tb,
                                        const Range& r, const float* y, float* f,
                                        const float* fbar, const double* ebar, float* ybar,
                                        hipStream_t st, bool grad, const CellOut& out) {
  WideArgs a = forward_backward_args(T, Tb, r, y, f, fbar, ebar, ybar, out);
  return grad ? list_run<true, true, false, true>(a, st)
              : list_run<true, true, false, false>(a, st);
}

// Cells of more nodes take the kernel of their own, which holds four nodes a
// thread or streams them.
bool use_cg_tail(const DeviceTables& T, const Range& r, const LaunchCfg& cfg) {
  return T.cell_done && r.tile_end > r.tile_begin &&
         use_lists(T, r, cfg, false, true, false) && T.max_cell_nodes <= 2 * kThreads;
}

hipError_t launch_qs_cg_iteration(const DeviceTables& T, const Range& r,
                                  const int64_t* node_off, const float* y,
                                  const double* plate, double k, double rel_tol, float* ybar,
                                  float* x, float* rv, float* p, float* Ap, double* state,
                                  const float* minv, const CellMask& mask, hipStream_t st,
                                  const Indenter& ind) {
  CellOut out;
  out.done = T.cell_done;
  WideArgs a = backward_args(T, r, y, p, nullptr, ybar, mask, PlateBwd{}, out);
  a.cg = cg_args(node_off, T.n_nodes, y, plate, k, rel_tol, ybar, x, rv, p, Ap, state, minv, &T,
                 ind);
  return ind.R > 0.0 ? list_go<16, false, true, false, false, kCgSphere>(a, st)
                        : list_go<16, false, true, false, false, kCgPlates>(a, st);
}

}  // namespace cm
