// Tile passes with K wavefronts per tile (forward, adjoint, both at once, and
// either with a plate step), the default launch of every pass with more tiles
// than lists.hip takes.
//
// One wavefront per tile (kernels.hip, backward.hip, fused.hip) walks the
// tile's chunks in sequence, at the latency of one chunk after the other (13
// to 25 us for 12 chunks, however small the batch), and holds a second chunk
// of registers for its prefetch and the per-lane sums.  Here the chunks of a
// tile go round its K wavefronts; each evaluates its chunk into registers and
// waits for its turn before it adds the result to the tile's LDS sums.  Turns
// follow the chunk order, so every addition -- the node sums of a chunk's four
// vertex slots, and the per-lane sums of energy and parameter gradient, which
// are in LDS here -- has the place that it has in the one-wavefront pass, and
// every result is bitwise the same.
//
// Measured (768-tet tiles of 2,054-node cells, a call with its finalize, one
// wavefront -> K), 650 / 3,250 / 52,000 tiles:
//   forward          19.7 -> 14.0   40.9 -> 38.5   478 -> 452 us
//   adjoint          24.9 -> 16.7   54.7 -> 47.2   639 -> 608
//   Hessian product  23.5 -> 15.1   48.8 -> 42.0   613 -> 553
//   both passes      31.2 -> 19.6   70.9 -> 58.1   843 -> 791
// (with the slot records of finalize.h, which both would have).
// Small launches are bound by the chain of turns (four dependent LDS
// read-modify-writes each), large ones as before by HBM (forward) or by VALU
// issue; two wavefronts share one tile's LDS and need 92 and 120 VGPRs
// (adjoint, both passes) instead of 145 and 162, so more of them are in
// flight.
#include <hip/hip_runtime.h>

#include "wide.h"

namespace cm {
namespace {

// LDS of a workgroup, in the order of the kernel's carve-up (every part a
// multiple of 16 bytes: nloc is a multiple of 4).
template <int K, bool FWD, bool BWD, bool GRAD>
size_t wide_lds(int nloc) {
  size_t b = (size_t)16 * nloc;
  if (FWD) b += (size_t)12 * nloc + 512;
  if (BWD) b += (size_t)20 * nloc;
  if (GRAD) b += 6 * 512;
  return b + 8 * K + 16;
}

// Adds (NEG: subtracts) v to the force sum and w to the ybar sum at byte
// offset o; the lanes of a vertex slot name distinct nodes (layout.h).
template <bool FWD, bool BWD, bool NEG>
__device__ __forceinline__ void add_slot(float* fs, float* gs, int o, const float v[3],
                                         const float w[3]) {
  float* f = FWD ? reinterpret_cast<float*>(reinterpret_cast<char*>(fs) + o) : nullptr;
  float* g = BWD ? reinterpret_cast<float*>(reinterpret_cast<char*>(gs) + o) : nullptr;
  float a[3], b[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if constexpr (FWD) a[c] = f[c];
    if constexpr (BWD) b[c] = g[c];
  }
  if constexpr (FWD) {
#pragma unroll
    for (int c = 0; c < 3; ++c) f[c] = NEG ? a[c] - v[c] : a[c] + v[c];
  }
  if constexpr (BWD) {
#pragma unroll
    for (int c = 0; c < 3; ++c) g[c] = NEG ? b[c] - w[c] : b[c] + w[c];
  }
}

template <int K, bool FWD, bool BWD, bool PL, bool GRAD>
__global__ __launch_bounds__(64 * K) void wide_kernel(WideArgs a) {
  extern __shared__ float4 lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nloc = a.nloc, nm = a.n_mat;
  // the arguments of the prologue in one round trip
  asm("" : "+s"(a.tile_begin)
      : "s"(a.tiles), "s"(a.chunks), "s"(a.ids), "s"(a.tile_mat), "s"(a.params), "s"(a.y),
        "s"(a.N), "s"(a.last_slot));
  if constexpr (BWD) asm("" : "+s"(a.tile_begin) : "s"(a.fbar), "s"(a.flags));

  const int t = a.tile_begin + xcd_block(blockIdx.x, a.n_tiles);
  TileDesc d = a.tiles[t];
  int mt = a.tile_mat[t];
  // (y.x, y.y, y.z, fbar.x or the plate step's flag) as float4, (fbar.y,
  // fbar.z) as float2, force and ybar sums as packed float3, per lane the
  // energy sum and the sums of V0 gp and V0 ge (three each)
  float4* ys = lds;
  float4* at = ys + nloc;
  double *el = nullptr, *th = nullptr;
  float *fs = nullptr, *gs = nullptr;
  float2* vs = nullptr;
  if constexpr (FWD) {
    el = reinterpret_cast<double*>(at);
    fs = reinterpret_cast<float*>(el + 64);
    at = reinterpret_cast<float4*>(fs + 3 * nloc);
  }
  if constexpr (BWD) {
    gs = reinterpret_cast<float*>(at);
    vs = reinterpret_cast<float2*>(gs + 3 * nloc);
    at = reinterpret_cast<float4*>(vs + nloc);
  }
  if constexpr (GRAD) {
    th = reinterpret_cast<double*>(at);
    at = reinterpret_cast<float4*>(th + 6 * 64);
  }
  int* cnt = reinterpret_cast<int*>(at);  // per wave: inverted, non-finite
  int* turn = cnt + 2 * K;                // the chunk whose turn it is

  // the sums start at zero, while the descriptor is on its way
  for (int i = tid; i < 3 * nloc / 4; i += 64 * K) {
    if constexpr (FWD) reinterpret_cast<float4*>(fs)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (BWD) reinterpret_cast<float4*>(gs)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (tid < 64) {
    if constexpr (FWD) el[tid] = 0.0;
    if constexpr (GRAD) {
#pragma unroll
      for (int c = 0; c < 6; ++c) th[64 * c + tid] = 0.0;
    }
  }
  if (tid == 0) *turn = 0;
  asm("" : "+s"(d.chunk_begin), "+s"(d.n_own), "+s"(mt));
  if (BWD && a.flags && a.flags[(int64_t)d.cell * a.flag_stride] == 0.0) return;

  // the first chunk's loads go out before the node gather
  TetRegs cur{};
  if (wave < d.n_chunks) load_tet(a.chunks + d.chunk_begin + wave, lane, cur);
  const int nl = d.n_own + d.n_shr;
  double mu = a.params[mt], kappa = a.params[nm + mt], w = a.params[2 * nm + mt];
  gather_nodes<64 * K, K == 4 ? 2 : 3, FWD, BWD, PL>(a, d, nl, tid, ys, vs, mu, kappa, w);
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
    const uint2 ix = cur.q;
    const bool on = ix.x != kEmptyLane;
    const int i0 = ix.x & 0xffff, i1 = ix.x >> 16;
    const int i2 = ix.y & 0xffff, i3 = ix.y >> 16;
    TetOut r;
    r.vU = r.vol = 0.0;
    r.inv = r.bad = false;
    if (on) eval_tet<FWD, BWD, GRAD>(cur, ys, vs, mat, eb, a.check, r);
    if constexpr (FWD) {
      ninv += __popcll(__ballot(r.inv));
      if (!BWD && a.check) nonfin += __popcll(__ballot(r.bad));
    }
    if (k + K < d.n_chunks) load_tet(a.chunks + d.chunk_begin + k + K, lane, cur);
    // byte offsets of the four vertices' sums, and the sums that slot 3 takes
    // the negative of
    const int o[4] = {12 * i0, 12 * i1, 12 * i2, 12 * i3};
    float hs[3], hbs[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if constexpr (FWD) hs[c] = r.h[0][c] + r.h[1][c] + r.h[2][c];
      if constexpr (BWD) hbs[c] = r.hb[0][c] + r.hb[1][c] + r.hb[2][c];
    }
    // This chunk's turn: the chunks before it have been added.  All K
    // wavefronts of the workgroup are resident and each takes its chunks in
    // order, so chunk k - 1, whose turn depends on chunk k - 2 and so on down
    // to chunk 0, is always being worked on: every wait ends.  The wavefront
    // whose turn it is goes before those that still evaluate theirs.
    while (__hip_atomic_load(turn, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != k)
      __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_s_setprio(3);
    if (on) {
      // vertex slots in order, each one read-modify-write of both sums; the
      // per-lane sums go between, where they wait for nothing of their own
      add_slot<FWD, BWD, false>(fs, gs, o[0], r.h[0], r.hb[0]);
      double e = 0.0, tp[3], te[3];
      if constexpr (FWD) e = el[lane];
      if constexpr (GRAD) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          tp[c] = th[64 * c + lane];
          te[c] = th[64 * (3 + c) + lane];
        }
      }
      add_slot<FWD, BWD, false>(fs, gs, o[1], r.h[1], r.hb[1]);
      if constexpr (FWD) el[lane] = e + r.vU;
      if constexpr (GRAD) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          th[64 * c + lane] = fma(r.vol, r.gp[c], tp[c]);
          th[64 * (3 + c) + lane] = fma(r.vol, r.ge[c], te[c]);
        }
      }
      add_slot<FWD, BWD, false>(fs, gs, o[2], r.h[2], r.hb[2]);
      add_slot<FWD, BWD, true>(fs, gs, o[3], hs, hbs);
    }
    if (lane == 0)
      __hip_atomic_store(turn, k + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_s_setprio(0);
  }
  if constexpr (FWD) {
    if (lane == 0) {
      cnt[2 * wave] = ninv;
      cnt[2 * wave + 1] = nonfin;
    }
  }
  __syncthreads();

  for (int l = tid; l < nl; l += 64 * K) {
    float fv[3], gv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if constexpr (FWD) fv[c] = fs[3 * l + c];
      if constexpr (BWD) gv[c] = gs[3 * l + c];
    }
    store_node<FWD, BWD, PL>(a, d, l, fv, gv, ys, vs, top, bot, gw);
  }
  if constexpr (GRAD) {
    for (int c = K - 1 - wave; c < 3; c += K) {
      const double v = wave_sum(fma(0.5 * eb, th[64 * (3 + c) + lane], -th[64 * c + lane]));
      if (lane == 0) a.tile_acc_b[3 * (int64_t)t + c] = v;
    }
  }
  if constexpr (FWD) {
    if (wave == K - 1) {
      const double eacc = wave_sum(el[lane]);
      if constexpr (PL) {
        const double fp = plate_share(d, ys, lane, top, a.pf.k);
        if (lane == 0) a.tile_plate[t] = fp;
      }
      if (lane == 0) {
        int ni = 0, nf = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          ni += cnt[2 * k];
          nf += cnt[2 * k + 1];
        }
        a.tile_acc[t] = eacc;
        a.tile_ninv[t] = ni;
        if (!BWD && a.check) a.tile_nonfin[t] = nf;
      }
    }
  }
}

template <int K, bool FWD, bool BWD, bool PL, bool GRAD>
hipError_t wide_go(const WideArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((wide_kernel<K, FWD, BWD, PL, GRAD>), dim3(a.n_tiles), dim3(64 * K),
                     (wide_lds<K, FWD, BWD, GRAD>(a.nloc)), st, a);
  return hipGetLastError();
}

template <bool FWD, bool BWD, bool PL, bool GRAD>
hipError_t wide_k(int K, const WideArgs& a, hipStream_t st) {
  return K == 4 ? wide_go<4, FWD, BWD, PL, GRAD>(a, st) : wide_go<2, FWD, BWD, PL, GRAD>(a, st);
}

}  // namespace

// Two wavefronts per tile were never slower than one, up to 52,000 tiles (the
// shared-mesh batch of 53,248, whose chunks come from the caches: 770 us
// both ways).  With few tiles the chain of a tile's chunks is what lasts, and
// four wavefronts shorten it further: K = 4 / 2 at 1,027 tiles 18.7 / 20.4 us
// forward, 23.1 / 25.4 adjoint, 28.7 / 29.3 both; at 1,495 (six per CU) 22.3
// / 24.4, 28.4 / 30.5, 35.1 / 36.2; at 1,690 26.2 / 25.3, 29.8 / 31.8, 37.6 /
// 37.9; at 2,340 31.6 / 31.4, 39.0 / 38.5, 48.2 / 49.3.  The Hessian-vector
// product (fewer registers) gains from four up to 6,500 tiles (81.0 / 82.3
// us; 9,750: 118.0 / 117.4).
int wide_waves(const Range& r, const LaunchCfg& cfg, size_t lds, bool hvp) {
  if (cfg.waves != 1 || cfg.blocks != 0) return 0;
  // the sums of a workgroup beside the tile's nodes (wide_lds)
  if (lds + 4096 > 65536) return 0;
  return r.tile_end - r.tile_begin <= (hvp ? 6500 : 1536) ? 4 : 2;
}

hipError_t launch_wide_forward(const DeviceTables& T, const Range& r, int K, const float* y,
                               float* f, hipStream_t st, const PlateFwd& pl, bool check) {
  const WideArgs a = forward_args(T, r, y, f, pl, check);
  return pl.plate ? wide_k<true, false, true, false>(K, a, st)
                  : wide_k<true, false, false, false>(K, a, st);
}

hipError_t launch_wide_backward(const DeviceTables& T, const Range& r, int K, const float* y,
                                const float* fbar, const double* ebar, float* ybar,
                                hipStream_t st, const CellMask& mask, const PlateBwd& pl,
                                bool grad) {
  const WideArgs a = backward_args(T, r, y, fbar, ebar, ybar, mask, pl);
  if (pl.plate)
    return grad ? wide_k<false, true, true, true>(K, a, st)
                : wide_k<false, true, true, false>(K, a, st);
  return grad ? wide_k<false, true, false, true>(K, a, st)
              : wide_k<false, true, false, false>(K, a, st);
}

hipError_t launch_wide_forward_backward(const DeviceTables& T, const DeviceTables& Tb,
                                        const Range& r, int K, const float* y, float* f,
                                        const float* fbar, const double* ebar, float* ybar,
                                        hipStream_t st, bool grad) {
  const WideArgs a = forward_backward_args(T, Tb, r, y, f, fbar, ebar, ybar);
  return grad ? wide_k<true, true, false, true>(K, a, st)
              : wide_k<true, true, false, false>(K, a, st);
}

}  // namespace cm
