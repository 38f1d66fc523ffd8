// Tile passes with K wavefronts per tile (forward, adjoint, both at once, and
// either with a plate step), the default launch of every pass.
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
// wavefront -> K), 156 / 650 / 3,250 / 52,000 tiles:
//   forward          17.9 -> 12.5   19.7 -> 15.6   40.9 -> 40.3   478 -> 475 us
//   adjoint          23.3 -> 13.6   24.9 -> 18.0   54.7 -> 48.7   639 -> 630
//   Hessian product  22.1 -> 12.6   23.5 -> 16.5   48.8 -> 43.8   613 -> 575
//   both passes      28.7 -> 15.9   31.2 -> 21.2   70.9 -> 59.8   843 -> 805
// Small launches are bound by the chain of turns (four dependent LDS
// read-modify-writes each), large ones as before by HBM (forward) or by VALU
// issue; two wavefronts share one tile's LDS and need 92 and 120 VGPRs
// (adjoint, both passes) instead of 145 and 162, so more of them are in
// flight.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "kernels.h"
#include "mr_tet.h"
#include "plate.h"

namespace cm {
namespace {

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
  PlateFwd pf;             // used when PL and FWD
  PlateBwd pb;             // used when PL and BWD
};

WideArgs wide_args(const DeviceTables& T, const Range& r, const float* y,
                   const int32_t* ids) {
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
  a.last_slot = T.n_slots > 0 ? (int32_t)T.n_slots - 1 : 0;
  return a;
}

// Loads grouped by data flow: each of these empty statements makes all of its
// values available at once, so that the compiler issues their loads together
// instead of each where its value is first used, one more round trip to
// memory for every step.
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
  const int64_t N = a.N;
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
  // Node gather: the ids of U nodes per thread, then their positions and
  // cotangents, each step's loads issued together (a loop over single nodes
  // waits for both steps every time, and a tile of 283 nodes makes two or
  // three rounds of 64 K threads).  Threads past the last node load a valid
  // one again.
  constexpr int U = K == 4 ? 2 : 3;
  double mu = a.params[mt], kappa = a.params[nm + mt], w = a.params[2 * nm + mt];
  for (int b = 0; b < nl; b += U * 64 * K) {
    const int l0 = b + tid;
    int32_t v[U];
    float yv[U][3], fv[U][3];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = a.ids[min(d.shr_begin + max(min(l0 + u * 64 * K, nl - 1) - d.n_own, 0),
                       a.last_slot)];
    together(v);
    // (the material has arrived when the first addresses are formed)
    asm("" : "+s"(mu), "+s"(kappa), "+s"(w), "+s"(d.own_begin));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int l = min(l0 + u * 64 * K, nl - 1);
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
      const int l = l0 + u * 64 * K;
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
    float h[3][3], hb[3][3];
    double vU = 0.0, gp[3], ge[3], vol = 0.0;
    bool inv = false, bad = false;
    if (on) {
      const float4 p0 = ys[i0], p1 = ys[i1], p2 = ys[i2], p3 = ys[i3];
      double Fd[3][3];
      float F[3][3], Cf[6];
      deformation_gradient(p0, p1, p2, p3, cur.B, Fd, F);
      Scalars sc;
      invariants(Fd, Cf, sc);
      if constexpr (FWD) {
        stress_forces(F, Cf, sc, cur.B, cur.V0, mat, h, vU);
        inv = !(sc.J > 0.0);
        if (!BWD && a.check) {
          float sum = 0.f;
#pragma unroll
          for (int c = 0; c < 3; ++c) sum += h[c][0] + h[c][1] + h[c][2];
          bad = !(isfinite(vU) && isfinite(sum));
        }
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
        adjoint_terms<GRAD>(F, dF, Cf, Kc, sc, cur.B, cur.V0, mat, eb, hb, gp, ge);
        vol = (double)cur.V0;
      }
    }
    if constexpr (FWD) {
      ninv += __popcll(__ballot(inv));
      if (!BWD && a.check) nonfin += __popcll(__ballot(bad));
    }
    if (k + K < d.n_chunks) load_tet(a.chunks + d.chunk_begin + k + K, lane, cur);
    // this chunk's turn: the chunks before it have been added
    // byte offsets of the four vertices' sums, and the sums that slot 3 takes
    // the negative of
    const int o[4] = {12 * i0, 12 * i1, 12 * i2, 12 * i3};
    float hs[3], hbs[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if constexpr (FWD) hs[c] = h[0][c] + h[1][c] + h[2][c];
      if constexpr (BWD) hbs[c] = hb[0][c] + hb[1][c] + hb[2][c];
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
      add_slot<FWD, BWD, false>(fs, gs, o[0], h[0], hb[0]);
      double e = 0.0, tp[3], te[3];
      if constexpr (FWD) e = el[lane];
      if constexpr (GRAD) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          tp[c] = th[64 * c + lane];
          te[c] = th[64 * (3 + c) + lane];
        }
      }
      add_slot<FWD, BWD, false>(fs, gs, o[1], h[1], hb[1]);
      if constexpr (FWD) el[lane] = e + vU;
      if constexpr (GRAD) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          th[64 * c + lane] = fma(vol, gp[c], tp[c]);
          th[64 * (3 + c) + lane] = fma(vol, ge[c], te[c]);
        }
      }
      add_slot<FWD, BWD, false>(fs, gs, o[2], h[2], hb[2]);
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
          a.ybar[g] = gv[0]; a.ybar[N + g] = gv[1]; a.ybar[2 * N + g] = gv[2];
        }
      }
    } else {
      const int64_t s = 3 * ((int64_t)d.shr_begin + l - d.n_own);
      if constexpr (FWD) {
        a.part[s] = fv[0]; a.part[s + 1] = fv[1]; a.part[s + 2] = fv[2];
      }
      if constexpr (BWD) {
        a.part_b[s] = gv[0]; a.part_b[s + 1] = gv[1]; a.part_b[s + 2] = gv[2];
      }
    }
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
        double fp = 0.0;
        for (int i = lane; i < d.n_own; i += 64) fp += plate_top_term(ys[i].z, top, a.pf.k);
        for (int j = lane; j < d.n_shr; j += 64) {
          const float4 p = ys[d.n_own + j];
          if (p.w != 0.f) fp += plate_top_term(p.z, top, a.pf.k);
        }
        fp = wave_sum(fp);
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
  WideArgs a = wide_args(T, r, y, pl.plate ? T.slot_node_first : T.slot_node);
  a.f = f;
  a.part = T.part;
  a.tile_acc = T.tile_acc;
  a.tile_plate = T.tile_plate;
  a.tile_ninv = T.tile_ninv;
  a.tile_nonfin = T.tile_nonfin;
  a.check = check ? 1 : 0;
  a.pf = pl;
  return pl.plate ? wide_k<true, false, true, false>(K, a, st)
                  : wide_k<true, false, false, false>(K, a, st);
}

hipError_t launch_wide_backward(const DeviceTables& T, const Range& r, int K, const float* y,
                                const float* fbar, const double* ebar, float* ybar,
                                hipStream_t st, const CellMask& mask, const PlateBwd& pl,
                                bool grad) {
  WideArgs a = wide_args(T, r, y, T.slot_node);
  if (fbar) a.fbar = fbar;
  a.has_fbar = fbar ? 1 : 0;
  a.ebar = ebar;
  a.ybar = ybar;
  a.part_b = T.part;
  a.tile_acc_b = T.tile_acc;
  a.flags = mask.flags;
  a.flag_stride = mask.stride;
  a.pb = pl;
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
  WideArgs a = wide_args(T, r, y, T.slot_node);
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
  return grad ? wide_k<true, true, false, true>(K, a, st)
              : wide_k<true, true, false, false>(K, a, st);
}

}  // namespace cm
