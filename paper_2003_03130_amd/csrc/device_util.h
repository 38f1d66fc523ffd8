// Device helpers shared by the forward and backward kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace cm {

// LDS written by one lane is read by other lanes of the same wavefront only
// after this point: LDS instructions of a wavefront execute in order, so a
// compiler-level fence plus a wave barrier is enough.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Stores and loads past the caches that other XCDs do not see: relaxed atomics
// of device scope (such a store has arrived once the wavefront has waited for
// it).
template <class T>
__device__ __forceinline__ void device_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T device_load(const T* p) {
  return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Three floats at base + 3 i (bytes below 4 GiB) in one access.
typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
constexpr int kDeviceScope = 16;  // the instructions' sc1 bit

__device__ __forceinline__ __amdgpu_buffer_rsrc_t device_rsrc(const float* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, -1, 0x00027000);
}
__device__ __forceinline__ void device_load3(const float* base, int32_t i, float (&v)[3]) {
  const u32x3_t r = __builtin_amdgcn_raw_buffer_load_b96(device_rsrc(base), 12 * i, 0,
                                                         kDeviceScope);
  v[0] = __uint_as_float(r.x);
  v[1] = __uint_as_float(r.y);
  v[2] = __uint_as_float(r.z);
}
__device__ __forceinline__ void device_store3(float* base, int32_t i, const float v[3]) {
  const u32x3_t r = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2])};
  __builtin_amdgcn_raw_buffer_store_b96(r, device_rsrc(base), 12 * i, 0, kDeviceScope);
}
template <bool DEVICE, class T>
__device__ __forceinline__ void store_as(T* p, T v) {
  if constexpr (DEVICE)
    device_store(p, v);
  else
    *p = v;
}
template <bool DEVICE, class T>
__device__ __forceinline__ T load_as(const T* p) {
  if constexpr (DEVICE) return device_load(p);
  return *p;
}

// Whether this workgroup is the last of `last` + 1 that count themselves in on
// *done, uniform over the workgroup; what they stored with device scope has then
// arrived.  The counter is zero again after the last.  flag: an int of LDS that
// nothing else uses any more.
__device__ __forceinline__ bool last_arrival(uint32_t* done, uint32_t last, int tid, int* flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) *flag = atomicInc(done, last) == last;
  __syncthreads();
  return *flag != 0;
}

// One lane's tetrahedron of a chunk: packed local indices, B and V0.
struct TetRegs {
  uint2 q;
  float B[9];
  float V0;
};

// Chunks are read once per pass: three 16-byte loads per lane, each row of
// the chunk 1,024 contiguous bytes (16-byte loads stream at about 1.5 times
// the rate of 4-byte ones), non-temporal so that the chunk stream does not
// displace the node data that neighbouring tiles reuse from the caches.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void load_tet(const TetChunk* ch, int lane,
                                         TetRegs& r) {
  const u32x4_t va = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(ch->a[lane]));
  const f32x4_t vb = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(ch->b[lane]));
  const f32x4_t vc = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(ch->c[lane]));
  r.q.x = va.x;
  r.q.y = va.y;
  r.V0 = __uint_as_float(va.z);
  r.B[0] = __uint_as_float(va.w);
  r.B[1] = vb.x; r.B[2] = vb.y; r.B[3] = vb.z; r.B[4] = vb.w;
  r.B[5] = vc.x; r.B[6] = vc.y; r.B[7] = vc.z; r.B[8] = vc.w;
}

// Adds the contributions h[0..2] of vertex slots 0..2 and -(h0 + h1 + h2) of
// slot 3 to the accumulators acc(i_s) (acc maps a tile-local node index to
// its three accumulator floats).  The layout guarantees that the active
// lanes of the wave name distinct nodes within each slot, so each slot is
// one LDS read and one LDS write per lane with no races; slots are processed
// in order (LDS instructions of a wavefront execute in order).
template <class Acc>
__device__ __forceinline__ void lds_accumulate(Acc acc, int i0, int i1, int i2,
                                               int i3, const float h[3][3]) {
  float* a = acc(i0);
  a[0] += h[0][0]; a[1] += h[0][1]; a[2] += h[0][2];
  a = acc(i1);
  a[0] += h[1][0]; a[1] += h[1][1]; a[2] += h[1][2];
  a = acc(i2);
  a[0] += h[2][0]; a[1] += h[2][1]; a[2] += h[2][2];
  a = acc(i3);
  a[0] -= h[0][0] + h[1][0] + h[2][0];
  a[1] -= h[0][1] + h[1][1] + h[2][1];
  a[2] -= h[0][2] + h[1][2] + h[2][2];
}

// Runs body(regs) over the n chunks ch[0..n) with the next chunk's loads in
// flight while the current one is evaluated; two register sets alternate, so
// no register copies are needed between chunks.  Every call site of body is
// reached with one fixed set of outstanding loads (one chunk in flight, or
// none at the last chunk), so the compiler waits only for the chunk that
// body reads.
// As for_each_chunk, with the first chunk's registers ra loaded by the
// caller (before the tile's nodes are staged, so that its loads are in
// flight meanwhile).
template <class Body>
__device__ __forceinline__ void for_each_chunk_from(const TetChunk* ch, int n,
                                                    int lane, TetRegs ra, Body body) {
  if (n <= 0) return;
  TetRegs rb;
  for (int k = 0;; k += 2) {
    if (k + 1 >= n) {
      body(ra);
      return;
    }
    load_tet(ch + k + 1, lane, rb);
    body(ra);
    if (k + 2 >= n) {
      body(rb);
      return;
    }
    load_tet(ch + k + 2, lane, ra);
    body(rb);
  }
}

template <class Body>
__device__ __forceinline__ void for_each_chunk(const TetChunk* ch, int n,
                                               int lane, Body body) {
  if (n <= 0) return;
  TetRegs ra;
  load_tet(ch, lane, ra);
  for_each_chunk_from(ch, n, lane, ra, body);
}

// Butterfly over the wavefront with offsets 32, 16, 8, 4, 2, 1: every lane ends
// with op over all lanes, in the order of that butterfly (op commutative).  The
// exchanges are register moves -- half-wave and row swaps, then rotations
// inside a row of 16, which reach lane ^ 8, and lane ^ 4, 2, 1 once the values
// repeat every 8, 4, 2 lanes -- instead of shuffles through LDS: about 150
// cycles for a double instead of 700.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int kRowRor8 = 0x128, kRowRor4 = 0x124, kQuadXor2 = 0x4e, kQuadXor1 = 0xb1;

template <int CTRL>
__device__ __forceinline__ int dpp_of(int v) {
  return (int)dpp_move<CTRL>((uint32_t)v);
}
template <int CTRL>
__device__ __forceinline__ float dpp_of(float v) {
  return __uint_as_float(dpp_move<CTRL>(__float_as_uint(v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_of(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  return __longlong_as_double(
      (long long)((uint64_t)dpp_move<CTRL>((uint32_t)(b >> 32)) << 32 |
                  dpp_move<CTRL>((uint32_t)b)));
}

// (a, b) = the values of a lane and of its partner, in one order on both.
__device__ __forceinline__ void swap32(int v, int& a, int& b) {
  const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  a = (int)r[0];
  b = (int)r[1];
}
__device__ __forceinline__ void swap16(int v, int& a, int& b) {
  const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
  a = (int)r[0];
  b = (int)r[1];
}
__device__ __forceinline__ void swap32(float v, float& a, float& b) {
  int i, j;
  swap32(__float_as_int(v), i, j);
  a = __int_as_float(i);
  b = __int_as_float(j);
}
__device__ __forceinline__ void swap16(float v, float& a, float& b) {
  int i, j;
  swap16(__float_as_int(v), i, j);
  a = __int_as_float(i);
  b = __int_as_float(j);
}
__device__ __forceinline__ double join(int hi, int lo) {
  return __longlong_as_double((long long)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo));
}
__device__ __forceinline__ void swap32(double v, double& a, double& b) {
  const uint64_t w = (uint64_t)__double_as_longlong(v);
  int l0, l1, h0, h1;
  swap32((int)(uint32_t)w, l0, l1);
  swap32((int)(uint32_t)(w >> 32), h0, h1);
  a = join(h0, l0);
  b = join(h1, l1);
}
__device__ __forceinline__ void swap16(double v, double& a, double& b) {
  const uint64_t w = (uint64_t)__double_as_longlong(v);
  int l0, l1, h0, h1;
  swap16((int)(uint32_t)w, l0, l1);
  swap16((int)(uint32_t)(w >> 32), h0, h1);
  a = join(h0, l0);
  b = join(h1, l1);
}

// The last four offsets: op over each row of 16 lanes.
template <class T, class Op>
__device__ __forceinline__ T row_reduce(T v, Op op) {
  v = op(v, dpp_of<kRowRor8>(v));
  v = op(v, dpp_of<kRowRor4>(v));
  v = op(v, dpp_of<kQuadXor2>(v));
  return op(v, dpp_of<kQuadXor1>(v));
}

template <class T, class Op>
__device__ __forceinline__ T wave_reduce(T v, Op op) {
  T a, b;
  swap32(v, a, b);
  v = op(a, b);
  swap16(v, a, b);
  v = op(a, b);
  return row_reduce(v, op);
}

__device__ __forceinline__ double wave_sum(double v) {
  return wave_reduce(v, [](double a, double b) { return a + b; });
}

__device__ __forceinline__ int wave_sum(int v) {
  return wave_reduce(v, [](int a, int b) { return a + b; });
}

__device__ __forceinline__ double wave_max(double v) {
  return wave_reduce(v, [](double a, double b) { return fmax(a, b); });
}

// Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous run of logical block ids so neighbouring tiles (which share
// nodes) run under the same L2.
__device__ __forceinline__ int xcd_block(int b, int G) {
  const int x = b & 7, j = b >> 3, q = G >> 3, r = G & 7;
  return x * q + (x < r ? x : r) + j;
}

// Tiles [t0, t1) of logical block lb out of G.
__device__ __forceinline__ void block_tiles(const Range& r, int& t0, int& t1) {
  const int G = gridDim.x;
  const int lb = xcd_block(blockIdx.x, G);
  const int64_t ntl = r.tile_end - r.tile_begin;
  t0 = r.tile_begin + (int)((int64_t)lb * ntl / G);
  t1 = r.tile_begin + (int)((int64_t)(lb + 1) * ntl / G);
}

inline int grid_for(const Range& r, const LaunchCfg& cfg) {
  const int64_t ntl = r.tile_end - r.tile_begin;
  const int64_t groups = (ntl + cfg.waves - 1) / cfg.waves;
  int64_t g = cfg.blocks > 0 ? std::min<int64_t>(cfg.blocks, groups) : groups;
  return (int)std::max<int64_t>(g, 1);
}

}  // namespace cm
