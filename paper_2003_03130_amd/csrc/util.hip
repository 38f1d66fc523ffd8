// Plain device copy: the reference kernel of known traffic against which the
// hardware byte counters (rocprofv3 FETCH_SIZE / WRITE_SIZE) are scaled.  It
// moves data the way the tile kernels stream their chunks: one dword per lane
// per load instruction, consecutive lanes on consecutive addresses.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "cellmech.h"
#include "handle.h"

namespace cm {
namespace {

constexpr int kCopyThreads = 256;

__global__ __launch_bounds__(kCopyThreads) void stream_copy_kernel(const float* src,
                                                                  float* dst, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * kCopyThreads;
  for (int64_t i = (int64_t)blockIdx.x * kCopyThreads + threadIdx.x; i < n; i += stride)
    dst[i] = src[i];
}

// Parameters from three strided device arrays into the handle's (mu[n],
// kappa[n], w[n]).  One launch in place of three copies, each of which took
// 2.6 us on the device and more on the host: with the two parameter updates
// of an autograd pass they were half of a single cell's time.
__global__ __launch_bounds__(256) void set_params_kernel(const double* mu, const double* kappa,
                                                         const double* w, int64_t s_mu,
                                                         int64_t s_kappa, int64_t s_w,
                                                         int64_t n, double* dst) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  dst[i] = mu[i * s_mu];
  dst[n + i] = kappa[i * s_kappa];
  dst[2 * n + i] = w[i * s_w];
}

}  // namespace
}  // namespace cm

extern "C" int cm_set_params_strided(cm_batch h, const double* mu, int64_t stride_mu,
                                     const double* kappa, int64_t stride_kappa,
                                     const double* w, int64_t stride_w, hipStream_t stream) {
  if (!h) return cm::api_fail(CM_EINVAL, "null handle");
  if (!mu || !kappa || !w) return cm::api_fail(CM_EINVAL, "null parameter array");
  if (stride_mu < 0 || stride_kappa < 0 || stride_w < 0)
    return cm::api_fail(CM_EINVAL, "strides must be >= 0");
  int cur = 0;
  CM_HIP(hipGetDevice(&cur));
  if (cur != h->device) CM_HIP(hipSetDevice(h->device));
  hipLaunchKernelGGL(cm::set_params_kernel, dim3((unsigned)((h->n_mat + 255) / 256)),
                     dim3(256), 0, stream, mu, kappa, w, stride_mu, stride_kappa, stride_w,
                     h->n_mat, const_cast<double*>(h->T.params));
  CM_HIP(hipGetLastError());
  h->params_set = true;
  return CM_OK;
}

extern "C" int cm_stream_copy(const float* src, float* dst, int64_t n, hipStream_t stream) {
  if (n < 0) return cm::api_fail(CM_EINVAL, "n must be >= 0");
  if (n == 0) return CM_OK;
  if (!src || !dst) return cm::api_fail(CM_EINVAL, "src and dst must be device pointers");
  const int64_t blocks = (n + cm::kCopyThreads - 1) / cm::kCopyThreads;
  const unsigned grid = (unsigned)(blocks < 65536 ? blocks : 65536);
  hipLaunchKernelGGL(cm::stream_copy_kernel, dim3(grid), dim3(cm::kCopyThreads), 0, stream, src, dst, n);
  CM_HIP(hipGetLastError());
  return CM_OK;
}
