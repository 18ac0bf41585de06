// The Gaussian transform of the noise stream on words of the caller's choice: part of the micro-benchmark library, not of the
// boundary.  The transform's short division and square root are defined to round like the general ones; only 2^24 radii and
// 2^24 angles exist, so a test puts all of them through this kernel and compares them with the checker.
#include "es_device.hpp"

namespace {

__global__ __launch_bounds__(256) void gauss_words_kernel(const uint32_t* __restrict__ xa, const uint32_t* __restrict__ xb, uint32_t n,
                                                          float* __restrict__ zc, float* __restrict__ zs) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < n) es::gauss_pair(xa[i], xb[i], zc[i], zs[i]);
}

}  // namespace

// Device pointers of n elements each, n <= 2^31; enqueued on `stream`.  Returns 0, or a HIP error code.
extern "C" int es_gauss_words(const uint32_t* xa_d, const uint32_t* xb_d, uint32_t n, float* zc_d, float* zs_d, void* stream) {
  if (!xa_d || !xb_d || !zc_d || !zs_d || n == 0 || n > (1u << 31)) return -1;
  hipLaunchKernelGGL(gauss_words_kernel, dim3((n + 255u) / 256u), dim3(256), 0, static_cast<hipStream_t>(stream), xa_d, xb_d, n, zc_d, zs_d);
  return (int)hipGetLastError();
}
