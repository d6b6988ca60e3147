// The fp32 -> 16-bit conversions of common.h as a kernel of their own, for a test that compares them with the
// integer definition over chosen bit patterns.  Linked into libvlac_safe.so only.
#include "common.h"

__global__ __launch_bounds__(256) void convert_check_kernel(const float* __restrict__ x, int n, uint16_t* __restrict__ bf,
                                                            uint16_t* __restrict__ h, uint32_t* __restrict__ bf2,
                                                            uint32_t* __restrict__ h2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float lo = x[i], hi = x[n - 1 - i];
  bf[i] = f2bf(lo);
  h[i] = f2h(lo);
  bf2[i] = f2bf2(lo, hi);
  h2[i] = f2h2(lo, hi);
}

// x device fp32 [n]; bf, h device uint16 [n]: every value alone; bf2, h2 device uint32 [n]: x[i] below x[n - 1 - i]
extern "C" int vlac_convert_check(const float* x, int n, uint16_t* bf, uint16_t* h, uint32_t* bf2, uint32_t* h2,
                                  void* stream) {
  if (!x || !bf || !h || !bf2 || !h2) return VLAC_E_NULL;
  if (n < 1) return VLAC_E_RANGE;
  hipLaunchKernelGGL(convert_check_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, x, n, bf, h, bf2, h2);
  return hipGetLastError() == hipSuccess ? VLAC_OK : VLAC_E_HIP;
}
