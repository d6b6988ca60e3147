// The fp32 -> 16-bit conversions of common.h and the SwiGLU quotient of gemm_epi.h as kernels of their own, for tests
// that compare them with the integer definition and with the division.  Linked into libvlac_safe.so only.
#include "common.h"
#include "gemm_epi.h"

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

__global__ __launch_bounds__(256) void silu_check_kernel(uint32_t first, int n, float* __restrict__ denominator,
                                                         float* __restrict__ got, uint32_t* __restrict__ differ) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint32_t u = first + (uint32_t)i;
  const float x = __uint_as_float(u), y = 1.f + __expf(-x), b = x / y, any = silu_any(x), a = fabsf(x) > kFarGate ? any : silu_quick(x);
  if (denominator) denominator[i] = y;
  if (got) got[i] = a;
  auto other = [&](float v) { return __float_as_uint(v) != __float_as_uint(b) && !(v != v && b != b); };
  if (other(a) || other(any)) {
    atomicAdd(differ, 1u);
    atomicMin(differ + 1, u);
  }
}

// The n fp32 values whose bits are first, first + 1, ...: differ[0] += those where a quotient as the epilogues make it is not
// x / (1 + e^-x) by the IEEE division, bit for bit (two NaN are alike), differ[1] = the least bits of one; denominator, got:
// device fp32 [n] or NULL
extern "C" int vlac_silu_check(uint32_t first, int n, float* denominator, float* got, uint32_t* differ, void* stream) {
  if (!differ) return VLAC_E_NULL;
  if (n < 1 || n > (1 << 30)) return VLAC_E_RANGE;
  hipLaunchKernelGGL(silu_check_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, first, n, denominator, got, differ);
  return hipGetLastError() == hipSuccess ? VLAC_OK : VLAC_E_HIP;
}
