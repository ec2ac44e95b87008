// Exhaustive device check of the decay's exponential (test infrastructure): for every
// fp32 bit pattern z, exp_value, exp_values (z among ordinary neighbours) and
// exp_values_table must equal the double exp rounded once, (float)exp((double)z) (NaN for
// NaN). Prints the number of values checked and of mismatches.
#include <hip/hip_runtime.h>

#include <cstdio>

#include "ssmq_device.hpp"

using namespace ssmq;

__device__ bool same(float got, float z) {
  const float want = static_cast<float>(exp(static_cast<double>(z)));
  return __float_as_uint(got) == __float_as_uint(want) || (got != got && want != want);
}

__global__ __launch_bounds__(256) void k_check_exp(unsigned long long* bad, unsigned long long* count) {
  __shared__ double tab[kExpTable];
  stage_exp_table(tab, threadIdx.x, 256);
  __syncthreads();
  unsigned long long b = 0, n = 0;
  for (uint64_t u = blockIdx.x * 256ull + threadIdx.x; u < (1ull << 32); u += gridDim.x * 256ull) {
    const float z = __uint_as_float(static_cast<uint32_t>(u));
    const float four[4] = {-0.25f, z, 1e-3f, -3.0f};  // ordinary neighbours of any z
    float e4[4];
    exp_values_table<4>(tab, four, e4);
    b += !same(exp_value(z), z) || !same(e4[1], z) || !same(e4[0], four[0]) || !same(e4[3], four[3]);
    exp_values<4>(four, e4);
    b += !same(e4[1], z) || !same(e4[0], four[0]) || !same(e4[2], four[2]) || !same(e4[3], four[3]);
    ++n;
  }
  atomicAdd(bad, b);
  atomicAdd(count, n);
}

#define CK(e) do { hipError_t r_ = (e); if (r_ != hipSuccess) { printf("HIP error %s\n", hipGetErrorString(r_)); return 1; } } while (0)

int main() {
  unsigned long long* d;
  CK(hipMalloc(&d, 2 * sizeof(unsigned long long)));
  CK(hipMemset(d, 0, 2 * sizeof(unsigned long long)));
  hipLaunchKernelGGL(k_check_exp, dim3(256 * 64), dim3(256), 0, 0, d, d + 1);
  CK(hipGetLastError());
  CK(hipDeviceSynchronize());
  unsigned long long h[2];
  CK(hipMemcpy(h, d, sizeof h, hipMemcpyDeviceToHost));
  CK(hipFree(d));
  printf("exp %llu %llu\n", h[1], h[0]);
  return h[0] ? 1 : 0;
}
