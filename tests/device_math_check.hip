// The device sequences of dfw_math.hpp and dfw_math_f32.hpp that stand for IEEE divisions and square roots,
// callable on arrays and over all FP32 arguments.  Built by tests/device_math.py, used by
// tests/test_gpu_device_math.py.
#include <hip/hip_runtime.h>

#include "../paper_2402_10914_amd/csrc/dfw_math.hpp"
#include "../paper_2402_10914_amd/csrc/dfw_math_f32.hpp"

namespace {

__global__ void k_f64(const double* x, double* rcp, double* s, double* is, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  rcp[i] = dfw::rcp_any(x[i]);
  dfw::sqrt_inv(x[i], s[i], is[i]);
}

__global__ void k_quotient(const double* x, double* q, double n, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) q[i] = dfw::quotient_any(n, x[i]);
}

__global__ void k_f32(const float* x, float* rcp, float* root, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  rcp[i] = dfw::cand::recip(x[i]);
  root[i] = dfw::cand::root(x[i]);
}

__device__ bool same(float a, float b) { return __float_as_uint(a) == __float_as_uint(b) || (a != a && b != b); }

// Arguments of [0, 2^32) as bits, kPer per thread: counts those whose reciprocal (bad[0]) or root (bad[1]) is
// not the compiler's division or root.
constexpr unsigned kPer = 1024;
__global__ void k_all(unsigned long long* bad) {
  const unsigned first = (blockIdx.x * blockDim.x + threadIdx.x) * kPer;
  unsigned n[2] = {0, 0};
  for (unsigned q = 0; q < kPer; ++q) {
    const float x = __uint_as_float(first + q);
    if (!same(dfw::cand::recip(x), 1.0f / x)) ++n[0];
    if (!same(dfw::cand::root(x), sqrtf(x))) ++n[1];
  }
  for (int k = 0; k < 2; ++k)
    if (n[k]) atomicAdd(bad + k, (unsigned long long)n[k]);
}

}  // namespace

// All pointers are device memory; work goes to the null stream and is waited for.
extern "C" int dm_f64(const double* x, double* rcp, double* s, double* is, int n) {
  if (n < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_f64, dim3((n + 255) / 256), dim3(256), 0, nullptr, x, rcp, s, is, n);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : hipDeviceSynchronize();
}

extern "C" int dm_quotient(const double* x, double* q, double n, int count) {
  if (count < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_quotient, dim3((count + 255) / 256), dim3(256), 0, nullptr, x, q, n, count);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : hipDeviceSynchronize();
}

extern "C" int dm_f32(const float* x, float* rcp, float* root, int n) {
  if (n < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_f32, dim3((n + 255) / 256), dim3(256), 0, nullptr, x, rcp, root, n);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : hipDeviceSynchronize();
}

extern "C" int dm_all_f32(unsigned long long* bad) {  // two counters, zeroed by the caller
  hipLaunchKernelGGL(k_all, dim3((1ull << 32) / kPer / 256), dim3(256), 0, nullptr, bad);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : hipDeviceSynchronize();
}
