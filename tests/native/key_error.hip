// How far the sampler's single-precision keys are from its exact ones, over every draw there is.
#include <hip/hip_runtime.h>

#include "a3_sample.hpp"

namespace {

// per thread: the largest error of its draws beyond the exact key's last place, in units of
// kKeyError (1 / weight + key)
__global__ __launch_bounds__(256) void k_key_error(uint32_t bias_q16, double* worst) {
  const double inv_bias = 1.0 / (double)bias_q16;
  const float inv_w = (float)inv_bias * 65536.0f;  // as the sampler has it
  const uint64_t threads = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t me = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double most = 0.0;
  for (uint64_t x = me; x < (1ull << 32); x += threads) {
    const double exact = (double)a3::sample_key((uint32_t)x, bias_q16, inv_bias) * 0x1p-32;
    const double key = (double)__uint_as_float(a3::approx_key((uint32_t)x, inv_w));
    const double err = (fabs(key - exact) - 0x1p-32) / ((double)a3::kKeyError * ((double)inv_w + exact));
    most = fmax(most, err);
  }
  worst[me] = most;
}

}  // namespace

// worst: blocks * 256 doubles of device memory
extern "C" int key_error(uint32_t bias_q16, uint32_t blocks, double* worst, void* stream) {
  if (bias_q16 < 65536u || blocks == 0 || !worst) return -1;
  hipLaunchKernelGGL(k_key_error, dim3(blocks), dim3(256), 0, (hipStream_t)stream, bias_q16, worst);
  return (int)hipGetLastError();
}
