// The backward's fp32 dQ accumulator: clearing it, and turning it into dQ. Memory-bound.
#include "common.hpp"

namespace vcja {
namespace {

// dq = bf16(scale * acc), four elements per thread; the first zero4 fours of each sample zero.
__global__ void dq_from_acc_kernel(const float* acc, __bf16* dq, size_t n4, size_t zero4, float scale) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const size_t at = blockIdx.y * n4 + i;
  const f32x4 x = i < zero4 ? f32x4{0.0f, 0.0f, 0.0f, 0.0f} : ((const f32x4*)acc)[at] * scale;
  ((bf16x4*)dq)[at] = bf16x4{(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]};
}

// Fused dQ: zeroes the fp32 accumulator (a kernel, not a memset, so that a captured graph
// replays it like any other node). n4 = elements / 4.
__global__ void zero_f32_kernel(float* x, size_t n4) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n4) ((f32x4*)x)[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
}

}  // namespace

hipError_t launch_zero_f32(float* x, size_t n, hipStream_t s) {
  const size_t n4 = n / 4;
  if (n4) hipLaunchKernelGGL(zero_f32_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, x, n4);
  return hipGetLastError();
}

hipError_t launch_dq_from_acc(const float* acc, __bf16* dq, int B, size_t per_sample, size_t zero, float scale,
                              hipStream_t s) {
  const size_t n4 = per_sample / 4;
  if (n4)
    hipLaunchKernelGGL(dq_from_acc_kernel, dim3((unsigned)((n4 + 255) / 256), B), dim3(256), 0, s, acc, dq, n4, zero / 4,
                       scale);
  return hipGetLastError();
}

}  // namespace vcja
