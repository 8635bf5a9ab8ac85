// Memory-bound passes: the backward's fp32 dQ accumulator cleared and turned into dQ, and the
// text rows of the branches where the branch's own grid does not write them.
#include <algorithm>

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

template <int D>
__global__ __launch_bounds__(256) void text_rows_kernel(TextRows t, int H, int N, int T) {
  const size_t first = (size_t)blockIdx.y * N * H * D;  // sample blockIdx.y alone: no division by its chunks
  t.x0 += first;
  if (t.x1) t.x1 += first;
  if (t.x2) t.x2 += first;
  if (t.lse) t.lse += (size_t)blockIdx.y * H * N;
  if (t.sum_a) t.sum_a += first;
  if (t.sum_b) t.sum_b += first;
  if (t.sum) t.sum += first;
  write_text_rows<D>(t, 1, H, N, T, threadIdx.x, blockIdx.x, gridDim.x);
}

}  // namespace

// In the branch's grid up to 24 chunks a thread, up to 16 with an LSE, whose index takes a
// division, and up to 8 with a sum, whose reads a thread waits for. Measured, us a call, in the grid
// / apart: temporal forward at 3.6 chunks 8.2 / 11.1, 13 9.7 / 10.5, 21 11.8 / 10.4, 64 24.3 / 10.8;
// with the sum at 3.6 9.7 / 10.9, 8 21.0 / 22.5, 11 12.1 / 10.7, 43 27.3 / 10.7; backward at 11 10.1 /
// 11.2, 21 11.8 / 11.2 and 9.4 / 11.3, 28 18.8 / 21.1, 32 12.0 / 11.2; spatial forward at 8 218.9 /
// 219.2, 21 67.1 / 63.4, 128 159 / 117, its backward at 21 108.2 / 108.7.
hipError_t place_text_rows(const TextRows& t, int B, int H, int N, int T, int head_dim, size_t threads, hipStream_t s,
                           int* in_grid) {
  const size_t per = (size_t)T * H * (head_dim / 8);
  const bool apart = B * per > (t.sum ? 8 : t.lse ? 16 : 24) * threads;
  *in_grid = apart ? 0 : T;
  if (!apart) return hipSuccess;
  const dim3 grid((unsigned)std::min<size_t>((per + 255) / 256, 1 << 20), B);
  if (head_dim == 128)
    hipLaunchKernelGGL(text_rows_kernel<128>, grid, dim3(256), 0, s, t, H, N, T);
  else
    hipLaunchKernelGGL(text_rows_kernel<64>, grid, dim3(256), 0, s, t, H, N, T);
  return hipGetLastError();
}

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
