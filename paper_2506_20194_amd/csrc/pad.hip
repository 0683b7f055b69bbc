// Zero-padded copies of matrices whose sizes or alignment the aligned products do
// not take: a layer of k = 3000 columns then runs on the same kernels as one of
// 3072, instead of on edge tiles with per-element bounds checks.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace duo {

namespace {

// One thread per four columns of dst; rows along blockIdx.y.
__global__ __launch_bounds__(256) void pad_copy_kernel(const float* __restrict__ src, int64_t lds, int rows, int cols,
                                                       float* __restrict__ dst, int64_t ldd, int rows_p, int cols_p,
                                                       float diag) {
  const int c = 4 * (blockIdx.x * 256 + threadIdx.x);
  if (c >= cols_p) return;
  for (int r = blockIdx.y; r < rows_p; r += gridDim.y) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = r < rows && c + e < cols;
      v[e] = in ? src[(int64_t)r * lds + c + e] : (r == c + e && r >= rows ? diag : 0.f);
    }
    *(float4*)(dst + (int64_t)r * ldd + c) = make_float4(v[0], v[1], v[2], v[3]);
  }
}

}  // namespace

duo_status pad_copy(const float* src, int64_t lds, int64_t rows, int64_t cols, float* dst, int64_t ldd, int64_t rows_p,
                    int64_t cols_p, float diag, hipStream_t s) {
  hipLaunchKernelGGL(pad_copy_kernel, dim3((unsigned)cdiv(cols_p, 1024), (unsigned)(rows_p < 4096 ? rows_p : 4096)),
                     dim3(256), 0, s, src, lds, (int)rows, (int)cols, dst, ldd, (int)rows_p, (int)cols_p, diag);
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

}  // namespace duo
