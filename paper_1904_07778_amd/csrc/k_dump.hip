// Dump kernel and the sum of a split launch's chunks.  Dump kernel: copy accumulators out for any number of arrays in one launch
// (a null source writes zeros: the same kernel clears accumulators).  A
// kernel rather than copies and memsets: one launch for all arrays, and it
// may be recorded into a captured graph.
#include "kernels.hpp"

namespace xeng {
namespace {

__global__ __launch_bounds__(256) void dump_kernel(DumpParams d) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int k = 0; k < d.count; ++k) {
    const int2* __restrict__ src = d.acc[k];
    int2* __restrict__ dst = d.dst[k];
    const int64_t n = d.n[k];
    if (src) {
      for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) dst[i] = src[i];
    } else {
      for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) dst[i] = int2{0, 0};
    }
  }
}

// dst[i] = prev[i] (or 0) + the sum of the n-long chunks of part: the end of
// a launch split along time.  Reads every chunk once, coalesced, 8 loads in
// flight per thread; bound by memory, or by its launch where n is small.
__global__ __launch_bounds__(256) void sum_chunks(const int2* prev, const int2* __restrict__ part, int2* dst,
                                                  int64_t n, int chunks) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    int2 s = prev ? prev[i] : int2{0, 0};
    for (int c = 0; c < chunks; c += 8) {
      int2 x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = part[min(c + k, chunks - 1) * n + i];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (c + k < chunks) s.x += x[k].x, s.y += x[k].y;
    }
    dst[i] = s;
  }
}

}  // namespace

hipError_t sum_launch(hipStream_t s, const int2* prev, const int2* part, int2* dst, int64_t n, int chunks) {
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(sum_chunks, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, s, prev, part, dst, n,
                     chunks);
  return hipGetLastError();
}

hipError_t dump_launch(int grid, hipStream_t s, const DumpParams& d) {
  hipLaunchKernelGGL(dump_kernel, dim3(grid), dim3(256), 0, s, d);
  return hipGetLastError();
}

}  // namespace xeng
