// Fixed-order sums over a workgroup of up to 1024 threads, shared by the kernels
// whose partial sums must agree bitwise.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gpk {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Block-wide sum in a fixed order; the result is valid in thread 0.  sh: one entry per wave.
__device__ __forceinline__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) r += sh[i];
  __syncthreads();
  return r;
}

}  // namespace gpk
