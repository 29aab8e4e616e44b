// The part of the HIP language that the transform kernels use, for a host
// compiler: one host thread per lane, a barrier per workgroup.
#pragma once

#include <cmath>
#include <cstddef>

#define __host__
#define __device__
#define __global__
#define __shared__
#define __forceinline__ inline
#define __align__(n) alignas(n)
#define __launch_bounds__(...)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))

struct HostDim3 {
  unsigned x = 1, y = 1, z = 1;
};
inline thread_local HostDim3 threadIdx, blockIdx;
inline HostDim3 blockDim, gridDim;
void __syncthreads();
