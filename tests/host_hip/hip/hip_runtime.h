// What the device headers need of the HIP runtime header to compile for the
// CPU: the element arithmetic then runs in a host program, with the fused
// multiply-adds and roundings it has on the GPU.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)

struct HostDim3 { unsigned x, y, z; };
static HostDim3 threadIdx, blockIdx, blockDim, gridDim;
typedef void* hipStream_t;
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1 };
inline int atomicAdd(int* p, int v) { *p += v; return *p - v; }
inline int __shfl_xor(int x, int, int) { return x; }
using std::fabs;
using std::isfinite;
using std::max;
using std::min;
