// What the host headers of csrc/ need of the HIP runtime, for compiling device
// code with a host compiler (tests/topk_host.cpp, tests/plan_host.cpp).
#pragma once
#include <stddef.h>
#include <stdint.h>
#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
typedef int hipError_t;
typedef void* hipStream_t;
constexpr hipError_t hipSuccess = 0;
inline hipError_t hipGetLastError() { return hipSuccess; }
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
