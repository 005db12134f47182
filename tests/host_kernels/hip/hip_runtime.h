// What the kernel sources need of HIP, for a build on the CPU in which a thread of a workgroup is one call of the kernel.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define __shared__ static __attribute__((section("lds")))

struct float4 { float x, y, z, w; };
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1 };
typedef void *hipStream_t;
inline hipError_t hipGetLastError() { return hipSuccess; }
extern dim3 threadIdx, blockIdx, gridDim;
using std::max;
using std::min;
