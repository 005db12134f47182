// The device helpers of the kernel sources, for the build on the CPU (host_kernels.cpp): addresses and barriers are
// those of the device, arithmetic across lanes is not formed.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

// host_kernels.cpp
void host_barrier();
void host_global(const void *at, int bytes);    // stops the program if it lies outside the workspace

namespace esrnn {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

template <int I, int N, class F>
inline void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

typedef const char *buf_rsrc;
inline buf_rsrc make_rsrc(const void *base) { return static_cast<const char *>(base); }
template <class V>
inline V &buf_at(buf_rsrc r, unsigned bytes)
{
    host_global(r + bytes, sizeof(V));
    return *reinterpret_cast<V *>(const_cast<char *>(r + bytes));
}
inline float buf_load(buf_rsrc r, unsigned lane_bytes, unsigned tile_bytes) { return buf_at<float>(r, lane_bytes + tile_bytes); }
inline f32x4 buf_load4(buf_rsrc r, unsigned lane_bytes, unsigned tile_bytes) { return buf_at<f32x4>(r, lane_bytes + tile_bytes); }
template <bool kStream = false>
inline void buf_store(buf_rsrc r, unsigned lane_bytes, unsigned tile_bytes, float v) { buf_at<float>(r, lane_bytes + tile_bytes) = v; }
template <bool kStream = false>
inline void buf_store4(buf_rsrc r, unsigned lane_bytes, f32x4 v) { buf_at<f32x4>(r, lane_bytes) = v; }

constexpr int kNeedWords = 8, kNeedMost = 32 * kNeedWords;
inline unsigned long long needed_classes(const unsigned *, int, int, int, int) { return ~0ull; }

inline void lds_barrier() { host_barrier(); }
inline float sigmoid_f(float x) { return 0.5f + 0.1f * x; }
inline float tanh_f(float x) { return 0.1f * x; }
inline float wave_sum(float v) { return v; }
inline float group16_sum(float v) { return v; }

}  // namespace esrnn

#define __syncthreads() host_barrier()
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_canonicalizef(x) (x)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_ds_read_tr16_b64_v4i16(at) (*(at))
