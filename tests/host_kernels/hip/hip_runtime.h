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
struct int4 { int x, y, z, w; };
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1 };
typedef void *hipStream_t;
enum { hipFuncAttributeMaxDynamicSharedMemorySize };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void *, int, int) { return hipSuccess; }
extern dim3 threadIdx, blockIdx, gridDim;
using std::max;
using std::min;

// ---- launches (host_kernels.cpp): thread(context) for every thread of the grid ----
extern float host_dynamic_lds[];
void host_run(dim3 grid, int threads, size_t dynamic_lds, void (*thread)(void *), void *context);
template <class F>
void host_launch(dim3 grid, int threads, size_t dynamic_lds, F &&f)
{
    host_run(grid, threads, dynamic_lds, [](void *c) { (*static_cast<std::remove_reference_t<F> *>(c))(); }, &f);
}

// ---- device builtins: addresses and barriers are those of the device, arithmetic across lanes is not formed ----
void host_barrier();                            // host_kernels.cpp
struct host_rsrc { const char *base; unsigned bytes; };
void host_read(host_rsrc r, unsigned at, int shared, void *to, int bytes);      // host_kernels.cpp, likewise
void host_write(host_rsrc r, unsigned at, int shared, const void *from, int bytes);
void host_wait(int but);                        // until this thread's stores are complete but for the last so many
template <class V>
inline V host_load(host_rsrc r, unsigned at, int aux)
{
    V v;
    host_read(r, at, aux & 16, &v, sizeof(V));
    return v;
}
template <class V>
inline void host_store(const V &v, host_rsrc r, unsigned at, int aux)
{
    host_write(r, at, aux & 16, &v, sizeof(V));
}
typedef unsigned host_b128 __attribute__((ext_vector_type(4)));
typedef host_rsrc __amdgpu_buffer_rsrc_t;
#define __builtin_amdgcn_make_buffer_rsrc(base, stride, range, flags) host_rsrc{static_cast<const char *>(base), (unsigned)(range)}
#define __builtin_amdgcn_raw_buffer_load_b32(r, lane, tile, aux) host_load<unsigned>(r, (lane) + (tile), aux)
#define __builtin_amdgcn_raw_buffer_load_b128(r, lane, tile, aux) host_load<host_b128>(r, (lane) + (tile), aux)
#define __builtin_amdgcn_raw_buffer_store_b32(v, r, lane, tile, aux) host_store<unsigned>(v, r, (lane) + (tile), aux)
#define __builtin_amdgcn_raw_buffer_store_b128(v, r, lane, tile, aux) host_store<host_b128>(v, r, (lane) + (tile), aux)
#define __syncthreads() host_barrier()
#define __ballot(x) ((void)(x), ~0ull)
#define __shfl_xor(v, off, width) (v)
#define __shfl(v, lane, width) (v)
#define __expf(x) (x)
#define __builtin_amdgcn_rcpf(x) (x)
#define __builtin_amdgcn_logf(x) (x)
#define __builtin_amdgcn_exp2f(x) (x)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_s_setprio(x) ((void)0)
void host_sleep();                              // host_kernels.cpp: before every look at another workgroup's words
unsigned long long host_ballot(bool complete);  // until what is waited for is there
#define __builtin_amdgcn_s_sleep(x) host_sleep()
#define __builtin_amdgcn_s_waitcnt(x) host_wait(((x) & 15) | ((x) >> 14 & 3) << 4)
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_update_dpp(old, v, control, rows, banks, bound) (v)
struct host_pair { unsigned v[2]; unsigned operator[](int i) const { return v[i]; } };
#define __builtin_amdgcn_permlane16_swap(a, b, fi, bc) host_pair{{(a), (b)}}
#define __builtin_amdgcn_permlane32_swap(a, b, fi, bc) host_pair{{(a), (b)}}
#define __builtin_canonicalizef(x) (x)
// (the operands count as used, so that the loads that bring them stay)
template <class V>
inline void host_use(const V &v) { __asm__ volatile("" : : "m"(v)); }
#define HOST_MFMA(a, b, c) (host_use(a), host_use(b), (c))
#define __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, x, y, z) HOST_MFMA(a, b, c)
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, x, y, z) HOST_MFMA(a, b, c)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) HOST_MFMA(a, b, c)
#define __builtin_amdgcn_ds_read_tr16_b64_v4i16(at) (*(at))
// (the other waves' bits count for the same wave here)
inline unsigned atomicAdd(unsigned *at, unsigned v) { const unsigned was = *at; *at += v; return was; }
inline unsigned atomicOr(unsigned *at, unsigned v) { return *at |= v; }
