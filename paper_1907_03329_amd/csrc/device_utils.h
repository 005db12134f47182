// Device helpers shared by the kernels: the 16x16x4 fp32 MFMA tile, LDS-only
// barrier, activation functions, wave reductions.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

namespace esrnn {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// compile-time loop: f(std::integral_constant<int, I>) for I = 0 .. N-1 (for indices that must be immediates:
// MFMA broadcast blocks, register sets that rotate through a loop)
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// f(std::integral_constant<int, k % N>, k) for k = 0, 1, ... while it returns true: a loop unrolled N times that is left
// from any of its parts.  (With parts that are skipped instead, the compiler sees ways around the requests in them, and waits
// for everything that is under way wherever one of them is used.)
template <int N, class F, int... I>
__device__ __forceinline__ bool round_of(F &&f, int first, std::integer_sequence<int, I...>)
{
    return (f(std::integral_constant<int, I>{}, first + I) && ...);
}
template <int N, class F>
__device__ __forceinline__ void rotate_while(F &&f)
{
    for (int first = 0; round_of<N>(f, first, std::make_integer_sequence<int, N>{}); first += N) {}
}

// D = A(16x4) * B(4x16) + C(16x16), fp32.  Lane l supplies A[l%16][l/16] and
// B[l/16][l%16]; it holds D[4*(l/16) + r][l%16] in component r.
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Buffer addressing for the wave-uniform tiles of the LSTM kernels: the tile's base is a scalar resource (built
// with scalar instructions from a pointer that is the same in every lane), the tile's offset inside it a scalar
// byte offset, the lane's share a 32-bit byte offset that never changes.  No address arithmetic is left on the
// vector ALU, whose cycles the fp32 MFMAs need.  A resource spans 4 GiB from its base (raw buffer, no stride, no
// range limit): callers rebase it per window position and keep the offsets inside one position.
typedef __amdgpu_buffer_rsrc_t buf_rsrc;
__device__ __forceinline__ buf_rsrc make_rsrc(const void *base, int bytes = -1)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ float buf_load(buf_rsrc r, unsigned lane_bytes, unsigned tile_bytes)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, lane_bytes, tile_bytes, 0));
}
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 buf_load4(buf_rsrc r, unsigned lane_bytes, unsigned tile_bytes)
{
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane_bytes, tile_bytes, 0));
}
// kStream: the value is not read again soon (streaming store)
template <bool kStream = false>
__device__ __forceinline__ void buf_store(buf_rsrc r, unsigned lane_bytes, unsigned tile_bytes, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, lane_bytes, tile_bytes, kStream ? 2 : 0);
}
// Four dwords.  The tile's offset belongs into the resource's base here, not into the scalar offset: the vector ALU
// may overwrite a register of a wide store right after it only with one wait state in between, and the compiler
// leaves that out where the scalar offset is a register (an exemption of older chips).  Seen on this chip: now and
// then the first dword of a stored quad held what the next instruction had written to its register.
template <bool kStream = false>
__device__ __forceinline__ void buf_store4(buf_rsrc r, unsigned lane_bytes, f32x4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, lane_bytes, 0, kStream ? 2 : 0);
}

// The same for data that another workgroup of the launch writes or reads, at any place of the chip (every XCD has an L2 of
// its own): written through to memory, read past the caches.
constexpr int kBufShared = 16;
__device__ __forceinline__ float buf_load_shared(buf_rsrc r, unsigned lane_bytes, unsigned tile_bytes)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, lane_bytes, tile_bytes, kBufShared));
}
__device__ __forceinline__ void buf_store_shared(buf_rsrc r, unsigned lane_bytes, unsigned tile_bytes, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, lane_bytes, tile_bytes, kBufShared);
}

// Which of the residue classes r, r + step, ... below d a forward pass has to compute for a series tile: bit i for class
// r + i step, the same in every lane (all ones without masks, or where there are more classes than bits).
constexpr int kNeedWords = 8, kNeedMost = 32 * kNeedWords;
__device__ __forceinline__ unsigned long long needed_classes(const unsigned *masks, int tile, int r, int step, int d)
{
    if (!masks || d > kNeedMost || d > 64 * step) return ~0ull;
    const int mine = r + (int)(threadIdx.x & 63) * step;
    const bool want = mine < d && ((masks[(size_t)tile * kNeedWords + (min(mine, d - 1) >> 5)] >> (mine & 31)) & 1);
    return __ballot(want);
}

// (by a workgroup of 256 threads)
template <class Words>
__device__ __forceinline__ void clear_words(const Words &w, int stride)
{
    for (int i = threadIdx.x; i < w.n; i += 256) w.at[i * stride] = 0u;
}

// Workgroup barrier that orders LDS traffic only: global loads and stores in
// flight are not waited for.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Natural logarithm of a normal positive number (series values, levels and seasonal factors are far from
// the denormal range): the hardware log2 without the rescaling path for denormals.
__device__ __forceinline__ float fast_log(float x) { return __builtin_amdgcn_logf(x) * 0.69314718055994531f; }

__device__ __forceinline__ float sigmoid_f(float x)
{
    return fast_rcp(1.0f + __expf(-x));
}

// tanh(x) = 1 - 2 / (1 + exp(2x)); saturates correctly at both ends.  exp(2x) = 2^(x * 2 log2(e)): one
// multiplication, with the same result as doubling x first (doubling is exact).
constexpr float kTanhExponent = 2.8853900817779268f, kSigmoidExponent = -1.4426950408889634f;
__device__ __forceinline__ float tanh_of_exponent(float e)
{
    return 1.0f - 2.0f * fast_rcp(1.0f + __builtin_amdgcn_exp2f(e));
}
__device__ __forceinline__ float sigmoid_of_exponent(float e) { return fast_rcp(1.0f + __builtin_amdgcn_exp2f(e)); }
__device__ __forceinline__ float tanh_f(float x) { return tanh_of_exponent(x * kTanhExponent); }

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// maximum over the ACTIVE lanes of the wave, the same value in every lane (wave-uniform)
__device__ __forceinline__ int wave_max_int(int v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return __builtin_amdgcn_readfirstlane(v);
}

// sum over the 16 lanes that share lane/16
__device__ __forceinline__ float group16_sum(float v)
{
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

}  // namespace esrnn
