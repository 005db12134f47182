// Dilated LSTM layer for small batches (Section 3.2, Table 1; Section 8.3 notes
// how little of a GPU such small cells use): forward and reverse kernels that
// give a workgroup FOUR series instead of sixteen.
//
// When series tiles x chains of a layer is far below the number of compute
// units, the 16-series kernels of lstm_kernels.hip leave most of the chip idle
// and the layer costs (positions of the longest chain) x (time of one position
// on one compute unit).  Both factors are attacked here: four times as many
// workgroups, and a position costs a quarter of the matrix work.
//
// Arithmetic.  v_mfma_f32_4x4x1_16B_f32: sixteen independent 4x4 outer products
// ("blocks") per instruction, one k-step.  Lane l belongs to block l/4; it
// supplies A[l%4] and B[l%4] of its block and holds D[0..3][l%4].  With its
// broadcast control (cbsz = 4, abid = b) all sixteen blocks take the A values
// of block b.  Here A carries the ACTIVATIONS of the four series for one
// column, broadcast from the block whose four lanes hold them, and B carries
// the weights: lane 16 g + u of a wave holds gate g of hidden unit u.  One
// instruction advances 16 units x 4 gates x 4 series by one column, and no
// operand has to be replicated over the blocks: a wave reads h_{p-d} of
// the four series from LDS with one 4-byte load per 16 columns.  (The input half
// comes from other waves, lstm_narrow_fwd.h.)  Four waves
// share the units; wave w owns w*HT .. w*HT+HT-1 (HT <= 16; the padded
// hidden size is 4*HT).  A lane ends up with one gate of one unit for the four
// series; a transpose between components and rows of sixteen lanes (four
// instructions) turns that into the four gates of one unit for ONE series, and
// the cell update is lane-local as in the 16-series kernels.
//
// The reverse kernel follows the 16-series one step by step (gate gradients,
// transposed contraction split over the waves along the contraction, weight
// gradient in accumulators for the whole launch) with these differences: the
// transposed contraction runs on the 4x4x1 instruction with the gate gradients
// broadcast straight from the registers of the lanes that computed them; the
// weight gradient contracts over the four series, which is exactly the k = 4 of
// ONE 16x16x4 instruction per 16x16 tile of dW (or half the k of a bf16 one, over
// four positions); the LDS arrays a position writes
// are double-buffered by position parity, which leaves one barrier per
// position.  Every LDS array is laid out [row][4 series], so that each access
// of a wave covers consecutive addresses.
//
// Waves that carry the recurrence are bound by the instructions they issue, so
// whatever it does not need is done by other waves: the inputs and their half
// of the pre-activations (forward, four more waves), and in the reverse kernel, where
// the grid leaves the room, all requests and the factors that do not depend on the
// recurrence (four more), the weight gradient and the input gradient (four more).
//
// Global operands.  A position takes a fraction of a microsecond here, less
// than the latency of HBM, so operands are requested several positions
// ahead into registers.  The forward kernel requests the inputs of
// four positions at a time, one or two such groups ahead; the reverse kernel requests a
// position and stages one in LDS in every position, with twelve waves in some that store nothing.
// A run of four positions is ONE straight run of
// instructions (the position loop inside it is unrolled): memory operations complete
// in order, and only with request and use in the same run does the compiler's wait for
// a request count the operations issued since instead of waiting for all of them.
// Lanes past HT repeat the last unit of the wave, operands and addresses alike, so no
// request sits behind a divergent branch.
//
// All tensors keep the layouts of the 16-series kernels (TL(R) tiles of 16
// series), so layers of both kinds mix freely and the weight-gradient
// reduction is unchanged; a workgroup touches 16-byte pieces of each row.
#pragma once

#include <type_traits>

#include "device_utils.h"
#include "esrnn_internal.h"

namespace esrnn {

namespace {

constexpr int kNW = 4;          // waves that share the units (twice as many run where there are two kinds of waves)
constexpr int kNT = 64 * kNW;

// D_blk[i][j] += A_ABID[i] * B_blk[j] for all 16 blocks: the A values of block ABID serve every block.
template <int ABID>
__device__ __forceinline__ f32x4 mfma4_bcast(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, ABID, 0);
}

// value of the same register in another lane of the quad: quad_perm control [a, b, c, d]
template <int CTRL>
__device__ __forceinline__ float quad_perm(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// 4x4 transpose between the components and the rows of sixteen lanes: row s, component c  <->  row c, component s.
__device__ __forceinline__ void row_transpose(f32x4 &v)
{
    // (the pair's elements are copied first: a bit cast of the second element itself takes the first one)
    auto swap16 = [](float &x, float &y) {          // row bit 0 against the choice of x or y
        const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
        const unsigned r0 = r[0], r1 = r[1];
        x = __builtin_bit_cast(float, r0);
        y = __builtin_bit_cast(float, r1);
    };
    auto swap32 = [](float &x, float &y) {          // row bit 1
        const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
        const unsigned r0 = r[0], r1 = r[1];
        x = __builtin_bit_cast(float, r0);
        y = __builtin_bit_cast(float, r1);
    };
    float v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];
    swap16(v0, v1);
    swap16(v2, v3);
    swap32(v0, v2);
    swap32(v1, v3);
    v = f32x4{v0, v1, v2, v3};
}

// LDS that the twelve-wave reverse kernels take only so that no two of their workgroups share a compute unit: more than half of the 160 KB
// together with the `used` bytes that they need.  They have at most one workgroup per compute unit; where registers leave room for two,
// chains would share their SIMDs.  With / without: first layer of 501 monthly series 110 / 119 us, of 512 hourly ones 271 / 266.
// Forward kernels leave that room: alone on the chip they are as fast, and several streams that serve small requests share compute units
// (four streams, forward passes of 1024 quarterly series 345 us each round instead of 365, of 64 monthly ones 315 instead of 360).
template <int used>
__device__ __forceinline__ void alone_on_compute_unit()
{
    constexpr int enough = 84 * 1024;
    if constexpr (used < enough) {
        __shared__ char rest[enough - used];
        asm volatile("" ::"v"((__attribute__((address_space(3))) char *)rest));
    }
}

// workgroups along x: groups of 32 = 8 tiles x 4 quarters
inline int narrow_grid_x(int NB) { return ((NB + 7) / 8) * 32; }

}  // namespace

}  // namespace esrnn
