// fp32 products on the bf16 matrix pipe, at fp32 accuracy.
//
// A float is the exact sum of three bf16 numbers: hi = x rounded to bf16, mid = the rest rounded to bf16, lo = what
// is left (24 significant bits = 8 + 8 + 8; each difference is exact).  A product x y is then the sum of nine
// products of bf16 numbers, each exact in fp32.  The six largest are formed: hi hi, hi mid, mid hi, mid mid, hi lo,
// lo hi.  (The method is published: G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", ARITH 2019.)  The three left out (mid lo, lo mid, lo lo)
// reach 2^-24 of |x y| together (x = y = 1.0038986: 0.99 2^-24), as much as the rounding of one fp32 product at its
// worst; their rms over all pairs of significands is 0.09 2^-24.  Sums are kept in fp32 accumulators.  Measured over
// 10^5 dot products of length 96 against float64: relative rms error 1.70e-7 with six terms, 1.70e-7 with all nine,
// 1.77e-7 with v_mfma_f32_16x16x4_f32; largest error over the sum of |x y| 2.66e-7, 2.66e-7, 2.79e-7.
//
// How the instruction rounds matters for sums over many positions and series (measured, 10^5 sums of 32 products): an
// accumulator smaller than the sum of products it receives loses its low bits downwards, 0.07 to 0.10 of a unit in the
// last place of the result on average for any accumulator up to a quarter of that sum; 0.02 to 0.04 at equal size, none
// from four times the sum on and none from zero.  v_mfma_f32_16x16x4_f32 has no such bias.
//
// Why: v_mfma_f32_16x16x32_bf16 does 8192 multiply-adds in 16 cycles, the fp32 instruction 1024 in 32; six of the
// one for eight of the other is 96 cycles against 256, and the bf16 instruction leaves the vector ALU of its SIMD
// about two instructions in its shadow, which the fp32 one does not.
//
// Operand layout of one instruction: lane (g = l / 16, n = l % 16) supplies 8 consecutive k, 8 g .. 8 g + 7, as
// four dwords of two bf16.  Which columns those k stand for is free as long as both operands agree.  Here a dword
// of lane g is a PAIR of columns that belong to lane group g (two unit tiles, or two gates of a unit), and the
// dwords of one instruction need not be of the same part: a contraction over `np` pairs is cut into full groups of
// four pairs (six instructions each) and a rest of one or two pairs, whose parts share instructions (two and three
// instructions; a rest of three pairs is padded to a full group).
#pragma once

#include "device_utils.h"

namespace esrnn {

// ---- output stage (head_kernels.hip): waves of a workgroup.  Eight (two per SIMD) where their corners of LDS and the
// operands kept there fit into 128 KB and a lane's sums into 256 registers.
constexpr int head_waves(int HT, int MO) { return (HT <= 10 && MO == 1) || (HT <= 8 && MO == 2) ? 8 : 4; }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// ---- how a contraction over np pairs is cut (host and device) ----
constexpr int tt_full(int np) { return (np + 1) / 4; }
constexpr int tt_rest(int np) { return np > 4 * tt_full(np) ? np - 4 * tt_full(np) : 0; }      // 0, 1, 2
constexpr int tt_b_quads(int np) { return 3 * tt_full(np) + tt_rest(np); }                     // operand that changes
constexpr int tt_a_quads(int np) { return 3 * tt_full(np) + (tt_rest(np) ? tt_rest(np) + 1 : 0); }   // weights
constexpr int tt_mfmas(int np) { return 6 * tt_full(np) + (tt_rest(np) ? tt_rest(np) + 1 : 0); }

// what dword d of weight quad q holds: the pair and the part (0 hi, 1 mid, 2 lo; -1: zero)
struct TtDword { int pair, part; };
constexpr TtDword tt_a_dword(int np, int q, int d)
{
    const int full = tt_full(np), base = 4 * full;
    if (q < 3 * full) return {4 * (q / 3) + d, q % 3};
    q -= 3 * full;
    if (tt_rest(np) == 1) {
        if (q == 0) return {base, d == 3 ? 1 : 0};           // with (hi, mid, lo, hi): hi hi, hi mid, hi lo, mid hi
        return {base, d == 0 ? 2 : (d == 1 ? 1 : -1)};       //                         lo hi, mid mid
    }
    if (q == 0) return {base + (d & 1), 0};                  // with (hi hi mid mid): hi hi, hi mid
    if (q == 1) return {base + (d & 1), 1};                  //                       mid hi, mid mid
    return {base + (d & 1), d < 2 ? 0 : 2};                  // with (lo lo hi hi):   hi lo, lo hi
}
// quads of instruction i
struct TtPair { int a, b; };
constexpr TtPair tt_mfma(int np, int i)
{
    const int full = tt_full(np);
    if (i < 6 * full) {
        const int g = 3 * (i / 6), k = i % 6;
        const int a[6] = {0, 1, 0, 1, 2, 0}, b[6] = {0, 0, 1, 1, 0, 2};
        return {g + a[k], g + b[k]};
    }
    i -= 6 * full;
    if (tt_rest(np) == 1) return {3 * full + i, 3 * full};
    return {3 * full + i, 3 * full + (i == 2 ? 1 : 0)};
}

// ---- how the reverse kernel (lstm_backward.h) deals its work (host and device) ----
// Up to 13 unit tiles; at 16 its weights and sums do not fit the registers of 16 waves.
constexpr bool bwd_three_term(int HT) { return HT <= 13; }
constexpr int bwd_even_tiles(int HT) { return HT + HT % 2; }
// Waves that carry the recurrence: one per SIMD where sixteen waves leave room for others that form its factors.
constexpr int bwd_chain_waves(int HT) { return HT <= 10 ? (HT >= 8 ? 4 : 1) : (HT + 1) / 2; }
constexpr int bwd_factor_waves(int HT) { return HT <= 10 ? HT / 2 : 0; }
constexpr int bwd_dw_waves(int HT) { return HT / 2; }
constexpr int bwd_h_row_tiles(int HT) { return (HT + 3) / 4; }
// unit tiles of x that do not fill a 16-row tile and find room in the last one of h
constexpr int bwd_merged_tiles(int HT, int KXT)
{
    return KXT >= 4 && KXT % 4 <= 4 * bwd_h_row_tiles(HT) - HT ? KXT % 4 : 0;
}
constexpr int bwd_x_row_tiles(int HT, int KXT) { return bwd_merged_tiles(HT, KXT) ? KXT / 4 : (KXT + 3) / 4; }
constexpr int bwd_waves(int HT, int KXT)
{
    return bwd_chain_waves(HT) + bwd_dw_waves(HT) + bwd_x_row_tiles(HT, KXT) + bwd_factor_waves(HT);
}
// dwords of its A operands: [row tiles of x, then of h][unit tile][part][64][2]
constexpr int bwd_pack_dwords(int HT, int KXT)
{
    return (bwd_x_row_tiles(HT, KXT) + bwd_h_row_tiles(HT)) * bwd_even_tiles(HT) * 3 * 128;
}

// quads of instruction i of one full group, smallest terms first
constexpr TtPair tt_group_rising(int i)
{
    const int a[6] = {0, 2, 1, 0, 1, 0}, b[6] = {2, 0, 1, 1, 0, 0};
    return {a[i], b[i]};
}

// Round to nearest even; a in the low half.  kOnce keeps the compiler from rounding a second time to get at the low half:
// two instructions fewer a pair, but a fixed order (the reverse kernel gains 3 %, the forward kernel loses as much).
template <bool kOnce = false>
__device__ __forceinline__ unsigned bf16_pack(float a, float b)
{
    bf16x2 v;
    v[0] = (__bf16)a;
    v[1] = (__bf16)b;
    unsigned r = __builtin_bit_cast(unsigned, v);
    if constexpr (kOnce) asm("" : "+v"(r));
    return r;
}

struct Parts { unsigned hi, mid, lo; };      // two bf16 each

template <bool kOnce = false>
__device__ __forceinline__ Parts split_pair(float a, float b)
{
#pragma clang fp contract(off)      // (the differences below are of the rounded a and b, not of what they were formed from)
    Parts p;
    p.hi = bf16_pack<kOnce>(a, b);
    const float a1 = a - __builtin_bit_cast(float, p.hi << 16), b1 = b - __builtin_bit_cast(float, p.hi & 0xffff0000u);
    p.mid = bf16_pack<kOnce>(a1, b1);
    const float a2 = a1 - __builtin_bit_cast(float, p.mid << 16), b2 = b1 - __builtin_bit_cast(float, p.mid & 0xffff0000u);
    p.lo = bf16_pack<kOnce>(a2, b2);
    return p;
}

// An infinite input (the logarithm of a zero observation) or weight as a number that still saturates what it is multiplied
// into: the parts of an infinity would be inf, NaN, NaN.  NaN stays NaN.  Inputs are logarithms, states and flags; neither
// they nor weights come near the limit otherwise.
__device__ __forceinline__ float splittable(float x)
{
    constexpr float limit = 0x1p100f;
    return __builtin_fabsf(x) > limit ? __builtin_copysignf(limit, x) : x;
}

__device__ __forceinline__ unsigned part_of(const Parts &p, int part)
{
    return part == 0 ? p.hi : part == 1 ? p.mid : part == 2 ? p.lo : 0u;
}

// LDS home of 16 rows x 16 series in one part, for operands that are read turned (lstm_backward.h): the four rows of a lane
// group as one 8-byte chunk per lane, [chunk][series], the second half shifted by 32 bytes.
constexpr int kPartBytes = 64 * 8 + 32;

typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 lds_read_transposed(const char *at)
{
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(at)));
}

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

}  // namespace esrnn
