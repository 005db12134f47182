// Reverse pass of a dilated LSTM layer on the 4-series kernels: the kernel template and its launcher, included by
// one translation unit per kind of workgroup (four waves / twelve waves) so that the two compile side by side.
#pragma once

#include "lstm_narrow_common.h"
#include "lstm_together.h"
#include "three_term.h"

namespace esrnn {

namespace {

// ---------------------------------------------------------------------------
// Reverse pass.  Per position p of a chain, descending:
//   A. every lane turns (dh, dc) of its (unit, series) into the four gate
//      pre-activation gradients da (registers; a copy goes to LDS for step C);
//   B. a wave multiplies W^T by the da of the units it owns: 4x4x1 MFMA with da
//      as the broadcast A operand, taken from the registers of the four lanes
//      that hold unit u, and the weights as B (a block is four consecutive
//      columns of [x ; h]); the four partial results meet in LDS (part);
//   -- barrier --
//   every lane sums the four partials of its own (unit, series): the recurrent
//      dh of the next position; the threads sum and store the input gradient;
//   C. dW += da (x) [x_p ; h_{p-d}], contraction over the four series; row tiles
//      dealt to the waves round-robin.  With twelve waves three bf16 16x16x32 MFMAs
//      per 16x16 tile and four positions (three_term.h), else one fp32 16x16x4 MFMA
//      per tile and position.
// da_all and part alternate between two copies by position parity: what a
// position writes was last read two positions earlier, one barrier ago.  So do the
// staged factors of step A, per thread of the chain waves (the third position of a chain
// is staged when the first one's have been taken, behind a barrier of its own).
// [x ; h] rows, which all waves of step C read, are in four buffers by position, or
// in two by groups of four positions, written with a group's last position.
// ---------------------------------------------------------------------------
struct NarrowBwdArgs {
    const float *wpack;   // [4][NG][4*HT][64]  operands of W^T: wave, column group, k-step (unit, gate), lane = column
    const float *xsrc;    // TL(4*KXT)
    const float *gates, *c, *hid;
    const float *gsrc[2];
    int n_gsrc;
    float *gdst;          // TL(4*KXT)
    float *dw_partial;    // [4*NB*chains][HT*CT][4][64]
    float *db_partial;    // [4*NB*chains][HT][4][4]
    int P, NB, d;
    const int32_t *pmax;  // [NB] positions the longest series of a 16-series tile has: its chains stop there
    const int32_t *lengths;
    const Scalars *sc;
    float two_lambda_cs;
    int B, T, I, H;
};

// (up to hidden 40 the kernel is held to 256 registers: two workgroups per compute unit, which the chains of a
// dilated layer need to run side by side)
// SPLIT: twelve waves.  Waves 0-3 carry the recurrence: steps A and B and the sums of the recurrent gradient, nothing else.
// Waves 4-7 do step C, the weight gradient, one barrier behind the recurrence, and sum and store the input gradient; waves
// 8-11 request and stage all operands.  All kinds take the same barriers (one per position).  For grids of at most one workgroup
// per compute unit: a chain wave is bound by the instructions it issues, and the SIMDs have the other waves' work while it
// waits.
// What bounds it: the chain alone takes 216 of 292 us for 512 hourly series (first layer, 24 + 40 columns, 649 positions),
// without step C 264, without staging 255.  What it took, us at 512 hourly, 501 monthly (20 + 50 columns, 211 positions) and 1024
// quarterly series (4 + 40 columns, 61 positions): eight waves, operands in chunks of four positions, step C in fp32 445, 224, 45; step C
// in bf16 alone 497, 236, 52 (the eight waves' second half became longer still); operands staged position by position, and
// factors of step A formed there 391, 188, 46; twelve waves 302, 172, 36; staging ahead of step C (s_setprio) 292, 169, 35.5.
// The kind with four waves, which has all of it on the chain waves, gained from staging by position too: hidden 64, two layers of 61 positions,
// 68 groups 217 -> 191 us, 130 groups 324 -> 284, dilation two 68 groups 116 -> 104.
// MODE: kLater, layers of one launch (lstm_together.h): this layer waits for the one above it, and its positions are counted; kLast,
// nobody waits for this one.
// Staging.  Every position of a chain stages one (the factors that the chain waves need of it, its row of [x ; h]) and requests one:
// a position's operands are in flight while kSets others pass.  In chunks of four, all requests in one position and all LDS writes in
// another, those two positions took twice as long as the others, for every wave of the workgroup.
constexpr int kSets = 4;
// Layers that follow another one request the gradient that it leaves only so many positions ahead of the staging (one, two or
// three are within 1 %).
constexpr int narrow_bwd_gradient_sets(int mode) { return mode == kLater ? 2 : 3; }
// Step C on the bf16 matrix pipe (three_term.h), four positions at a time (kGroup).  (At 13 unit tiles of x, and above, sums and
// operands are more registers than a lane has where three waves share a SIMD.)
constexpr bool narrow_bwd_three_term(int HT, int KXT, bool split) { return split && HT <= 13 && KXT < 13; }
constexpr int kGroup = 4;
constexpr int narrow_bwd_threads(bool split) { return split ? 3 * kNT : kNT; }
static_assert(kGroup == kSets, "positions are unrolled by the group");

template <int HT, int KXT, bool SPLIT, int MODE>
struct NarrowBwdLds {                                   // (references: an object each where nothing else has to fit)
    static constexpr int KX = 4 * KXT, HP = 4 * HT, KT4 = KX + HP;
    static constexpr int NG = (KT4 + 63) / 64;          // groups of 64 columns of [x ; h]
    static constexpr int CT = (KT4 + 15) / 16;          // 16-column tiles of dW
    static constexpr bool kThree = narrow_bwd_three_term(HT, KXT, SPLIT);
    static constexpr int PC = NG * 64 < KT4 + 1 ? NG * 64 : KT4 + 1;    // columns of part (those past KT4 share one)
    // rows of [x_p ; h_{p-d}]: [position][column][series], or as operands of step C: [group][column tile][(hi mid), (lo hi)][lane]
    using Rows = std::conditional_t<kThree, u32x4[2][CT][2][64], float[kGroup][CT * 64]>;
    using Part = float[2][kNW][PC * 4];
    using Staged = f32x4[2][2][kNT];
    float (&da_all)[2][HP * 16];             // [unit][series][gate]
    Part &part;                              // partial W^T da of every wave [column][series]
    Staged &lc;                              // per thread: the factors of a position
    Rows &xh;
    static constexpr size_t at_part = sizeof(float) * 2 * HP * 16, at_lc = at_part + sizeof(Part), at_xh = at_lc + sizeof(Staged), bytes = at_xh + sizeof(Rows);
    static __device__ __forceinline__ NarrowBwdLds in(char *at)
    {
        return {reinterpret_cast<float (&)[2][HP * 16]>(*at), reinterpret_cast<Part &>(at[at_part]),
                reinterpret_cast<Staged &>(at[at_lc]), reinterpret_cast<Rows &>(at[at_xh])};
    }
};

// One workgroup: quarter q of series tile bt, residue classes chain, chain + chains, ...  (With twelve waves one class: a grid with fewer
// chains than classes is too large for them.  Without the loops over classes the first layer of 501 monthly series takes 115 us instead
// of 110, of 512 hourly ones as long.)
template <int HT, int KXT, bool CP, bool SPLIT, int MODE>
__device__ __forceinline__ void lstm_backward_narrow_body(const NarrowBwdArgs &a, const NarrowBwdLds<HT, KXT, SPLIT, MODE> &lds, int bt, int q,
                                                          int chain, int chains, const Progress &progress)
{
    using Lds = NarrowBwdLds<HT, KXT, SPLIT, MODE>;
    using std::integral_constant;
    static_assert(SPLIT || MODE == kAlone, "");
    constexpr bool kWaits = MODE != kAlone, kCounts = MODE == kLater;
    constexpr int KX = Lds::KX, HP = Lds::HP, KT4 = Lds::KT4, NG = Lds::NG, CT = Lds::CT;
    constexpr bool kThree = Lds::kThree;
    constexpr int kAhead = narrow_bwd_gradient_sets(MODE);
    // 16-row tiles of dW per wave (a row tile = 4 units x 4 gates).  With twelve waves, tiles that are left when every wave has as many are
    // shared by kShare waves, which take every kShare-th column tile of it.  (A whole one more in the first wave: up to 12 registers in
    // scratch memory at hidden 50, layers of one launch.  With four waves it is the other way round.)
    constexpr int MTW = (HT + kNW - 1) / kNW;
    constexpr int kLeft = SPLIT ? HT % kNW : 0, kFull = SPLIT ? HT / kNW : MTW, kShare = kLeft ? kNW / kLeft : 1, CL = kLeft ? (CT + kShare - 1) / kShare : 1;
    static_assert(kLeft != 3, "tiles that are left are shared by 4 or 2 waves");
    // elements (column, series) of [x ; h] that a thread brings: number tid, and tid + kNT where there are as many
    constexpr bool kTwo = 4 * KT4 > kNT;
    static_assert(4 * KX <= kNT && 4 * KT4 <= 2 * kNT, "the second one is of h");

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = SPLIT ? (wv & (kNW - 1)) : wv;
    const int kind = SPLIT ? wv / kNW : 0;          // 0 chain, 1 weight gradient, 2 staging
    const int blk = lane >> 2, j = lane & 3;
    // All four workgroups of a 16-series tile stop at the tile's longest series: what lies beyond is
    // neither computed here nor read by any later kernel.
    const int Pt = a.pmax[bt];
    const bool valid = blk < HT;
    const int unit = w * HT + min(blk, HT - 1);     // blocks past HT repeat the last unit
    const int lane_off = unit * 16 + 4 * q + j;
    // input gradient: thread t sums and stores element t mod 4*KX (threads past 4*KX repeat earlier ones)
    const int tid = (int)threadIdx.x & (kNT - 1);
    const int dx_el = tid % (4 * KX);
    const bool first_x = tid < 4 * KX;
    const bool first = tid < 4 * KT4, second = kTwo && tid + kNT < 4 * KT4, second_any = kTwo && 64 * w + kNT < 4 * KT4;
    auto element_bytes = [&](int el) { return 4 * ((el >> 2) * 16 + 4 * q + (el & 3)); };
    const int at_x = element_bytes(min(tid, 4 * KX - 1)), at_h = element_bytes(min(max(tid - 4 * KX, 0), 4 * HP - 1)),
              at_h2 = element_bytes(min(tid + kNT - 4 * KX, 4 * HP - 1));
    // operands of the weight-gradient tiles inside 64 consecutive floats of da_all / xh
    const int ar_off = 16 * (lane & 3) + 4 * (lane >> 4) + ((lane & 15) >> 2);   // unit l%4, series l/16, gate (l%16)/4
    const int xb_off = 4 * (lane & 15) + (lane >> 4);                            // column l%16, series l/16

    const int left_tile = kFull * kNW + w / kShare, left_col = w % kShare;      // (of the tile that this wave shares)
    f32x4 dw[kFull > 0 ? kFull : 1][CT], dw_left[CL];
#pragma unroll
    for (int t = 0; t < kFull; ++t)
#pragma unroll
        for (int nb = 0; nb < CT; ++nb) dw[t][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nb = 0; nb < CL; ++nb) dw_left[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 dbacc = f32x4{0.f, 0.f, 0.f, 0.f};
    // (columns past KT4 stay zero)
    for (int e = threadIdx.x; e < (int)(sizeof(lds.xh) / sizeof(float)); e += narrow_bwd_threads(SPLIT)) reinterpret_cast<float *>(&lds.xh)[e] = 0.0f;

    auto store_dw = [&]() {
        const size_t partix = (size_t)(4 * bt + q) * chains + chain;
        auto store = [&](int mt, int nb, const f32x4 &v) {
            float *dst = a.dw_partial + (partix * (HT * CT) + mt * CT + nb) * 256 + lane;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) dst[rr * 64] = v[rr];
        };
#pragma unroll
        for (int t = 0; t < kFull; ++t)
            if (SPLIT || w + kNW * t < HT) {
#pragma unroll
                for (int nb = 0; nb < CT; ++nb) store(w + kNW * t, nb, dw[t][nb]);
            }
        if constexpr (kLeft > 0) {
#pragma unroll
            for (int nb = 0; nb < CL; ++nb)
                if (left_col + kShare * nb < CT) store(left_tile, left_col + kShare * nb, dw_left[nb]);
        }
    };

    // ---- requests and staging of one position, whose number in the chain is `set` modulo kSets
    Below above(progress, Pt);
    const float g2_scale = a.n_gsrc >= 2 ? 1.0f : 0.0f;
    int n_valid = 0;
    float pen = 0.0f;
    if constexpr (CP) {
        const int col = bt * kTileN + 4 * q + j;
        const int len = col < a.B ? min(max(a.lengths[col], 0), a.T) : 0;
        n_valid = len - a.I - a.H + 1;
        pen = MODE == kAlone || a.sc ? a.two_lambda_cs * a.sc->inv_n_cs : 0.0f;
    }
    f32x4 s_gates[kSets];       // (native vectors: arrays of the HIP float4 class do not stay in registers)
    float s_c[kSets], s_a[kSets], s_b[kSets], s_x[kSets], s_h[kSets], s_h2[kSets];
    auto tile_at = [](const float *array, unsigned tile, unsigned floats) {
        return reinterpret_cast<const char *>(array) + (unsigned long long)tile * (4u * floats);
    };
    auto earlier = [&](int p) { return p >= a.d ? p - a.d : p; };       // (stays at the chain's first)
    auto request_gradient = [&](auto setc, int p) {
        constexpr int set = decltype(setc)::value;
        const unsigned tile = (unsigned)p * a.NB + bt;
        const buf_rsrc r0 = make_rsrc(tile_at(a.gsrc[0], tile, HP * 16)), r1 = make_rsrc(tile_at(a.gsrc[1], tile, HP * 16));
        s_a[set] = kWaits ? buf_load_shared(r0, 4 * lane_off, 0) : buf_load(r0, 4 * lane_off, 0);
        s_b[set] = kWaits ? buf_load_shared(r1, 4 * lane_off, 0) : buf_load(r1, 4 * lane_off, 0);
    };
    auto request = [&](auto setc, int p) {
        constexpr int set = decltype(setc)::value;
        const unsigned tile = (unsigned)p * a.NB + bt, before = tile - (p >= a.d ? (unsigned)a.d * a.NB : 0u);
        __builtin_amdgcn_sched_barrier(0);
        s_gates[set] = buf_load4(make_rsrc(tile_at(a.gates, tile, 4 * HP * 16)), 16 * lane_off, 0);
        s_c[set] = buf_load(make_rsrc(tile_at(a.c, tile, HP * 16)), 4 * lane_off, 0);
        if constexpr (!kWaits) request_gradient(setc, p);
        const buf_rsrc r_h = make_rsrc(tile_at(a.hid, before, HP * 16));
        s_x[set] = buf_load(make_rsrc(tile_at(a.xsrc, tile, KX * 16)), at_x, 0);
        if constexpr (4 * KX < kNT) s_h[set] = buf_load(r_h, at_h, 0);
        if constexpr (kTwo) s_h2[set] = buf_load(r_h, at_h2, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // Factors of step A that do not depend on the recurrent gradient: dh = gs + dhreg; dc = dcreg + dh ad + pc;
    // da = (dc ki, dc kf, dc kg, dh ko); dcreg = dc f.
    float even[2] = {0.0f, 0.0f};
    Parts pair[2] = {{0, 0, 0}, {0, 0, 0}};
    auto write_rows = [&](int at, int e, Parts p1) {
        if constexpr (kThree) {
            const int el = tid + e * kNT, l = (el >> 2 & 15) + 16 * (el & 3);
            if (e == 0 ? first : second) {
                u32x4 (&to)[2][64] = lds.xh[at][el >> 6];
                const Parts p0 = pair[e];
                to[0][l] = u32x4{p0.hi, p1.hi, p0.mid, p1.mid};
                to[1][l] = u32x4{p0.lo, p1.lo, p0.hi, p1.hi};
            }
        }
    };
    // (`at`: the buffer of the group of rows)
    auto stage = [&](auto setc, int p, int at) {
        constexpr int set = decltype(setc)::value;
        const bool has_prev = p >= a.d;
        const f32x4 v = s_gates[set];                      // input, forget, candidate, output gate
        const float c = s_c[set], cp = has_prev ? s_c[(set + 1) % kSets] : 0.0f, tc = tanh_f(c);
        float gs = s_a[set] + g2_scale * s_b[set];
        if constexpr (kWaits) gs = above.checked(gs);
        lds.lc[set & 1][0][tid] = f32x4{v[0] * v[2] * (1.0f - v[0]), v[1] * cp * (1.0f - v[1]), v[0] * (1.0f - v[2] * v[2]),
                                        v[3] * tc * (1.0f - v[3])};
        lds.lc[set & 1][1][tid] = f32x4{gs, v[3] * (1.0f - tc * tc), v[1], CP && p < n_valid ? pen * c : 0.0f};
        const float h1 = 4 * KX < kNT && has_prev ? s_h[set] : 0.0f;
        auto row = [&](int e, float v) {
            if constexpr (!kThree) {
                if (e == 0 ? first : second) lds.xh[set][tid + e * kNT] = v;
            } else if constexpr (set % 2 == 0) {
                even[e] = __builtin_canonicalizef(v);       // (a register of its own: that of the request is the next one's)
            } else {
                const Parts p = split_pair<true>(even[e], v);
                if constexpr (set == 1) pair[e] = p;
                else write_rows(at, e, p);
            }
        };
        row(0, first_x ? s_x[set] : h1);
        if constexpr (kTwo)
            if (second_any) row(1, has_prev ? s_h2[set] : 0.0f);
    };
    int p_stage = 0, p_ask = 0, p_gradient = 0;         // positions that come next
    // of a position that is the k-th of its group: stages the second one after it
    auto staging = [&](auto kc, int at) {
        constexpr int k = decltype(kc)::value, set = (k + 2) % kSets;
        if constexpr (kWaits) {
            above.wait_falling(p_gradient);
            request_gradient(integral_constant<int, (set + kAhead) % kSets>{}, p_gradient);
            p_gradient = earlier(p_gradient);
        }
        stage(integral_constant<int, set>{}, p_stage, at);
        p_stage = earlier(p_stage);
        request(integral_constant<int, set>{}, p_ask);
        p_ask = earlier(p_ask);
    };
    // requests ahead of a chain that ends at p_last, and staging of its first two positions
    auto staging_start = [&](int p_last) {
        p_ask = p_stage = p_gradient = p_last;
        static_for<0, kSets>([&](auto setc) {
            request(setc, p_ask);
            p_ask = earlier(p_ask);
        });
        if constexpr (kWaits) {
            above.wait_falling(earlier(p_gradient));
            static_for<0, 2>([&](auto setc) {
                request_gradient(setc, p_gradient);
                p_gradient = earlier(p_gradient);
            });
        }
        __syncthreads();            // LDS free: initial clearing, or the last position of the previous chain
        static_for<0, 2>([&](auto setc) {
            stage(setc, p_stage, 0);
            p_stage = earlier(p_stage);
            request(setc, p_ask);
            p_ask = earlier(p_ask);
        });
        lds_barrier();
        if constexpr (SPLIT) lds_barrier();         // (the third position takes the place of the first)
        if constexpr (kWaits) static_for<2, 2 + kAhead>([&](auto setc) {
            above.wait_falling(p_gradient);
            request_gradient(integral_constant<int, decltype(setc)::value % kSets>{}, p_gradient);
            p_gradient = earlier(p_gradient);
        });
    };
    // ---- sum and store of one position's input gradient
    auto input_gradient = [&](int p, int par) {
        const float dxv = (lds.part[par][0][dx_el] + lds.part[par][1][dx_el]) + (lds.part[par][2][dx_el] + lds.part[par][3][dx_el]);
        const buf_rsrc to = make_rsrc(tile_at(a.gdst, (unsigned)p * a.NB + bt, KX * 16));
        const int at = (dx_el >> 2) * 16 + 4 * q + (dx_el & 3);
        if constexpr (kCounts) buf_store_shared(to, 4 * at, 0, dxv);
        else buf_store(to, 4 * at, 0, dxv);
    };
    // ---- C: weight gradient of one position, k = the four series; da in lds.da_all[par], [x ; h] in lds.xh[k]
    auto step_c = [&](int par, int k) {
        if constexpr (!kThree) {
            float xb[CT];
#pragma unroll
            for (int nb = 0; nb < CT; ++nb) xb[nb] = lds.xh[k][64 * nb + xb_off];
            // row 4*gate + u of a tile mt is gate `gate` of unit 4*mt + u
#pragma unroll
            for (int t = 0; t < kFull; ++t) {
                if (SPLIT || w + kNW * t < HT) {
                    const float ar = lds.da_all[par][64 * (w + kNW * t) + ar_off];
#pragma unroll
                    for (int nb = 0; nb < CT; ++nb) dw[t][nb] = mfma16(ar, xb[nb], dw[t][nb]);
                }
            }
            if constexpr (kLeft > 0) {
                const float ar = lds.da_all[par][64 * left_tile + ar_off];
#pragma unroll
                for (int nb = 0; nb < CL; ++nb) dw_left[nb] = mfma16(ar, lds.xh[k][64 * min(left_col + kShare * nb, CT - 1) + xb_off], dw_left[nb]);
            }
        }
    };
    // ---- C in groups of four positions, k = position and series (two positions in a dword), two terms of a product in one
    // instruction: da as (hi hi), (mid mid), (hi lo), [x ; h] as (hi mid), (lo hi).  A group is gathered and split while its positions
    // pass, and multiplied, a part of the column tiles at a time, while those of the next one do.
    unsigned da_p[kThree ? MTW : 1][3][2], da_c[kThree ? MTW : 1][3][2];    // parts of the group that passes, and of the one before it
    float da_even[kThree ? MTW : 1];
    auto group_start = [&]() {
#pragma unroll
        for (int t = 0; t < MTW; ++t)
#pragma unroll
            for (int m = 0; m < 3; ++m) da_c[t][m][0] = da_c[t][m][1] = 0;
    };
    auto gather_pair = [&](int t, int pair, float even, float odd) {
        const Parts p = split_pair<true>(even, odd);
        da_p[t][0][pair] = p.hi;
        da_p[t][1][pair] = p.mid;
        da_p[t][2][pair] = p.lo;
    };
    // da of position k of a group
    auto gather = [&](auto kc) {
        constexpr int k = decltype(kc)::value;
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
            const float v = lds.da_all[k & 1][64 * (t < kFull ? w + kNW * t : left_tile) + ar_off];
            if constexpr (k % 2 == 0) da_even[t] = v;
            else gather_pair(t, k / 2, da_even[t], v);
        }
    };
    // no da from position `rest` of a group on
    auto gather_none = [&](int rest) {
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
            if (rest == 1) gather_pair(t, 0, da_even[t], 0.0f);
            gather_pair(t, 1, rest == 3 ? da_even[t] : 0.0f, 0.0f);
        }
    };
    auto group_done = [&]() {
#pragma unroll
        for (int t = 0; t < MTW; ++t)
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                da_c[t][m][0] = da_p[t][m][0];
                da_c[t][m][1] = da_p[t][m][1];
            }
    };
    // the k-th quarter of the column tiles of the group before, whose rows lie in buffer `at`; smallest terms first
    auto multiply = [&](auto kc, int at) {
        constexpr int k = decltype(kc)::value, first = k * CT / kGroup, end = (k + 1) * CT / kGroup;
        if constexpr (kThree) {
            auto quad = [&](int t, int m) {         // (hi lo), (mid mid), (hi hi)
                const unsigned (&c)[3][2] = da_c[t];
                const int a = m == 1 ? 1 : 0, b = 2 - m;
                return u32x4{c[a][0], c[a][1], c[b][0], c[b][1]};
            };
            static_for<first, end>([&](auto nbc) {
                constexpr int nb = decltype(nbc)::value;
                const u32x4 x0 = lds.xh[at][nb][0][lane], x1 = lds.xh[at][nb][1][lane];
#pragma unroll
                for (int m = 0; m < 3; ++m)
#pragma unroll
                    for (int t = 0; t < kFull; ++t) dw[t][nb] = mfma_bf16(quad(t, m), m == 0 ? x1 : x0, dw[t][nb]);
                if constexpr (MTW > 3) __builtin_amdgcn_sched_barrier(0);       // (for its registers)
            });
            // (backwards through the quarters: the first one has the fewest of the others)
            if constexpr (kLeft > 0) static_for<k * CL / kGroup, (k + 1) * CL / kGroup>([&](auto nbc) {
                constexpr int nb = CL - 1 - decltype(nbc)::value;
                const int col = min(left_col + kShare * nb, CT - 1);
                const u32x4 x0 = lds.xh[at][col][0][lane], x1 = lds.xh[at][col][1][lane];
#pragma unroll
                for (int m = 0; m < 3; ++m) dw_left[nb] = mfma_bf16(quad(kFull, m), m == 0 ? x1 : x0, dw_left[nb]);
            });
        }
    };
    // Both kinds of waves meet once more after a chain's last position: the last input gradients are in memory; the rows of a last
    // group of one position are in LDS.
    auto last_barrier = [](int n) { return kCounts || (kThree && n % kGroup == 1); };
    if constexpr (SPLIT) {
        // the same barriers as the chain waves below: start of a chain, first staging, first factors taken, one per position
        if (kind == 2) {
            __builtin_amdgcn_s_setprio(2);      // (what the chain waits for before what nothing does)
            for (int r0 = chain; r0 < a.d && r0 < Pt; r0 += chains) {
                const int n = (Pt - r0 + a.d - 1) / a.d;
                staging_start(r0 + (n - 1) * a.d);
                int at = 0;             // buffer of the group that is staged
                auto position = [&](auto kc) {
                    staging(kc, at);
                    lds_barrier();
                };
                if (int groups = n / kGroup) do {
                    static_for<0, kGroup>(position);
                    at ^= 1;
                } while (--groups);
                const int rest = n % kGroup;
                static_for<0, kGroup - 1>([&](auto kc) {
                    if (decltype(kc)::value < rest) position(kc);
                });
                // (the rows of a group are written with its last position, or here)
                if (rest == 1) {
                    write_rows(at, 0, Parts{0, 0, 0});
                    if constexpr (kTwo) write_rows(at, 1, Parts{0, 0, 0});
                }
                if (last_barrier(n)) lds_barrier();
            }
            return;
        }
        if (kind == 1) {
            for (int r0 = chain; r0 < a.d && r0 < Pt; r0 += chains) {
                const int n = (Pt - r0 + a.d - 1) / a.d;
                int p = r0 + (n - 1) * a.d, counted = -a.d, before = 1;     // (buffer of the group that is multiplied)
                __syncthreads();
                lds_barrier();
                lds_barrier();
                if constexpr (kThree) group_start();
                auto position = [&](auto kc) {
                    constexpr int k = decltype(kc)::value;
                    // (what a wave stores behind the input gradient that is counted next: a count and another one)
                    if constexpr (kCounts) stores_complete_but<2>();
                    lds_barrier();
                    if constexpr (kCounts) progress.publish(max(counted, 0), w == 0);
                    counted += a.d;
                    input_gradient(p, k & 1);
                    p -= a.d;
                    if constexpr (kThree) {
                        multiply(kc, before);
                        gather(kc);
                    } else {
                        step_c(k & 1, k);
                    }
                };
                if (int groups = n / kGroup) do {
                    static_for<0, kGroup>(position);
                    if constexpr (kThree) group_done();
                    before ^= 1;
                } while (--groups);
                const int rest = n % kGroup;
                static_for<0, kGroup - 1>([&](auto kc) {
                    if (decltype(kc)::value < rest) position(kc);
                });
                if constexpr (kCounts) stores_complete_but<0>();
                if (last_barrier(n)) lds_barrier();
                if constexpr (kCounts) progress.publish(n * a.d, w == 0);
                if constexpr (kThree) {
                    // the rest of the last whole group, and the positions after it
                    static_for<0, kGroup>([&](auto kc) {
                        if (decltype(kc)::value >= rest) multiply(kc, before);
                    });
                    if (rest > 0) {
                        gather_none(rest);
                        group_done();
                        static_for<0, kGroup>([&](auto kc) { multiply(kc, before ^ 1); });
                    }
                }
            }
            store_dw();
            return;
        }
        __builtin_amdgcn_s_setprio(3);      // (ahead of the other waves of the SIMD)
    }

    float wreg[NG][4 * HT];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int k = 0; k < 4 * HT; ++k) wreg[g][k] = a.wpack[(((size_t)w * NG + g) * (4 * HT) + k) * 64 + lane];
    // (waited for here: in the loop the waits for them stay in every other position)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int k = 0; k < 4 * HT; ++k) asm volatile("" : "+v"(wreg[g][k]));

    for (int r0 = chain; r0 < a.d && r0 < Pt; r0 += chains) {
        const int n = (Pt - r0 + a.d - 1) / a.d;
        int p = r0 + (n - 1) * a.d;
        float dcreg = 0.0f, dhreg = 0.0f;
        if constexpr (SPLIT) {
            __syncthreads();
            lds_barrier();
        } else {
            staging_start(p);
        }
        // factors of the first position; those of position i+1 are read before the barrier that ends position i
        f32x4 f0 = lds.lc[0][0][tid], f1 = lds.lc[0][1][tid];
        lds_barrier();
        // One position; `staged` runs after the next one's factors have been read and before the
        // barrier.
        auto position = [&](auto parc, auto staged) {
            constexpr int par = decltype(parc)::value;
            // ---- A: gate gradients of (unit, series)
            const float dh = f1[0] + dhreg;
            float dc = dcreg + dh * f1[1];
            if constexpr (CP) dc += f1[3];
            const f32x4 da = f32x4{dc * f0[0], dc * f0[1], dc * f0[2], dh * f0[3]};
            dcreg = dc * f1[2];
            dbacc += da;
            *reinterpret_cast<f32x4 *>(&lds.da_all[par][16 * unit + 4 * j]) = da;    // for step C
            // ---- B: partial W^T da over the k-steps (unit, gate) of this wave; da of unit u is
            // broadcast from the registers of block u.  Two chains of dependent instructions: the two
            // column groups, or with one group two accumulators (more would cost the second resident
            // workgroup its registers at hidden 40).
            constexpr int kBwdAcc = NG == 1 ? 2 : 1;
            f32x4 acc[NG][kBwdAcc];
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[g][0] = acc[g][kBwdAcc - 1] = f32x4{0.f, 0.f, 0.f, 0.f};
            static_for<0, HT>([&](auto ic) {
                constexpr int ul = decltype(ic)::value;
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    acc[g][0] = mfma4_bcast<ul>(da[0], wreg[g][4 * ul + 0], acc[g][0]);
                    acc[g][1 % kBwdAcc] = mfma4_bcast<ul>(da[1], wreg[g][4 * ul + 1], acc[g][1 % kBwdAcc]);
                }
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    acc[g][2 % kBwdAcc] = mfma4_bcast<ul>(da[2], wreg[g][4 * ul + 2], acc[g][2 % kBwdAcc]);
                    acc[g][3 % kBwdAcc] = mfma4_bcast<ul>(da[3], wreg[g][4 * ul + 3], acc[g][3 % kBwdAcc]);
                }
            });
            // lane l of group g holds column 64g + l for the four series
#pragma unroll
            for (int g = 0; g < NG; ++g)
                *reinterpret_cast<f32x4 *>(&lds.part[par][w][min(64 * g + lane, Lds::PC - 1) * 4]) =
                    kBwdAcc == 2 ? acc[g][0] + acc[g][1] : acc[g][0];
            f0 = lds.lc[par ^ 1][0][tid];
            f1 = lds.lc[par ^ 1][1][tid];
            staged();
            lds_barrier();
            // ---- sums of the four partials: recurrent dh of this lane; input gradient
            {
                const int e = 4 * (KX + unit) + j;
                dhreg = (lds.part[par][0][e] + lds.part[par][1][e]) + (lds.part[par][2][e] + lds.part[par][3][e]);
            }
            if constexpr (!SPLIT) input_gradient(p, par);        // (else the other waves' work)
            p -= a.d;
        };
        if constexpr (SPLIT) {
            if (int pairs = n / 2) do {
                position(integral_constant<int, 0>{}, [] {});
                position(integral_constant<int, 1>{}, [] {});
            } while (--pairs);
            if (n & 1) position(integral_constant<int, 0>{}, [] {});
            if (last_barrier(n)) lds_barrier();
        } else {
            auto whole = [&](auto kc) {
                constexpr int k = decltype(kc)::value;
                position(integral_constant<int, (k & 1)>{}, [&] { staging(kc, 0); });
                step_c(k & 1, k);
            };
            if (int groups = n / kGroup) do {
                static_for<0, kGroup>(whole);
            } while (--groups);
            static_for<0, kGroup - 1>([&](auto kc) {
                if (decltype(kc)::value < n % kGroup) whole(kc);
            });
        }
    }

    if constexpr (!SPLIT) store_dw();
    const size_t partix = (size_t)(4 * bt + q) * chains + chain;
    // bias gradient: sum over the four series (the lanes of a quad)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        float v = dbacc[rr];
        v += quad_perm<0xB1>(v);
        v += quad_perm<0x4E>(v);
        dbacc[rr] = v;
    }
    if (valid && j == 0) {
        float *dst = a.db_partial + partix * (HT * 16) + (size_t)unit * 4;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) dst[rr] = dbacc[rr];
    }
}

template <int HT, int KXT, bool CP, bool SPLIT>
__global__ void __launch_bounds__(narrow_bwd_threads(SPLIT), (!SPLIT && HT <= 10) ? 2 : 1) lstm_backward_narrow_kernel(NarrowBwdArgs a)
{
    using Lds = NarrowBwdLds<HT, KXT, SPLIT, kAlone>;
    __shared__ __align__(16) float da_all[2][Lds::HP * 16];
    __shared__ __align__(16) typename Lds::Part part;
    __shared__ __align__(16) typename Lds::Staged lc;
    __shared__ __align__(16) typename Lds::Rows xh;
    if constexpr (SPLIT) alone_on_compute_unit<(int)Lds::bytes>();
    // The four workgroups of a 16-series tile share every 64-byte row of the tile.  Consecutive workgroup
    // ids go round the 8 XCDs, each with its own L2: ids x, x+8, x+16, x+24 of a group of 32 are the four
    // quarters of ONE tile, so they land on the same XCD at about the same time and a row is fetched from
    // HBM once, not four times (measured before: 2.3-2.8 times the algorithmic bytes).
    const int bt = (blockIdx.x >> 5) * 8 + (blockIdx.x & 7), q = (blockIdx.x >> 3) & 3;
    if (bt >= a.NB) return;     // the grid is padded to whole groups of 32 (before any barrier)
    lstm_backward_narrow_body<HT, KXT, CP, SPLIT, kAlone>(a, Lds{da_all, part, lc, xh}, bt, q, blockIdx.y, gridDim.y, Progress{});
}

template <int HT, int KXT, bool SPLIT>
hipError_t run_nbwd(const NarrowBwdArgs &a, int chains, hipStream_t st)
{
    const dim3 grid(narrow_grid_x(a.NB), chains);
    if (a.sc) lstm_backward_narrow_kernel<HT, KXT, true, SPLIT><<<grid, narrow_bwd_threads(SPLIT), 0, st>>>(a);
    else lstm_backward_narrow_kernel<HT, KXT, false, SPLIT><<<grid, narrow_bwd_threads(SPLIT), 0, st>>>(a);
    return hipGetLastError();
}

inline NarrowBwdArgs narrow_backward_args(const Plan &pl, int layer, const int32_t *lengths, float *ws)
{
    const LayerPlan &lp = pl.layer[layer];
    NarrowBwdArgs a{};
    const bool cp = lp.first_in_block && pl.cfg.lambda_cs != 0.0f;
    a.lengths = lengths;
    a.sc = cp ? reinterpret_cast<const Scalars *>(ws + pl.scalars) : nullptr;
    a.two_lambda_cs = 2.0f * pl.cfg.lambda_cs;
    a.B = pl.B; a.T = pl.T; a.I = pl.I; a.H = pl.H;
    a.wpack = ws + lp.wpack_bwd; a.xsrc = ws + lp.xsrc; a.gates = ws + lp.gates; a.c = ws + lp.c;
    a.hid = ws + lp.hid;
    a.n_gsrc = lp.n_gsrc < 2 ? lp.n_gsrc : 2;
    a.gsrc[0] = ws + lp.gsrc[0];
    a.gsrc[1] = ws + (lp.n_gsrc > 2 ? pl.gsum : lp.gsrc[lp.n_gsrc >= 2 ? 1 : 0]);
    a.gdst = ws + lp.gdst; a.dw_partial = ws + lp.dw_partial; a.db_partial = ws + lp.db_partial;
    a.P = pl.P; a.NB = pl.NB; a.d = lp.dil;
    a.pmax = reinterpret_cast<const int32_t *>(ws + pl.pmax);
    return a;
}

template <bool SPLIT>
hipError_t launch_narrow_bwd(const Plan &pl, int layer, const int32_t *lengths, float *ws, hipStream_t st)
{
    const LayerPlan &lp = pl.layer[layer];
    const NarrowBwdArgs a = narrow_backward_args(pl, layer, lengths, ws);
#define X(HT_, KXT_) if (pl.HT == HT_ && lp.KXT == KXT_) return run_nbwd<HT_, KXT_, SPLIT>(a, lp.chains_bwd, st);
    ESRNN_LSTM_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace esrnn
