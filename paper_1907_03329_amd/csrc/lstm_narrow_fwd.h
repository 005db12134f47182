// Forward pass of a dilated LSTM layer on the 4-series kernels (see lstm_narrow_common.h for the tiling): the
// kernel template and its launcher, included by one translation unit per residual wiring (plain layer / last layer
// of a residual block) so that the two compile side by side.
#pragma once

#include "lstm_narrow_common.h"
#include "lstm_together.h"

namespace esrnn {

namespace {

struct NarrowFwdArgs {
    const float *wpack;   // [4][KT4][64]  weight operands: wave, input column, lane (gate l/16 of unit l%16 of the wave)
    const float *bias;    // caller's bias vector [4h]
    const float *xsrc;    // TL(4*KXT)
    float *gates;         // TL(HP) x [4]
    float *c, *hid;       // TL(HP)
    const float *resid;   // TL(HP) or null
    float *out;           // TL(HP) or null: resid + hid
    int P, NB, d, h;
    const int32_t *pmax;  // [NB] positions the longest series of a 16-series tile has: its chains stop there
    const int32_t *lengths;
    float *cs_partial;    // [4*NB * gridDim.y] (cell-state penalty, CP instantiations only)
    int B, T, I, H;
};

// positions per chunk of staged inputs: fewer where a chunk cannot be requested before the layer below has all of it
constexpr int narrow_fwd_chunk(int mode) { return mode == kLater ? 4 : 8; }

// Input half of the pre-activations, by position parity: one object for all kinds of layers of a kernel, each of which has
// arrays of its own otherwise (hidden 64, three kinds and two of 16 series: 131 200 bytes, past the 128 KB that are safe).
__device__ __forceinline__ f32x4 (&input_halves())[2][kNW][64]
{
    __shared__ f32x4 half[2][kNW][64];
    return half;
}

// Waves 0-3 carry the recurrence; waves 4-7, on the same SIMDs, bring the inputs and form the input half of the next
// position's pre-activations (with the bias), which does not depend on it: the chain then has 4 HT instead of
// 4 (KXT + HT) matrix instructions a position, and no request of its own.  Both kinds meet the same barriers.
// 512 hourly series, first layer (24 + 40 columns, 649 positions): 348 -> 331 us (333 -> 317 us for 333); 501 monthly ones
// (20 + 50 columns, 211 positions): 123 -> 115 us; 16 quarterly ones (4 + 40 columns, 61 positions): 30.3 -> 27.7 us.  (Three
// accumulators, which need no wait states between the matrix instructions: 340 us.)  What bounds it is the issue of one
// wave and what the input wave of its SIMD takes from it: without the input half 264 of 327 us.  Gates in the rows of sixteen
// lanes, which four instructions transpose (26 between the lanes of a quad), and stores through pointers that move on
// (13 scalar instructions a position instead of some 20 scalar and vector ones for addresses): 327 -> 290 us for 512 hourly
// series, 114 -> 108 us for 501 monthly ones, 27.7 -> 25.7 us for 16 quarterly ones.
//
// One workgroup: quarter q of series tile bt, residue classes chain, chain + chains, ... (of several layers in one launch:
// its only one).
// CP: the layer's cell states enter the cell-state penalty; OUT: the layer ends a residual block (reads the
// block input, writes the block output).
template <int HT, int KXT, bool CP, bool OUT, int MODE>
__device__ __forceinline__ void lstm_forward_narrow_body(const NarrowFwdArgs &a, int bt, int q, int chain, int chains, const Progress &progress)
{
    constexpr int KX = 4 * KXT, HP = 4 * HT, CH = narrow_fwd_chunk(MODE);
    constexpr int XG = (KX + 15) / 16, HG = (HP + 15) / 16;   // groups of 16 columns (one register each)
    // inputs x_p of a chunk of positions [column][series], by chunk parity (+ 64 floats that take the writes of
    // the threads with no input row, so that staging is the same instruction stream in every thread)
    __shared__ float xc[2][CH][XG * 64 + 64];
    __shared__ float rc[OUT ? 2 : 1][OUT ? CH : 1][kNT];      // residual input of a thread's (unit, series), likewise
    __shared__ float hb[2][HG * 64];            // h_{p-d} [unit][series], by position parity
    f32x4 (&half)[2][kNW][64] = input_halves();
    // positions whose stores may still be under way when the next one is counted: a position of a first layer takes less
    // time than a store
    constexpr int kBehind = MODE == kFirst ? 3 : 1, kStores = OUT ? 4 : 3;

    const int lane = threadIdx.x & 63, tid = threadIdx.x & (kNT - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = wave & (kNW - 1);
    const int blk = lane & 15, j = lane >> 4;   // unit of the wave; gate of the products, series of the cell update
    // All four workgroups of a 16-series tile stop at the tile's longest series: what lies beyond is
    // neither computed here nor read by any later kernel.
    const int Pt = a.pmax[bt];
    const int unit = w * HT + min(blk, HT - 1);     // lanes past HT repeat the last unit
    // element of this lane inside the TL(HP) block of one (position, series tile)
    const int lane_off = unit * 16 + 4 * q + j;
    // columns past KX / HP in the last group of 16 are never written: zero once (their weights do not exist)
    for (int e = threadIdx.x; e < 2 * CH * (XG * 64 + 64); e += 2 * kNT) (&xc[0][0][0])[e] = 0.0f;
    for (int e = threadIdx.x; e < 2 * HG * 64; e += 2 * kNT) (&hb[0][0])[e] = 0.0f;

    if (wave >= kNW) {
        // =========================== input waves ===========================
        float wx[KX];
#pragma unroll
        for (int k = 0; k < KX; ++k) wx[k] = a.wpack[((size_t)w * (KX + HP) + k) * 64 + lane];
        // before the transpose a lane holds gate j of its unit for the four series
        const float bias = unit < a.h ? a.bias[j * a.h + unit] : 0.0f;
        // cooperative input load: thread t < 4*KX brings row t/4 of series t%4 (the others repeat row 0)
        const bool x_thread = tid < 4 * KX;
        const int x_off = (x_thread ? tid >> 2 : 0) * 16 + 4 * q + (tid & 3);
        const int x_slot = x_thread ? tid : XG * 64 + lane;
        Below below(progress);
        for (int r = chain; r < a.d && r < Pt; r += chains) {
            const int n = (Pt - r + a.d - 1) / a.d;            // positions of this chain: r, r+d, ...
            float xs[CH], rs[CH];
            auto load_chunk = [&](int c) {
#pragma unroll
                for (int ii = 0; ii < CH; ++ii) {
                    const size_t tile = (size_t)(r + min(c * CH + ii, n - 1) * a.d) * a.NB + bt;
                    if constexpr (MODE == kLater) {
                        xs[ii] = buf_load_shared(make_rsrc(a.xsrc + tile * (KX * 16)), 4 * x_off, 0);
                        rs[ii] = OUT ? buf_load_shared(make_rsrc(a.resid + tile * (HP * 16)), 4 * lane_off, 0) : 0.0f;
                    } else {
                        xs[ii] = (a.xsrc + tile * (KX * 16))[x_off];
                        rs[ii] = OUT ? (a.resid + tile * (HP * 16))[lane_off] : 0.0f;
                    }
                }
            };
            // before a chunk is requested: the layer below has all of it
            auto await_chunk = [&](int c) {
                if constexpr (MODE == kLater) below.wait(r + min(c * CH + CH - 1, n - 1) * a.d);
            };
            // after the barrier of the i-th position
            auto count = [&](int i) {
                if constexpr (MODE != kAlone) progress.publish(max(i - kBehind, 0) * a.d, w == 0);
            };
            auto flush_chunk = [&](int c) {
#pragma unroll
                for (int ii = 0; ii < CH; ++ii) {
                    xc[c & 1][ii][x_slot] = MODE == kLater ? below.checked(xs[ii]) : xs[ii];
                    if constexpr (OUT) rc[c & 1][ii][tid] = MODE == kLater ? below.checked(rs[ii]) : rs[ii];
                }
            };
            // input half of the position in slot ii of the chunk of parity cpar, left for the position of parity par
            auto input_half = [&](int cpar, int ii, int par) {
                float vx[XG];
#pragma unroll
                for (int m = 0; m < XG; ++m) vx[m] = xc[cpar][ii][64 * m + lane];
                f32x4 acc0 = f32x4{bias, bias, bias, bias}, acc1 = f32x4{0.f, 0.f, 0.f, 0.f};
                static_for<0, KX / 2>([&](auto ic) {
                    constexpr int k = 2 * decltype(ic)::value;
                    acc0 = mfma4_bcast<k % 16>(vx[k / 16], wx[k], acc0);
                    acc1 = mfma4_bcast<(k + 1) % 16>(vx[k / 16], wx[k + 1], acc1);
                });
                half[par][w][lane] = acc0 + acc1;
            };
            await_chunk(0);
            load_chunk(0);
            __syncthreads();            // LDS free: initial clearing, or the last position of the previous chain
            flush_chunk(0);
            lds_barrier();
            input_half(0, 0, 0);
            lds_barrier();
            // Whole chunks: the body of a chunk is one straight run of instructions, and requests are staged in the run that
            // issued them, two positions before its end: the first position of the next chunk is formed in the last one.
            int c = 0;
            for (; (c + 1) * CH <= n; ++c) {
                await_chunk(c + 1);
                load_chunk(c + 1);              // (row indices stop at the chain's last position)
                static_for<0, CH>([&](auto iic) {
                    constexpr int ii = decltype(iic)::value;
                    if constexpr (ii == CH - 2) flush_chunk(c + 1);
                    if constexpr (ii == CH - 1) input_half((c + 1) & 1, 0, 0);
                    else input_half(c & 1, ii + 1, (ii + 1) & 1);
                    lds_barrier();
                    count(c * CH + ii);
                });
            }
            // the last, partial chunk
            for (int i = c * CH; i < n; ++i) {
                input_half(c & 1, min(i + 1 - c * CH, CH - 1), (i + 1) & 1);
                lds_barrier();
                count(i);
            }
            if constexpr (MODE != kAlone) {
                lds_barrier();                                 // (all stores of the chain are complete)
                progress.publish(n * a.d, w == 0);
            }
        }
        if constexpr (CP) __syncthreads();
        return;
    }

    // =========================== chain waves ===========================
    // (ahead of the input wave of the same SIMD: what that one does has a whole position's time)
    __builtin_amdgcn_s_setprio(3);
    const bool valid = blk < HT;
    float wh[HP];
#pragma unroll
    for (int k = 0; k < HP; ++k) wh[k] = a.wpack[((size_t)w * (KX + HP) + KX + k) * 64 + lane];
    int n_valid = 0;
    float csq = 0.0f;
    if constexpr (CP) {
        const int col = bt * kTileN + 4 * q + j;
        const int len = col < a.B ? min(max(a.lengths[col], 0), a.T) : 0;
        n_valid = len - a.I - a.H + 1;
    }
    for (int r = chain; r < a.d && r < Pt; r += chains) {
        const int n = (Pt - r + a.d - 1) / a.d;
        float creg = 0.0f;
        __syncthreads();
        for (int e = tid; e < 4 * HP; e += kNT) hb[0][e] = 0.0f;    // start of a chain: zero state
        lds_barrier();
        lds_barrier();
        // What a position leaves in memory is stored while the next one waits for its first operands from LDS, through
        // scalar pointers that move on by a position.
        f32x4 gates;
        float cell, hidden, output;
        const size_t first = ((size_t)r * a.NB + bt) * (HP * 16), step = (size_t)a.d * a.NB * (HP * 16);
        float *at_gates = a.gates + 4 * first, *at_c = a.c + first, *at_hid = a.hid + first, *at_out = OUT ? a.out + first : nullptr;
        auto store = [&]() {
            buf_store4<true>(make_rsrc(at_gates), 16 * lane_off, gates);
            buf_store(make_rsrc(at_c), 4 * lane_off, 0, cell);     // (plain: the four quarter-row writes of a tile then merge in L2)
            if constexpr (MODE == kAlone) {
                buf_store(make_rsrc(at_hid), 4 * lane_off, 0, hidden);
                if (OUT) buf_store(make_rsrc(at_out), 4 * lane_off, 0, output);
            } else {
                buf_store_shared(make_rsrc(at_hid), 4 * lane_off, 0, hidden);
                if (OUT) buf_store_shared(make_rsrc(at_out), 4 * lane_off, 0, output);
            }
            at_gates += 4 * step;
            at_c += step;
            at_hid += step;
            if (OUT) at_out += step;
        };
        auto position = [&](int i, auto parc, auto firstc) {
            constexpr int par = decltype(parc)::value;
            const int p = r + i * a.d;
            // h_{p-d} of the four series: lane (b, s) of register m holds unit 16m + b of series s
            float vh[HG];
#pragma unroll
            for (int m = 0; m < HG; ++m) vh[m] = hb[par][64 * m + lane];
            // two accumulators: consecutive instructions never depend on each other (measured: one, three and four are
            // slower)
            f32x4 acc0 = half[par][w][lane], acc1 = f32x4{0.f, 0.f, 0.f, 0.f};
            const float res = OUT ? rc[OUT ? (i / CH) & 1 : 0][OUT ? i % CH : 0][tid] : 0.0f;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!decltype(firstc)::value) store();
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, HP / 2>([&](auto ic) {
                constexpr int k = 2 * decltype(ic)::value;
                acc0 = mfma4_bcast<k % 16>(vh[k / 16], wh[k], acc0);
                acc1 = mfma4_bcast<(k + 1) % 16>(vh[k / 16], wh[k + 1], acc1);
            });
            f32x4 pre = acc0 + acc1;        // gate j of the unit, series 0..3
            row_transpose(pre);             // gates 0..3 of the unit, series j
            const float gi = sigmoid_f(pre[0]);
            const float gf = sigmoid_f(pre[1]);
            const float gg = tanh_f(pre[2]);
            const float go = sigmoid_f(pre[3]);
            const float cn = gf * creg + gi * gg;
            const float hn = go * tanh_f(cn);
            creg = cn;
            if constexpr (CP) csq += (valid && p < n_valid) ? cn * cn : 0.0f;
            hb[par ^ 1][4 * unit + j] = hn;
            gates = f32x4{gi, gf, gg, go};
            cell = cn;
            hidden = hn;
            output = res + hn;
            if constexpr (MODE != kAlone) stores_complete_but<kBehind * kStores>();
            lds_barrier();
        };
        using std::integral_constant;
        position(0, integral_constant<int, 0>{}, std::true_type{});
        int i = 1;
        for (; i + 1 < n; i += 2) {
            position(i, integral_constant<int, 1>{}, std::false_type{});
            position(i + 1, integral_constant<int, 0>{}, std::false_type{});
        }
        if (i < n) position(i, integral_constant<int, 1>{}, std::false_type{});
        store();
        if constexpr (MODE != kAlone) {
            stores_complete_but<0>();
            lds_barrier();
        }
    }
    if constexpr (CP) {
        __shared__ float s_cs[kNW];
        const float tot = wave_sum(csq);
        if (lane == 0) s_cs[w] = tot;
        __syncthreads();
        if (threadIdx.x == 0 && (MODE == kAlone || a.cs_partial))
            a.cs_partial[(4 * bt + q) * chains + chain] = (s_cs[0] + s_cs[1]) + (s_cs[2] + s_cs[3]);
    }
}

template <int HT, int KXT, bool CP, bool OUT>
__global__ void __launch_bounds__(2 * kNT) lstm_forward_narrow_kernel(NarrowFwdArgs a)
{
    // The four workgroups of a 16-series tile share every 64-byte row of the tile.  Consecutive workgroup
    // ids go round the 8 XCDs, each with its own L2: ids x, x+8, x+16, x+24 of a group of 32 are the four
    // quarters of ONE tile, so they land on the same XCD at about the same time and a row is fetched from
    // HBM once, not four times (measured before: 2.3-2.8 times the algorithmic bytes).
    const int bt = (blockIdx.x >> 5) * 8 + (blockIdx.x & 7), q = (blockIdx.x >> 3) & 3;
    if (bt >= a.NB) return;     // the grid is padded to whole groups of 32 (before any barrier)
    lstm_forward_narrow_body<HT, KXT, CP, OUT, kAlone>(a, bt, q, blockIdx.y, gridDim.y, Progress{});
}

template <int HT, int KXT, bool OUT>
hipError_t run_nfwd(const NarrowFwdArgs &a, int chains, hipStream_t st)
{
    const dim3 grid(narrow_grid_x(a.NB), chains);
    if (a.cs_partial) lstm_forward_narrow_kernel<HT, KXT, true, OUT><<<grid, 2 * kNT, 0, st>>>(a);
    else lstm_forward_narrow_kernel<HT, KXT, false, OUT><<<grid, 2 * kNT, 0, st>>>(a);
    return hipGetLastError();
}

inline NarrowFwdArgs narrow_forward_args(const Plan &pl, int layer, const int32_t *lengths, const float *weights, float *ws)
{
    const LayerPlan &lp = pl.layer[layer];
    const bool cp = lp.first_in_block && pl.cfg.lambda_cs != 0.0f;
    return NarrowFwdArgs{ws + lp.wpack_fwd, weights + lp.b_off, ws + lp.xsrc, ws + lp.gates, ws + lp.c, ws + lp.hid,
                    lp.out ? ws + lp.resid : nullptr, lp.out ? ws + lp.out : nullptr, pl.P, pl.NB, lp.dil, pl.h,
                    reinterpret_cast<const int32_t *>(ws + pl.pmax), lengths, cp ? ws + lp.cs_partial : nullptr, pl.B, pl.T, pl.I, pl.H};
}

template <bool OUT>
hipError_t launch_narrow_fwd(const Plan &pl, int layer, const int32_t *lengths, const float *weights, float *ws,
                             hipStream_t st)
{
    const LayerPlan &lp = pl.layer[layer];
    const NarrowFwdArgs a = narrow_forward_args(pl, layer, lengths, weights, ws);
#define X(HT_, KXT_) if (pl.HT == HT_ && lp.KXT == KXT_) return run_nfwd<HT_, KXT_, OUT>(a, lp.chains, st);
    ESRNN_LSTM_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace esrnn
