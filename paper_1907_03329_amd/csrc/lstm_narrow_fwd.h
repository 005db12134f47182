// Forward pass of a dilated LSTM layer on the 4-series kernels (see lstm_narrow_common.h for the tiling): the
// kernel template and its launcher, included by one translation unit per residual wiring (plain layer / last layer
// of a residual block) so that the two compile side by side.
#pragma once

#include "lstm_narrow_common.h"
#include "lstm_together.h"

namespace esrnn {

namespace {

struct NarrowFwdArgs {
    const float *wpack;   // [4][4*HT][64] weights of h: wave, column, lane (gate l/16 of unit l%16 of the wave), then
                          // [4][column tiles][KXT][64] those of x: columns (gate, unit of the wave)
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

// positions whose input half is formed together: the 16 rows of a matrix instruction are four positions of four series
constexpr int kInputGroup = 4;

// Input half of the pre-activations, two groups of positions: one object for all kinds of layers of a kernel, each of which has
// arrays of its own otherwise.  A place a wave takes the columns that only pad.
using InputHalves = f32x4[2][kInputGroup][kNW][64 + 1];
__device__ __forceinline__ InputHalves &input_halves()
{
    __shared__ InputHalves half;
    return half;
}

// Waves 0-3 carry the recurrence; waves 4-7, on the same SIMDs, bring the inputs and form the input half of the
// pre-activations (with the bias), which does not depend on it: x of four positions and four series is the 16 rows of
// v_mfma_f32_16x16x4, a wave's gates and units the columns, and a lane ends up with what one lane of the chain
// wave takes, four series of a gate and unit.  The chain then has 4 HT matrix instructions a position, and no request of its own.
// Both kinds meet the same barriers.
// What bounds it: the chain, 230 of 250 us without stores and input half (512 hourly series, first layer, 24 + 40 columns, 649
// positions): some 150 ns a position from the state's LDS write over the barrier to its read, 40 matrix instructions of 3.7 ns,
// the gates.  Input half on the 4x4x1 instruction, a position at a time: 295 us; 512 monthly series (12 + 50 columns, 211 positions)
// 100 -> 90 us; all layers of 16 quarterly ones in one launch 44 -> 41 us.  With three-term bf16 products the input waves need fewer
// cycles of the matrix pipe but hold 1.5 times the weights (later layers of hidden 50: 180 registers, and no second workgroup on a compute
// unit; now 125), and infinite operands become finite ones: 268 us; step of 64 hourly series 10 us more.  All columns of x requested by every
// wave: forecasts of 333 hourly series 362 instead of 345 us, forward pass of 64 monthly ones 175.9 instead of 172.6.  (With one unit tile of x,
// dealt columns cost 16 quarterly series 2 us of 64.)  Tried: stores spread over the matrix
// instructions (within 2 %), three accumulators instead of two, contraction split over the rows of a wave, ten waves (nothing gained: the
// barrier takes longer, 186 ns instead of 150).
//
// One workgroup: quarter q of series tile bt, residue classes chain, chain + chains, ... (of several layers in one launch:
// its only one).
// CP: the layer's cell states enter the cell-state penalty; OUT: the layer ends a residual block (reads the
// block input, writes the block output).
// COUNTED: a first layer counts every so many positions.
template <int HT, int KXT, bool CP, bool OUT, int MODE, int COUNTED = 1>
__device__ __forceinline__ void lstm_forward_narrow_body(const NarrowFwdArgs &a, int bt, int q, int chain, int chains, const Progress &progress)
{
    constexpr int KX = 4 * KXT, HP = 4 * HT;
    constexpr int HG = (HP + 15) / 16;          // groups of 16 columns (one register each)
    constexpr int kStoreStep = 1;          // pairs of matrix instructions between two stores
    __shared__ float rc[OUT ? 2 : 1][OUT ? kInputGroup : 1][kNT];      // residual input of a thread's (unit, series), by group of positions
    __shared__ float hb[2][HG * 64];            // h_{p-d} [unit][series], by position parity
    InputHalves &half = input_halves();
    // Every input wave needs all columns of x.  Each requests a quarter of them, a position before the products, and they meet in LDS; a
    // layer that follows another one has no position to spare, and every wave of it requests them all.
    constexpr bool kDealt = MODE != kLater && KXT > 1;
    constexpr int NX = kDealt ? (KXT + kNW - 1) / kNW : KXT;
    __shared__ float x_dealt[kDealt ? KXT : 1][64];     // [unit tile][lane of the operand]
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
    // columns past HP in the last group of 16 are never written: zero once (their weights do not exist)
    for (int e = threadIdx.x; e < 2 * HG * 64; e += 2 * kNT) (&hb[0][0])[e] = 0.0f;
    if (a.h < HP)
        for (int e = threadIdx.x; e < 2 * kInputGroup * kNW * (64 + 1); e += 2 * kNT) (&half[0][0][0][0])[e] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (wave >= kNW) {
        // =========================== input waves ===========================
        // x (16 rows: position, series) times W_x^T (columns: gate, unit of the wave)
        constexpr int TILES = (HT + 3) / 4;
        const float *wpack = a.wpack + (size_t)kNW * HP * 64 + (size_t)w * TILES * KXT * 64 + lane;
        float wx[TILES][KXT];
        float bias[TILES];
        // where a column goes: gate in rows of sixteen lanes.  (What a unit that only pads has there stays zero: infinite inputs times its
        // weights of zero would be its state.)
        int to[TILES];
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
#pragma unroll
            for (int k = 0; k < KXT; ++k) wx[t][k] = wpack[(t * KXT + k) * 64];
            const int c = 16 * t + blk, gate = c / HT, u = w * HT + c % HT;
            const bool exists = c < HP && u < a.h;
            bias[t] = exists ? a.bias[gate * a.h + u] : 0.0f;
            to[t] = exists ? 16 * gate + c % HT : 64;
        }
        Below below(progress);
        for (int r = chain; r < a.d && r < Pt; r += chains) {
            const int n = (Pt - r + a.d - 1) / a.d;            // positions of this chain: r, r+d, ...
            float xs[NX], rs[kInputGroup];
            // requests of the four positions from the i-th on (past the chain its last)
            auto request = [&](int i) {
                // before them, the layer below has all of it
                if constexpr (MODE == kLater) below.wait(r + min(i + kInputGroup - 1, n - 1) * a.d);
                const int first = min(i, n - 1), mine = min(i + (blk >> 2), n - 1) - first;     // this lane's position (not before the first)
                const size_t tile = (size_t)(r + first * a.d) * a.NB + bt;
                const int at = j * 16 + 4 * q + (blk & 3);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (MODE == kLater) {
                    // (d NB is at most 256 workgroups here: 32 bits)
                    const buf_rsrc x = make_rsrc(a.xsrc + tile * (KX * 16));
                    const int from = 4 * (mine * a.d * a.NB * (KX * 16) + at);
#pragma unroll
                    for (int k = 0; k < NX; ++k) xs[k] = buf_load_shared(x, from, 256 * k);
                } else {
                    const float *x = a.xsrc + (tile + (size_t)(mine * a.d) * a.NB) * (KX * 16) + at;
#pragma unroll
                    for (int k = 0; k < NX; ++k) xs[k] = x[64 * (kDealt ? min(w + kNW * k, KXT - 1) : k)];
                }
                if constexpr (OUT) {
#pragma unroll
                    for (int g = 0; g < kInputGroup; ++g) {
                        const buf_rsrc res = make_rsrc(a.resid + ((size_t)(r + min(i + g, n - 1) * a.d) * a.NB + bt) * (HP * 16));
                        rs[g] = MODE == kLater ? buf_load_shared(res, 4 * lane_off, 0) : buf_load(res, 4 * lane_off, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            // what has been requested: operands (in LDS, or in registers of their own, those of the requests are the next ones'), residual
            // inputs in LDS
            float xq[KXT];
            auto arrive = [&](int par) {
#pragma unroll
                for (int k = 0; k < NX; ++k) {
                    if constexpr (!kDealt) xq[k] = __builtin_canonicalizef(MODE == kLater ? below.checked(xs[k]) : xs[k]);
                    else if (w + kNW * k < KXT) x_dealt[w + kNW * k][lane] = xs[k];
                }
                if constexpr (OUT) {
#pragma unroll
                    for (int g = 0; g < kInputGroup; ++g) rc[par][g][tid] = MODE == kLater ? below.checked(rs[g]) : rs[g];
                }
            };
            // (behind a barrier after the arrival)
            auto collect = [&]() {
                if constexpr (kDealt) {
#pragma unroll
                    for (int k = 0; k < KXT; ++k) xq[k] = x_dealt[k][lane];
                }
            };
            // column tiles [from, end), left for the group of parity par: a lane has position j, its column, and four series
            auto products = [&](auto from, auto end, int par) {
                static_for<decltype(from)::value, decltype(end)::value>([&](auto tc) {
                    constexpr int t = decltype(tc)::value;
                    f32x4 sum = f32x4{bias[t], bias[t], bias[t], bias[t]};
#pragma unroll
                    for (int k = 0; k < KXT; ++k) sum = mfma16(xq[k], wx[t][k], sum);
                    half[par][j][w][to[t]] = sum;
                });
            };
            // after the barrier of the i-th position
            auto count = [&](int i) {
                if constexpr (MODE != kAlone) progress.publish(max(i - kBehind, 0) * a.d, w == 0);
            };
            using std::integral_constant;
            constexpr integral_constant<int, 0> none;
            constexpr integral_constant<int, TILES> all;
            request(0);
            __syncthreads();            // LDS free: initial clearing, or the last position of the previous chain
            arrive(0);
            if constexpr (MODE != kLater) request(kInputGroup);
            if constexpr (kDealt) lds_barrier();
            collect();
            products(none, all, 0);
            lds_barrier();
            // Four positions are one straight run of instructions, in which the next four's input half is formed.  A layer that
            // follows another one requests them here, else they have been requested in the run before.
            int i = 0, par = 1;
            if (int groups = n / kInputGroup) do {
                static_for<0, kInputGroup>([&](auto kc) {
                    constexpr int k = decltype(kc)::value;
                    if constexpr (MODE == kLater) {
                        if constexpr (k == 0) request(i + kInputGroup);
                        if constexpr (k == 2) {
                            arrive(par);
                            products(none, integral_constant<int, TILES / 2>{}, par);
                        }
                        if constexpr (k == 3) products(integral_constant<int, TILES / 2>{}, all, par);
                    } else {
                        if constexpr (k == 0) {
                            arrive(par);
                            request(i + 2 * kInputGroup);
                        } else {
                            if constexpr (k == 1) collect();
                            products(integral_constant<int, (k - 1) * TILES / 3>{}, integral_constant<int, k * TILES / 3>{}, par);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);      // (a third of the products in every position, not all in one)
                    lds_barrier();
                    if constexpr (k % COUNTED == 0) count(i + k);
                });
                i += kInputGroup;
                par ^= 1;
            } while (--groups);
            for (; i < n; ++i) {
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
    for (int k = 0; k < HP; ++k) wh[k] = a.wpack[((size_t)w * HP + k) * 64 + lane];
    const int half_lane = 16 * j + min(blk, HT - 1);
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
        if constexpr (kDealt) lds_barrier();
        lds_barrier();
        // What a position leaves in memory is stored while the next one waits for its first operands from LDS, through
        // scalar pointers that move on by a position.
        f32x4 gates;
        float cell, hidden, output;
        const size_t first = ((size_t)r * a.NB + bt) * (HP * 16), step = (size_t)a.d * a.NB * (HP * 16);
        float *at_gates = a.gates + 4 * first, *at_c = a.c + first, *at_hid = a.hid + first, *at_out = OUT ? a.out + first : nullptr;
        auto store = [&](auto partc) {
            constexpr int part = decltype(partc)::value;
            if constexpr (part == 0) {
                buf_store4<true>(make_rsrc(at_gates), 16 * lane_off, gates);
                at_gates += 4 * step;
            }
            if constexpr (part == 1) {
                buf_store(make_rsrc(at_c), 4 * lane_off, 0, cell);     // (plain: the four quarter-row writes of a tile then merge in L2)
                at_c += step;
            }
            if constexpr (part == 2) {
                if constexpr (MODE == kAlone) buf_store(make_rsrc(at_hid), 4 * lane_off, 0, hidden);
                else buf_store_shared(make_rsrc(at_hid), 4 * lane_off, 0, hidden);
                at_hid += step;
            }
            if constexpr (OUT && part == 3) {
                if constexpr (MODE == kAlone) buf_store(make_rsrc(at_out), 4 * lane_off, 0, output);
                else buf_store_shared(make_rsrc(at_out), 4 * lane_off, 0, output);
                at_out += step;
            }
        };
        int p = r, group = 0;           // (parity of the group of positions)
        auto position = [&](auto kc, auto firstc) {
            constexpr int k = decltype(kc)::value, par = k & 1;
            // h_{p-d} of the four series: lane (b, s) of register m holds unit 16m + b of series s
            float vh[HG];
#pragma unroll
            for (int m = 0; m < HG; ++m) vh[m] = hb[par][64 * m + lane];
            // two accumulators: consecutive instructions never depend on each other (measured: one, three and four are
            // slower)
            f32x4 acc0 = half[group][k][w][half_lane], acc1 = f32x4{0.f, 0.f, 0.f, 0.f};
            const float res = OUT ? rc[OUT ? group : 0][OUT ? k : 0][tid] : 0.0f;
            static_for<0, HP / 2>([&](auto ic) {
                constexpr int i = decltype(ic)::value, k = 2 * i;
                // (a store between two matrix instructions: 275 -> 268 us)
                if constexpr (!decltype(firstc)::value && i % kStoreStep == 0 && i / kStoreStep < 4) {
                    __builtin_amdgcn_sched_barrier(0);
                    store(std::integral_constant<int, i / kStoreStep>{});
                    __builtin_amdgcn_sched_barrier(0);
                }
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
            p += a.d;
            if constexpr (MODE != kAlone) stores_complete_but<kBehind * kStores>();
            lds_barrier();
        };
        using std::integral_constant;
        // (the first position has nothing to store yet)
        position(integral_constant<int, 0>{}, std::true_type{});
        int left = n - 1;
        while (left > 0) {
            // positions 1, 2, 3 of a group and 0 of the next one
            position(integral_constant<int, 1>{}, std::false_type{});
            if (left == 1) break;
            position(integral_constant<int, 2>{}, std::false_type{});
            if (left == 2) break;
            position(integral_constant<int, 3>{}, std::false_type{});
            if (left == 3) break;
            group ^= 1;
            position(integral_constant<int, 0>{}, std::false_type{});
            left -= 4;
        }
        static_for<0, 4>(store);
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

// (four waves a SIMD, two workgroups a compute unit)
template <int HT, int KXT, bool CP, bool OUT>
__global__ void __launch_bounds__(2 * kNT, 4) lstm_forward_narrow_kernel(NarrowFwdArgs a)
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
