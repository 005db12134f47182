// Forward pass of a dilated LSTM layer (Section 3.2, Table 1), 16 series per workgroup: the kernel template and its
// launcher, included by one translation unit per kind of layer so that they compile side by side.
//
// Parallel structure.  Series never interact, and a layer with dilation d is d independent recurrences over the
// interleaved position classes p = r (mod d).  A workgroup owns 16 series and one or more residue classes r (grid =
// series tiles x chains) and walks each class in order with the recurrent state on chip: h through LDS, c in
// registers.  No grid-level synchronisation, no recurrent traffic through global memory.
//
// Arithmetic.  The gate contraction W [x_p ; h_{p-d}] runs on the bf16 matrix pipe with fp32 accuracy (three_term.h):
// the weights are the A operand, split once per call by the set-up kernel and held in registers for the whole launch;
// the activations of the 16 series are the B operand, split by the wave that loads (x) or computes (h) them and
// handed to the others through LDS.  Row order of the A operand: row 4g+r of unit tile mt is gate r of hidden unit
// 4mt+g, so that a lane holds the four gate pre-activations of one unit of one series and the cell update needs no
// cross-lane traffic.  Of W waves, wave s owns the unit tiles s and s + W and brings the input tiles W - 1 - s and
// 2 W - 1 - s (the waves with a unit tile fewer bring an input tile more).
//
// The bias is added last, by the multiply-add that scales a pre-activation for its exponential; only what the rounding of
// the scaled bias leaves out goes in with the products.  Products added to the bias would all be rounded at its size, and
// not at random: inputs and states vary little, so the sum of their leading parts takes few values, and what rounding
// cuts off the bias is the same at every position.  Against float64, mean error of a unit's pre-activations over 2624
// positions, biases around 1.5, hidden 32 to 64: 8 - 11e-8 (bias first 10 - 17e-8, fp32 matrix instruction 8 - 11e-8), rms
// 36 - 51e-8 (44 - 65e-8, 46 - 68e-8).  No vector instruction more than with the bias first (forecasts 1 % faster).
//
// Order of a position: the recurrent half, on top of the input half formed one position earlier; the cell update,
// whose hidden state goes to LDS; then the input half of the next position, which does not depend on the recurrence
// and fills the matrix pipe while the waves run apart; the input of the position after that goes from registers to
// LDS and the one after it is requested.  One barrier per position.
//
// What bounds it: the activation stash.  A position writes 6 h floats per series (activated gates, cell, hidden) and
// reads its input; at 4096 series and hidden 40 that is 281 MB a layer (361 MB with the block's residual read and
// written), 50 us at the rates a plain stream of stores or loads reaches here (5.3 - 6.3 TB/s and 6.4 - 6.8 TB/s).
// Measured: 52 - 55 us (64 - 70 us with the residual); with the fp32 matrix instruction 72 us, bound by the issue of
// matrix and vector instructions.  Monthly shape (240 steps, hidden 50, 1.26 GB a layer, 1.64 GB with the residual):
// 350 - 355 us (380 - 390 us).  First layers 61 us from 79 us and 240 - 255 us from 338 us.
#pragma once

#include "esrnn_internal.h"
#include "lstm_together.h"
#include "three_term.h"

namespace esrnn {

namespace {

struct LstmFwdArgs {
    const u32x4 *wpack;   // [HT][quads of x, then of h][64]
    const float *bpack;   // [HT][4][4]
    const float *xsrc;    // TL(4*KXT)
    float *gates;         // [P][NB][HT][64][4]
    float *c, *hid;       // TL(HP)
    const float *resid;   // TL(HP)                  (layers that end a residual block)
    float *out;           // TL(HP): resid + hid
    int NB, d;
    const int32_t *pmax;  // [NB] positions the longest series of a tile has: the tile's chains stop there
    // cell-state penalty (Section 8.4) of a block's first layer
    const int32_t *lengths;
    float *cs_partial;    // [NB * gridDim.y] sums of squared cell states over valid window positions
    int B, T, I, H;
    int stash;            // 0: no reverse pass follows, gates and cell states stay on chip
    const unsigned *need; // [NB][kNeedWords] residue classes to compute (null: all)
};

// LDS home of the three parts of a 4-row operand tile, [quad][dword][lane] with two bf16 per dword.  SEG: the tiles
// 8 SEG .. 8 SEG + 7 of an operand of NP pairs of tiles.
template <int NP, int SEG>
struct TileHome {
    static constexpr int full = tt_full(NP), rest = tt_rest(NP);
    static constexpr bool in_full = SEG < full;
    // byte offset of this lane's element of the tile
    static __device__ __forceinline__ unsigned at(int tile, int lane)
    {
        const int i = tile & 7;
        if (in_full) return SEG * 3 * 1024 + (i >> 1) * 256 + (i & 1) * 2 + lane * 4;
        return full * 3 * 1024 + (rest == 2 ? (i >> 1) * 256 : 0) + (i & 1) * 2 + lane * 4;
    }
    static __device__ __forceinline__ void store(char *buf, unsigned at, float v)
    {
        const Parts p = split_pair(v, v);
        auto put = [&](int off, unsigned x) { *reinterpret_cast<unsigned short *>(buf + at + off) = (unsigned short)x; };
        if constexpr (in_full) {
            put(0, p.hi); put(1024, p.mid); put(2048, p.lo);
        } else if constexpr (rest == 1) {
            put(0, p.hi); put(256, p.mid); put(512, p.lo); put(768, p.hi);
        } else {
            put(0, p.hi); put(512, p.mid); put(1024, p.lo); put(1536, p.hi);
        }
    }
};

// Waves of a workgroup.  Up to ten unit tiles: eight (wave s owns the tiles s and s + 8), two workgroups per compute
// unit.  More: one wave per tile - with two tiles the weights of a wave take more than 128 registers, and a second
// workgroup no longer fits beside it (hidden 50 at 4096 series, 240 steps: 254 / 335 / 362 us for layers 0, 1, 2 with
// eight waves, 257 / 319 / 340 us with thirteen; hidden 40, 72 steps: 52 us with eight, 56 us with ten).
constexpr int fwd_waves(int HT) { return HT <= 10 ? 8 : HT; }

// One workgroup of W waves: series tile bt, residue classes chain, chain + chains, ...
// CP: the layer's cell states enter the cell-state penalty; OUT: the layer ends a residual block (reads the block
// input, writes the block output); STASH: a reverse pass may follow - without it gates and cell states stay on chip, and
// only the residue classes that are asked for are computed.  (An instantiation of its own: a switch at run time cost the
// layers of a training step 3 us each.)  LATER: the layer below runs in the same launch (lstm_together.h).
template <int HT, int KXT, int W, bool CP, bool OUT, bool STASH, bool LATER>
__device__ __forceinline__ void lstm_forward_body(const LstmFwdArgs &a, int bt, int chain, int chains, const Progress &progress)
{
    constexpr int NPX = (KXT + 1) / 2, NPH = (HT + 1) / 2;
    constexpr int AX = tt_a_quads(NPX), AH = tt_a_quads(NPH), BX = tt_b_quads(NPX), BH = tt_b_quads(NPH);
    constexpr int MTW = (HT + W - 1) / W, XTW = (KXT + W - 1) / W;   // unit tiles and input tiles per wave
    static_assert(W == 8 || (MTW == 1 && XTW == 1), "tile s + W j lies in segment j, or there is one tile");
    __shared__ __align__(16) char h_lds[2][BH * 1024];               // parts of h_{p-d}, by position parity
    __shared__ __align__(16) char x_lds[2][BX * 1024];               // parts of x_p
    __shared__ f32x4 rest_lds[HT][4];                                // what the rounding of that left out of the bias

    const int lane = threadIdx.x & 63;
    const int s = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave index, known to be uniform
    const int sx = W - 1 - s;                                        // first input tile of this wave
    const int Pt = a.pmax[bt];      // positions past the tile's longest series are never computed (nor read later)
    unsigned long long need = ~0ull;
    if constexpr (!STASH) {
        need = needed_classes(a.need, bt, chain, chains, a.d);
        if (need == 0) return;                                       // (before any barrier)
    }

    u32x4 wx[MTW][AX], wh[MTW][AH];
    f32x4 scaled[MTW];                                               // the bias as the exponentials take it
#pragma unroll
    for (int j = 0; j < MTW; ++j) {
        const int mt = min(s + W * j, HT - 1);                       // (a tile past HT is never computed)
        const u32x4 *w = a.wpack + (size_t)mt * (AX + AH) * 64 + lane;
#pragma unroll
        for (int q = 0; q < AX; ++q) wx[j][q] = w[q * 64];
#pragma unroll
        for (int q = 0; q < AH; ++q) wh[j][q] = w[(AX + q) * 64];
        const float4 bv = *reinterpret_cast<const float4 *>(a.bpack + (mt * 4 + (lane >> 4)) * 4);
        const float b[4] = {bv.x, bv.y, bv.z, bv.w};
        f32x4 rest;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float k = r == 2 ? kTanhExponent : kSigmoidExponent;
            scaled[j][r] = b[r] * k;
            // (nothing is left out of an infinite one, and inf - inf would be NaN)
            rest[r] = __builtin_isinf(scaled[j][r]) ? 0.0f : __builtin_fmaf(b[r], k, -scaled[j][r]) * (1.0f / k);
        }
        if ((lane & 15) == 0 && s + W * j < HT) rest_lds[mt][lane >> 4] = rest;
    }
    // halves of pairs that no tile fills stay zero
    for (int i = threadIdx.x; i < 2 * BH * 256; i += 64 * W) reinterpret_cast<unsigned *>(h_lds)[i] = 0u;
    for (int i = threadIdx.x; i < 2 * BX * 256; i += 64 * W) reinterpret_cast<unsigned *>(x_lds)[i] = 0u;

    // positions below this take part in the loss for this lane's series (CP only)
    int n_valid = 0;
    // sums of squared cell states, as the waves of the layer's own launch have them: by tile where they have one each
    constexpr int CS = W < fwd_waves(HT) ? MTW : 1;
    float csq[CS] = {};
    if constexpr (CP) {
        const int col = bt * kTileN + (lane & 15);
        const int len = col < a.B ? min(max(a.lengths[col], 0), a.T) : 0;
        n_valid = len - a.I - a.H + 1;
    }
    const unsigned lane4 = 4 * lane, lane16 = 16 * lane;             // this lane's bytes inside a tile

    // All chains of this workgroup, for a wave with NJ unit tiles, the first one in segment SH of its operand, and
    // NX input tiles, the first one in segment SX.  All are compile-time numbers so that a position is one straight
    // run of instructions, and the wait for an input counts exactly the stores issued since it was requested (memory
    // operations complete in order; behind a branch the wait also covers the newest stores: 0.72 us a position at 16
    // series instead of 0.60).
    Below below(progress);
    auto walk = [&](auto njc, auto nxc, auto shc, auto sxc) {
        constexpr int NJ = decltype(njc)::value, NX = decltype(nxc)::value;
        constexpr int SH = decltype(shc)::value, SX = decltype(sxc)::value;
        unsigned h_at[MTW], x_at[XTW];
        static_for<0, NJ>([&](auto jc) { constexpr int j = decltype(jc)::value; h_at[j] = TileHome<NPH, SH + j>::at(s, lane); });
        static_for<0, NX>([&](auto jc) { constexpr int j = decltype(jc)::value; x_at[j] = TileHome<NPX, SX + j>::at(sx, lane); });
        auto load_x = [&](int p, float (&v)[XTW]) {
            if constexpr (LATER && NX > 0) below.wait<kWidePollSleep>(min(p, Pt - 1));
            const buf_rsrc rx = make_rsrc(a.xsrc + ((size_t)min(p, Pt - 1) * a.NB + bt) * (KXT * 64));
#pragma unroll
            for (int j = 0; j < NX; ++j) v[j] = LATER ? buf_load_shared(rx, lane4, (sx + W * j) * 256) : buf_load(rx, lane4, (sx + W * j) * 256);
            if constexpr (LATER && NX > 0) below.look();       // (for the next time: what it brings is not waited for here)
        };
        auto store_x = [&](int buf, const float (&v)[XTW]) {
            static_for<0, NX>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                TileHome<NPX, SX + j>::store(x_lds[buf], x_at[j], splittable(LATER ? below.checked(v[j]) : v[j]));
            });
        };
        auto load_res = [&](int p, float (&v)[MTW]) {
            if constexpr (OUT) {
                if constexpr (LATER && NX == 0) below.wait<kWidePollSleep>(min(p, Pt - 1));
                const buf_rsrc rr = make_rsrc(a.resid + ((size_t)min(p, Pt - 1) * a.NB + bt) * HT * 64);
#pragma unroll
                for (int j = 0; j < NJ; ++j) v[j] = LATER ? buf_load_shared(rr, lane4, (s + W * j) * 256) : buf_load(rr, lane4, (s + W * j) * 256);
            }
        };
        auto read_quad = [&](const char *buf, int q) {
            u32x4 v;
#pragma unroll
            for (int d = 0; d < 4; ++d) v[d] = reinterpret_cast<const unsigned *>(buf)[(q * 4 + d) * 64 + lane];
            return v;
        };
        f32x4 acc[MTW];
        // acc = Wx x (+ the rest of the bias), from the parts in x_lds[buf]
        auto input_part = [&](int buf) {
            u32x4 b[BX];
#pragma unroll
            for (int q = 0; q < BX; ++q) b[q] = read_quad(x_lds[buf], q);
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[j] = rest_lds[min(s + W * j, HT - 1)][lane >> 4];
            static_for<0, tt_mfmas(NPX)>([&](auto ic) {
                constexpr TtPair t = tt_mfma(NPX, decltype(ic)::value);
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[j] = mfma_bf16(wx[j][t.a], b[t.b], acc[j]);
            });
        };

        for (int r = chain; r < a.d && r < Pt; r += chains) {
            if constexpr (!STASH) {
                const bool want = need & 1;
                need = need >> 1 | 1ull << 63;
                if (!want) continue;
            }
            // start of a chain: zero state, input part of the first position, parts of the second input in LDS
            float creg[MTW], xv[XTW], x1[XTW];
#pragma unroll
            for (int j = 0; j < NJ; ++j) creg[j] = 0.0f;
            load_x(r, xv);
            load_x(r + a.d, x1);
            __syncthreads();            // LDS free: initial clearing, or the last position of the previous chain
            for (int i = threadIdx.x; i < BH * 256; i += 64 * W) reinterpret_cast<unsigned *>(h_lds[0])[i] = 0u;
            store_x(0, xv);
            store_x(1, x1);
            load_x(r + 2 * a.d, xv);
            // residual input of the block: this position's, and the next one's on its way
            float res[MTW], res1[MTW];
            load_res(r, res);
            load_res(r + a.d, res1);
            lds_barrier();
            input_part(0);
            lds_barrier();              // x_lds[0] is written again in the first position

            int par = 0;
            for (int p = r; p < Pt; p += a.d, par ^= 1) {
                // this position's tiles of the stash and the outputs: scalar bases, scalar tile offsets
                const size_t pb = (size_t)p * a.NB + bt;
                const buf_rsrc r_c = make_rsrc(a.c + pb * HT * 64), r_hid = make_rsrc(a.hid + pb * HT * 64);
                // recurrent part
                {
                    u32x4 b[BH];
#pragma unroll
                    for (int q = 0; q < BH; ++q) b[q] = read_quad(h_lds[par], q);
                    static_for<0, tt_mfmas(NPH)>([&](auto ic) {
                        constexpr TtPair t = tt_mfma(NPH, decltype(ic)::value);
#pragma unroll
                        for (int j = 0; j < NJ; ++j) acc[j] = mfma_bf16(wh[j][t.a], b[t.b], acc[j]);
                    });
                }
                static_for<0, NJ>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    const int mt = s + W * j;
                    const float gi = sigmoid_of_exponent(acc[j][0] * kSigmoidExponent + scaled[j][0]);
                    const float gf = sigmoid_of_exponent(acc[j][1] * kSigmoidExponent + scaled[j][1]);
                    const float gg = tanh_of_exponent(acc[j][2] * kTanhExponent + scaled[j][2]);
                    const float go = sigmoid_of_exponent(acc[j][3] * kSigmoidExponent + scaled[j][3]);
                    const float cn = gf * creg[j] + gi * gg;
                    const float hn = go * tanh_f(cn);
                    creg[j] = cn;
                    if constexpr (CP) csq[CS > 1 ? j : 0] += p < n_valid ? cn * cn : 0.0f;
                    TileHome<NPH, SH + j>::store(h_lds[par ^ 1], h_at[j], hn);
                    // gates and cell state are read again only by the reverse pass: streaming stores
                    if constexpr (STASH) {
                        buf_store4<true>(make_rsrc(a.gates + (pb * HT + mt) * 256), lane16, f32x4{gi, gf, gg, go});
                        buf_store<true>(r_c, lane4, mt * 256, cn);
                    }
                    buf_store(r_hid, lane4, mt * 256, hn);
                    if constexpr (OUT) buf_store(make_rsrc(a.out + pb * HT * 64), lane4, mt * 256, (LATER ? below.checked(res[j]) : res[j]) + hn);
                });
                input_part(par ^ 1);
                store_x(par, xv);
                load_x(p + 3 * a.d, xv);
                if constexpr (OUT) {
#pragma unroll
                    for (int j = 0; j < NJ; ++j) res[j] = res1[j];
                    load_res(p + 2 * a.d, res1);
                }
                lds_barrier();
            }
        }
    };
    // (wave-uniform choices; every version meets the same barriers)
    using std::integral_constant;
    constexpr bool kTwo = W != 8 && HT > 8, kTwoX = W != 8 && KXT > 8;   // one tile per wave, operand of two segments
    auto with_x = [&](auto njc, auto shc) {
        if (sx + W * (XTW - 1) >= KXT) walk(njc, integral_constant<int, XTW - 1>{}, shc, integral_constant<int, 0>{});
        else if (kTwoX && sx >= 8) walk(njc, integral_constant<int, XTW>{}, shc, integral_constant<int, kTwoX ? 1 : 0>{});
        else walk(njc, integral_constant<int, XTW>{}, shc, integral_constant<int, 0>{});
    };
    if (s + W * (MTW - 1) >= HT) with_x(integral_constant<int, MTW - 1>{}, integral_constant<int, 0>{});
    else if (kTwo && s >= 8) with_x(integral_constant<int, MTW>{}, integral_constant<int, kTwo ? 1 : 0>{});
    else with_x(integral_constant<int, MTW>{}, integral_constant<int, 0>{});
    if constexpr (CP) {
        constexpr int N = fwd_waves(HT);
        __shared__ float s_cs[W * CS];
#pragma unroll
        for (int j = 0; j < CS; ++j) {
            const float tot = wave_sum(csq[j]);
            if (lane == 0) s_cs[s + W * j] = tot;
        }
        __syncthreads();
        if (threadIdx.x == 0 && (!LATER || a.cs_partial)) {
            float t = 0.0f;
            for (int i = 0; i < N; ++i) t += s_cs[i];
            a.cs_partial[bt * chains + chain] = t;
        }
    }
}

template <int HT, int KXT, bool CP, bool OUT, bool STASH>
__global__ void __launch_bounds__(64 * fwd_waves(HT), 4) lstm_forward_kernel(LstmFwdArgs a)
{
    lstm_forward_body<HT, KXT, fwd_waves(HT), CP, OUT, STASH, false>(a, blockIdx.x, blockIdx.y, gridDim.y, Progress{});
}

template <int HT, int KXT, bool OUT>
hipError_t run_fwd(const LstmFwdArgs &a, int chains, hipStream_t st)
{
    const dim3 grid(a.NB, chains);
    // (with the cell-state penalty there is only the general kernel: it writes the stash and computes every class)
    if (a.cs_partial) lstm_forward_kernel<HT, KXT, true, OUT, true><<<grid, 64 * fwd_waves(HT), 0, st>>>(a);
    else if (a.stash) lstm_forward_kernel<HT, KXT, false, OUT, true><<<grid, 64 * fwd_waves(HT), 0, st>>>(a);
    else lstm_forward_kernel<HT, KXT, false, OUT, false><<<grid, 64 * fwd_waves(HT), 0, st>>>(a);
    return hipGetLastError();
}

inline LstmFwdArgs forward_args(const Plan &pl, int layer, const int32_t *lengths, float *ws, const ForwardMode &mode)
{
    const LayerPlan &lp = pl.layer[layer];
    const bool cp = lp.first_in_block && pl.cfg.lambda_cs != 0.0f;
    return LstmFwdArgs{reinterpret_cast<const u32x4 *>(ws + lp.wpack_fwd), ws + lp.bias_pack, ws + lp.xsrc, ws + lp.gates,
                       ws + lp.c, ws + lp.hid, lp.out ? ws + lp.resid : nullptr, lp.out ? ws + lp.out : nullptr, pl.NB,
                       lp.dil, reinterpret_cast<const int32_t *>(ws + pl.pmax), lengths, cp ? ws + lp.cs_partial : nullptr,
                       pl.B, pl.T, pl.I, pl.H, mode.stash ? 1 : 0,
                       mode.need ? mode.need + (size_t)layer * pl.NB * kNeedWords : nullptr};
}

}  // namespace

}  // namespace esrnn
