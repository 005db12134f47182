// Reverse pass of a dilated LSTM layer on the 4-series kernels: the kernel template and its launcher, included by
// one translation unit per kind of workgroup (four waves / eight waves) so that the two compile side by side.
#pragma once

#include "lstm_narrow_common.h"
#include "lstm_together.h"

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
//   C. dW += da (x) [x_p ; h_{p-d}]: one 16x16x4 MFMA per 16x16 tile of dW, k =
//      the four series; row tiles dealt to the waves round-robin.
// da_all and part alternate between two copies by position parity: what a
// position writes was last read two positions earlier, one barrier ago.  The
// staged operands of a chunk of positions: per-thread values (gates, cell
// states, arriving gradient) in a buffer that the same thread reads, or with
// eight waves that of the chain wave with the same number, in two by chunk parity;
// [x ; h] rows, which the whole workgroup reads, in two buffers by chunk parity.
// ---------------------------------------------------------------------------
struct NarrowBwdArgs {
    const float *wpack;   // [4][NG][4*HT][64]  operands of W^T: wave, column group, k-step (unit, gate), lane = column
    const float *xsrc;    // TL(4*KXT)
    const float *gates, *c;
    ptrdiff_t hid_minus_xsrc;   // hidden states TL(HP), as an offset in floats from xsrc (both lie in the workspace)
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
// SPLIT: eight waves.  Waves 0-3 carry the recurrence: steps A and B and the sums of the recurrent gradient, nothing else.
// Waves 4-7 request and stage all operands, and one barrier behind the recurrence do step C, the weight gradient, and sum
// and store the input gradient.  Both kinds take the same barriers (one per position).  For grids of at most one workgroup
// per compute unit: a chain wave is bound by the instructions it issues, and the SIMDs have the other waves' work while it
// waits.  (With requests, staging and input gradient on the chain waves the first layer of 512 hourly series took 491 us,
// now 440; that of 501 monthly ones 247 us, now 221; that of 16 quarterly ones 43.6 us, now 39.7.)
// MODE: kLater, layers of one launch (lstm_together.h): this layer waits for the one above it, and its positions are counted; kLast,
// nobody waits for this one.
// Positions per chunk of staged operands, and places for them: two chunks where one wave writes and another reads.  Fewer in layers
// that follow another one in their launch, which request a chunk when the layer above has all of it (16 quarterly series, step 155.5
// -> 152.3 us, 100 178.5 -> 176.5 us); but not in the launch's last layer, whose chain of neighbouring positions has no time
// for a round trip every two of them (161.5 us; 20 hourly series 1017 -> 1176 us).
constexpr int narrow_bwd_chunk(int mode) { return mode == kLater ? 2 : 4; }
// Chunks of [x ; h] rows held: with two positions a chunk the next one is staged while step C of the one before the present is under way.
constexpr int narrow_bwd_rows(int mode) { return narrow_bwd_chunk(mode) == 2 ? 4 : 2; }
constexpr int narrow_bwd_slots(bool split, int mode) { return (split ? 2 : 1) * narrow_bwd_chunk(mode); }

template <int HT, int KXT, bool SPLIT, int MODE>
struct NarrowBwdLds {                                   // (references: an object each where nothing else has to fit)
    static constexpr int KX = 4 * KXT, HP = 4 * HT, KT4 = KX + HP;
    static constexpr int CH = narrow_bwd_chunk(MODE);
    static constexpr int NG = (KT4 + 63) / 64;          // groups of 64 columns of [x ; h]
    static constexpr int CT = (KT4 + 15) / 16;          // 16-column tiles of dW
    float (&da_all)[2][HP * 16];             // [unit][series][gate]
    float (&part)[2][kNW][NG * 64 * 4];        // partial W^T da of every wave [column][series]
    f32x4 (&lc)[narrow_bwd_slots(SPLIT, MODE)][2][kNT];   // per thread: activated gates; c, c_{p-d}, two gradient sources
    float (&xhc)[narrow_bwd_rows(MODE)][CH][CT * 64];                        // [column of x_p ; h_{p-d}][series]
    static constexpr size_t at_part = sizeof(float) * 2 * HP * 16, at_lc = at_part + sizeof(float) * 2 * kNW * NG * 64 * 4,
                            at_xhc = at_lc + sizeof(f32x4) * narrow_bwd_slots(SPLIT, MODE) * 2 * kNT, bytes = at_xhc + sizeof(float) * narrow_bwd_rows(MODE) * CH * CT * 64;
    static __device__ __forceinline__ NarrowBwdLds in(char *at)
    {
        return {reinterpret_cast<float (&)[2][HP * 16]>(*at), reinterpret_cast<float (&)[2][kNW][NG * 64 * 4]>(at[at_part]),
                reinterpret_cast<f32x4 (&)[narrow_bwd_slots(SPLIT, MODE)][2][kNT]>(at[at_lc]), reinterpret_cast<float (&)[narrow_bwd_rows(MODE)][CH][CT * 64]>(at[at_xhc])};
    }
};

// One workgroup: quarter q of series tile bt, residue classes chain, chain + chains, ...
template <int HT, int KXT, bool CP, bool SPLIT, int MODE>
__device__ __forceinline__ void lstm_backward_narrow_body(const NarrowBwdArgs &a, const NarrowBwdLds<HT, KXT, SPLIT, MODE> &lds, int bt, int q,
                                                          int chain, int chains, const Progress &progress)
{
    using Lds = NarrowBwdLds<HT, KXT, SPLIT, MODE>;
    static_assert(SPLIT || MODE == kAlone, "");
    constexpr bool kWaits = MODE != kAlone, kCounts = MODE == kLater;
    constexpr int KX = Lds::KX, HP = Lds::HP, KT4 = Lds::KT4, CH = Lds::CH, NG = Lds::NG, CT = Lds::CT;
    constexpr int MTW = (HT + kNW - 1) / kNW;    // 16-row tiles of dW per wave (a row tile = 4 units x 4 gates)
    constexpr int XH_PER = (4 * KT4 + kNT - 1) / kNT;
    constexpr int SLOTS = narrow_bwd_slots(SPLIT, MODE), ROWS = narrow_bwd_rows(MODE);

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = SPLIT ? (wv & (kNW - 1)) : wv;
    const bool dw_wave = SPLIT && wv >= kNW;
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
    // operands of the weight-gradient tiles inside 64 consecutive floats of da_all / xhc
    const int ar_off = 16 * (lane & 3) + 4 * (lane >> 4) + ((lane & 15) >> 2);   // unit l%4, series l/16, gate (l%16)/4
    const int xb_off = 4 * (lane & 15) + (lane >> 4);                            // column l%16, series l/16

    f32x4 dw[MTW][CT];
#pragma unroll
    for (int t = 0; t < MTW; ++t)
#pragma unroll
        for (int nb = 0; nb < CT; ++nb) dw[t][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 dbacc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int e = threadIdx.x; e < ROWS * CH * CT * 64; e += SPLIT ? 2 * kNT : kNT) (&lds.xhc[0][0][0])[e] = 0.0f;   // columns past KT4 stay zero

    auto store_dw = [&]() {
        const size_t partix = (size_t)(4 * bt + q) * chains + chain;
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
            const int mt = w + kNW * t;
            if (mt < HT) {
#pragma unroll
                for (int nb = 0; nb < CT; ++nb) {
                    float *dst = a.dw_partial + (partix * (HT * CT) + mt * CT + nb) * 256 + lane;
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) dst[rr * 64] = dw[t][nb][rr];
                }
            }
        }
    };
    // ---- requests and staging of a chunk: the c * CH + ii-th positions from the end of a chain that ends at p_last and has
    // n positions (requests past the chain repeat the last)
    Below above(progress);
    f32x4 s_gt[CH], s_o[CH];     // (native vectors: arrays of the HIP float4 class do not stay in registers)
    float s_xh[CH][XH_PER];
    auto load_chunk = [&](int c, int n, int p_last) {
#pragma unroll
        for (int ii = 0; ii < CH; ++ii) {
            const int p = p_last - min(c * CH + ii, n - 1) * a.d;
            const size_t pb = (size_t)p * a.NB + bt;
            const size_t pbd = (size_t)(p >= a.d ? p - a.d : p) * a.NB + bt;
            const size_t e = pb * (HP * 16) + lane_off;
            s_gt[ii] = reinterpret_cast<const f32x4 *>(a.gates)[e];
            const float g0 = kWaits ? buf_load_shared(make_rsrc(a.gsrc[0] + pb * (HP * 16)), 4 * lane_off, 0) : a.gsrc[0][e];
            const float g1 = kWaits ? buf_load_shared(make_rsrc(a.gsrc[1] + pb * (HP * 16)), 4 * lane_off, 0) : a.gsrc[1][e];
            s_o[ii] = f32x4{a.c[e], a.c[pbd * (HP * 16) + lane_off], g0, g1};
#pragma unroll
            for (int k = 0; k < XH_PER; ++k) {
                const int el = min(tid + k * kNT, 4 * KT4 - 1);
                const int col = el >> 2, jj = el & 3;
                // one base pointer and a per-lane offset (a per-lane choice between two pointers would be
                // fetched from the argument block in memory, with a wait, before every request)
                const ptrdiff_t off = col < KX ? (ptrdiff_t)((pb * KX + col) * 16)
                                               : a.hid_minus_xsrc + (ptrdiff_t)((pbd * HP + (col - KX)) * 16);
                s_xh[ii][k] = a.xsrc[off + 4 * q + jj];
            }
        }
    };
    auto flush_chunk = [&](int c, int n, int p_last) {
#pragma unroll
        for (int ii = 0; ii < CH; ++ii) {
            const bool has_prev = p_last - min(c * CH + ii, n - 1) * a.d >= a.d;
            const int slot = SPLIT ? (c & 1) * CH + ii : ii;
            lds.lc[slot][0][tid] = s_gt[ii];
            if constexpr (kWaits) s_o[ii][2] = above.checked(s_o[ii][2]);
            lds.lc[slot][1][tid] = s_o[ii];
#pragma unroll
            for (int k = 0; k < XH_PER; ++k) {
                const int el = tid + k * kNT;
                if (el < 4 * KT4) lds.xhc[c & (ROWS - 1)][ii][el] = (el < 4 * KX || has_prev) ? s_xh[ii][k] : 0.0f;
            }
        }
    };
    // ---- sum and store of one position's input gradient
    auto input_gradient = [&](int p, int par) {
        const float dxv = (lds.part[par][0][dx_el] + lds.part[par][1][dx_el]) + (lds.part[par][2][dx_el] + lds.part[par][3][dx_el]);
        float *to = a.gdst + ((size_t)p * a.NB + bt) * (KX * 16);
        const int at = (dx_el >> 2) * 16 + 4 * q + (dx_el & 3);
        if constexpr (kCounts) buf_store_shared(make_rsrc(to), 4 * at, 0, dxv);
        else to[at] = dxv;
    };
    // ---- C: weight gradient of one position, k = the four series; da in lds.da_all[par], [x ; h] in lds.xhc[cpar][ii]
    auto step_c = [&](int par, int cpar, int ii) {
        float xb[CT];
#pragma unroll
        for (int nb = 0; nb < CT; ++nb) xb[nb] = lds.xhc[cpar][ii][64 * nb + xb_off];
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
            const int mt = w + kNW * t;
            if (mt < HT) {
                // row 4*gate + u of the tile is gate `gate` of unit 4*mt + u
                const float ar = lds.da_all[par][64 * mt + ar_off];
#pragma unroll
                for (int nb = 0; nb < CT; ++nb) dw[t][nb] = mfma16(ar, xb[nb], dw[t][nb]);
            }
        }
    };
    if constexpr (SPLIT) {
        if (dw_wave) {
            // the same barriers as the chain waves below: start of a chain, first staging, one per position
            for (int r0 = chain; r0 < a.d && r0 < Pt; r0 += chains) {
                const int n = (Pt - r0 + a.d - 1) / a.d, p_last = r0 + (n - 1) * a.d;
                // the layer above has all of a chunk before it is requested
                auto await_chunk = [&](int c) {
                    if constexpr (kWaits) above.wait_falling(p_last - min(c * CH + CH - 1, n - 1) * a.d, Pt);
                };
                auto complete_but = [&](auto stores) {
                    if constexpr (kCounts) stores_complete_but<decltype(stores)::value>();
                };
                auto count = [&](int positions) {
                    if constexpr (kCounts) progress.publish(max(positions, 0) * a.d, w == 0);
                };
                using std::integral_constant;
                await_chunk(0);
                load_chunk(0, n, p_last);
                __syncthreads();
                flush_chunk(0, n, p_last);
                lds_barrier();
                int c = 0;
                for (; (c + 1) * CH <= n; ++c) {
                    // (what a wave stores behind the input gradient that is counted next: another one, and in between a count)
                    complete_but(integral_constant<int, 2>{});
                    await_chunk(c + 1);
                    load_chunk(c + 1, n, p_last);
                    static_for<0, CH>([&](auto iic) {
                        constexpr int ii = decltype(iic)::value;
                        const int i = c * CH + ii;
                        // (the chain reads a position's operands in the interval before it)
                        if constexpr (ii == CH - 2) {
                            flush_chunk(c + 1, n, p_last);
                            complete_but(integral_constant<int, 1>{});
                        }
                        if constexpr (ii == CH - 1) complete_but(integral_constant<int, 2>{});
                        lds_barrier();
                        count(i - 1);
                        step_c(i & 1, c & (ROWS - 1), ii);
                        input_gradient(p_last - i * a.d, i & 1);
                    });
                }
                for (int i = c * CH; i < n; ++i) {
                    complete_but(integral_constant<int, 1>{});
                    lds_barrier();
                    count(i - 1);
                    step_c(i & 1, c & (ROWS - 1), i - c * CH);
                    input_gradient(p_last - i * a.d, i & 1);
                }
                if constexpr (kCounts) {
                    stores_complete_but<0>();
                    lds_barrier();
                    count(n);
                }
            }
            store_dw();
            return;
        }
        __builtin_amdgcn_s_setprio(3);      // (ahead of the other wave of the SIMD)
    }

    float wreg[NG][4 * HT];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int k = 0; k < 4 * HT; ++k) wreg[g][k] = a.wpack[(((size_t)w * NG + g) * (4 * HT) + k) * 64 + lane];
    const float g2_scale = a.n_gsrc >= 2 ? 1.0f : 0.0f;
    int n_valid = 0;
    float pen = 0.0f;
    if constexpr (CP) {
        const int col = bt * kTileN + 4 * q + j;
        const int len = col < a.B ? min(max(a.lengths[col], 0), a.T) : 0;
        n_valid = len - a.I - a.H + 1;
        pen = MODE == kAlone || a.sc ? a.two_lambda_cs * a.sc->inv_n_cs : 0.0f;
    }

    for (int r0 = chain; r0 < a.d && r0 < Pt; r0 += chains) {
        const int n = (Pt - r0 + a.d - 1) / a.d;
        const int p_last = r0 + (n - 1) * a.d;
        if constexpr (!SPLIT) load_chunk(0, n, p_last);
        float dcreg = 0.0f, dhreg = 0.0f;
        __syncthreads();            // LDS free: initial clearing, or the last position of the previous chain
        if constexpr (!SPLIT) flush_chunk(0, n, p_last);
        lds_barrier();

        // per-thread operands of the first position; those of position i+1 are read before the barrier
        // that ends position i
        f32x4 gt = lds.lc[0][0][tid];      // activated input, forget, candidate, output gate
        f32x4 o = lds.lc[0][1][tid];       // c, c_{p-d}, gradient sources
        // One position: the i-th from the end of the chain, staged in slot ii of the chunk buffers of parity
        // cpar; the per-thread operands of the next position are in slot `next`.  `staged` runs after they
        // have been read and before the barrier (the staging of the next chunk goes there).
        auto position = [&](int i, int ii, int cpar, int next, auto staged) {
            const int par = i & 1;
            const int p = p_last - i * a.d;
            const bool has_prev = p >= a.d;
            // ---- A: gate gradients of (unit, series)
            const float dh = o[2] + g2_scale * o[3] + dhreg;
            const float tc = tanh_f(o[0]);
            const float dh_o = dh * gt[3];          // (shared products formed once)
            float dc = dcreg + dh_o * (1.0f - tc * tc);
            if constexpr (CP) dc += p < n_valid ? pen * o[0] : 0.0f;
            const float cp = has_prev ? o[1] : 0.0f;
            const float dc_i = dc * gt[0], dc_f = dc * gt[1];
            f32x4 da;
            da[0] = dc_i * gt[2] * (1.0f - gt[0]);
            da[1] = dc_f * cp * (1.0f - gt[1]);
            da[2] = dc_i * (1.0f - gt[2] * gt[2]);
            da[3] = dh_o * tc * (1.0f - gt[3]);
            dcreg = dc_f;
            if (valid) dbacc += da;
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
                *reinterpret_cast<f32x4 *>(&lds.part[par][w][(64 * g + lane) * 4]) =
                    kBwdAcc == 2 ? acc[g][0] + acc[g][1] : acc[g][0];
            // per-thread operands of the next position (staged at least one barrier ago)
            gt = lds.lc[next][0][tid];
            o = lds.lc[next][1][tid];
            staged();
            lds_barrier();
            // ---- sums of the four partials: recurrent dh of this lane; input gradient
            {
                const int e = 4 * (KX + unit) + j;
                dhreg = (lds.part[par][0][e] + lds.part[par][1][e]) + (lds.part[par][2][e] + lds.part[par][3][e]);
            }
            if constexpr (!SPLIT) {         // (the other waves' work where there are some)
                input_gradient(p, par);
                step_c(par, cpar, ii);
            }
        };
        if constexpr (SPLIT) {
            // (slots by position modulo two chunks)
            int i = 0;
            for (; i + 1 < n; i += 2) {
                position(i, 0, 0, (i + 1) & (SLOTS - 1), [] {});
                position(i + 1, 0, 0, (i + 2) & (SLOTS - 1), [] {});
            }
            if (i < n) position(i, 0, 0, 0, [] {});
            if constexpr (kCounts) lds_barrier();       // (the last input gradients are in memory)
            continue;
        }
        // Whole chunks: one straight run of instructions each.  The operands of the next chunk are requested
        // at its start and staged one position before its end (after this thread has read its operands of the
        // chunk's last position): request and use in the same run, so the wait for a request counts the
        // memory operations issued since instead of waiting for all of them.
        int c = 0;
        for (; (c + 1) * CH <= n; ++c) {
            load_chunk(c + 1, n, p_last);   // (requests past the chain repeat its last position)
            static_for<0, CH>([&](auto iic) {
                constexpr int ii = decltype(iic)::value;
                position(c * CH + ii, ii, c & 1, (ii + 1) % CH, [&] {
                    if constexpr (ii == CH - 2) flush_chunk(c + 1, n, p_last);
                });
            });
        }
        // the last, partial chunk (staged by the run before it, or by the start of the chain)
        for (int i = c * CH; i < n; ++i) position(i, i - c * CH, c & 1, min(i + 1, n - 1) - c * CH, [] {});
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
__global__ void __launch_bounds__(SPLIT ? 2 * kNT : kNT, (!SPLIT && HT <= 10) ? 2 : 1) lstm_backward_narrow_kernel(NarrowBwdArgs a)
{
    using Lds = NarrowBwdLds<HT, KXT, SPLIT, kAlone>;
    __shared__ __align__(16) float da_all[2][Lds::HP * 16];
    __shared__ __align__(16) float part[2][kNW][Lds::NG * 64 * 4];
    __shared__ __align__(16) f32x4 lc[narrow_bwd_slots(SPLIT, kAlone)][2][kNT];
    __shared__ float xhc[2][Lds::CH][Lds::CT * 64];
    // The four workgroups of a 16-series tile share every 64-byte row of the tile.  Consecutive workgroup
    // ids go round the 8 XCDs, each with its own L2: ids x, x+8, x+16, x+24 of a group of 32 are the four
    // quarters of ONE tile, so they land on the same XCD at about the same time and a row is fetched from
    // HBM once, not four times (measured before: 2.3-2.8 times the algorithmic bytes).
    const int bt = (blockIdx.x >> 5) * 8 + (blockIdx.x & 7), q = (blockIdx.x >> 3) & 3;
    if (bt >= a.NB) return;     // the grid is padded to whole groups of 32 (before any barrier)
    lstm_backward_narrow_body<HT, KXT, CP, SPLIT, kAlone>(a, Lds{da_all, part, lc, xhc}, bt, q, blockIdx.y, gridDim.y, Progress{});
}

template <int HT, int KXT, bool SPLIT>
hipError_t run_nbwd(const NarrowBwdArgs &a, int chains, hipStream_t st)
{
    const dim3 grid(narrow_grid_x(a.NB), chains);
    if (a.sc) lstm_backward_narrow_kernel<HT, KXT, true, SPLIT><<<grid, SPLIT ? 2 * kNT : kNT, 0, st>>>(a);
    else lstm_backward_narrow_kernel<HT, KXT, false, SPLIT><<<grid, SPLIT ? 2 * kNT : kNT, 0, st>>>(a);
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
    a.hid_minus_xsrc = (ptrdiff_t)lp.hid - (ptrdiff_t)lp.xsrc;
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
