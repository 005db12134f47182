// Reverse pass of a dilated LSTM layer (Section 3.2, Table 1), one launch per layer, 16 series per workgroup: the
// launcher, and the kernel for hidden sizes above 52 (lstm_backward.h has the one for the others; the forward pass
// and the parallel structure: lstm_forward.h).
//
// Arithmetic.  fp32 MFMA (16x16x4) with the transposed weights as the A operand, held in registers for the whole
// launch, and the gate gradients of 16 series as the B operand.
#include "device_utils.h"
#include "esrnn_internal.h"
#include "three_term.h"

namespace esrnn {

namespace {

// ---------------------------------------------------------------------------
// Per position p of a chain (descending):
//   A. every lane turns (dh, dc) of its hidden unit into the four gate
//      pre-activation gradients da (registers), and leaves them in LDS next to
//      [x_p ; h_{p-d}] for step C;
//   B. transposed contraction d[x_p ; h_{p-d}] = W^T da on the MFMA, split over
//      the waves along the contraction: a wave multiplies the k-steps of the
//      units it owns, whose da it has just computed, so no operand crosses
//      waves; the four partial results meet in LDS and every wave sums the
//      output tiles it needs next (the recurrent dh of its own units) in a
//      fixed order.  The row order of the output tiles (row 4g+r of tile mb is
//      row g of input unit tile 4mb+r) keeps the result one unit tile per 64
//      lanes;
//   C. weight gradient dW += da (x) [x_p ; h_{p-d}]: contraction over the 16
//      series on the MFMA, both operands read transposed from LDS; whole rows
//      of tiles per wave, in accumulators for the whole launch.
// Steps A and B are the recurrence: position p - d cannot start before the
// recurrent dh of p is summed.  Step C only consumes what A leaves in LDS.
// Four "chain" waves do A and B, and four "dW" waves do C one position behind
// them: after the barrier that completes position p they read da and [x ; h] of
// p from one LDS copy while the chain waves fill the other copy with p - d.
// One workgroup of eight waves per compute unit; one barrier per position,
// taken by all eight waves.
//
// fp32 MFMAs and vector instructions of a SIMD do not run at the same time on
// this chip (esrnn_probe_issue_overlap measures it): what the elementwise work
// and the address arithmetic cost is taken from the matrix pipe, so both are
// kept short.
// ---------------------------------------------------------------------------
struct LstmBwdArgs {
    const float *wpack;   // [MB][4*HT][64]
    const float *xsrc;    // TL(4*KXT)
    const float *gates, *c, *hid;
    const float *gsrc[2]; // TL(HP): the gradient arriving at the hidden output is the sum of these
    int n_gsrc;           // 1 or 2; gsrc[1] repeats gsrc[0] when there is one
    float *gdst;          // TL(4*KXT)
    float *dw_partial;    // [NB*chains][HT*MB][4][64]
    float *db_partial;    // [NB*chains][HT][4][4]
    int NB, d;
    const int32_t *pmax;  // [NB] positions the longest series of a tile has: the tile's chains stop there
    // cell-state penalty (Section 8.4) of a block's first layer, kernels instantiated with CP only
    const int32_t *lengths;
    const Scalars *sc;
    float two_lambda_cs;
    int B, T, I, H;
};

template <int HT, int KXT, bool CP>
__global__ void __launch_bounds__(128 * kLstmWaves, 1) lstm_backward_split_kernel(LstmBwdArgs a)
{
    constexpr int W = kLstmWaves;
    constexpr int KT = KXT + HT;
    constexpr int MB = KT / 4;                       // 16-row tiles of [x ; h]
    static_assert(HT % W == 0 && KXT % W == 0 && KT % 4 == 0, "every wave owns as many tiles as the others, none is padding");
    constexpr int MTW = HT / W;                      // unit tiles per wave
    constexpr int QXW = KXT / W;                     // input unit tiles finalised per wave
    constexpr int NT = 64 * W;                       // threads of the chain waves
    constexpr int DA_ROWS = 16 * HT;
    constexpr int XH_PER_THREAD = KT / W;
    constexpr int XH_ROWS = 16 * MB;

    __shared__ float da_lds[2][DA_ROWS * kLdsPad];   // [mt][4*gate + unit][series]
    __shared__ float xh_lds[2][XH_ROWS * kLdsPad];   // [row of x ; h][series]
    __shared__ float part_lds[2][W][MB * 4][64];     // partial d[x ; h] of every chain wave
    static_assert(2 * (DA_ROWS * kLdsPad + XH_ROWS * kLdsPad + W * MB * 4 * 64) * 4 <= 128 * 1024,
                  "LDS budget of the reverse kernel");

    const int lane = threadIdx.x & 63, bt = blockIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index, known to be uniform
    const bool chain = wv < W;
    const int s = wv & (W - 1);
    const int Pt = a.pmax[bt];      // the chains of this tile stop at its longest series
    const int g = lane >> 4, n = lane & 15;
    for (int i = threadIdx.x; i < 2 * XH_ROWS * kLdsPad; i += 2 * NT) (&xh_lds[0][0])[i] = 0.0f;
    for (int i = threadIdx.x; i < 2 * DA_ROWS * kLdsPad; i += 2 * NT) (&da_lds[0][0])[i] = 0.0f;
    const size_t part = (size_t)bt * gridDim.y + blockIdx.y;

    if (!chain) {
        // ---- dW waves: rows (W-1-s) + W*j of the weight gradient, in accumulators for the whole launch
        f32x4 dw[MTW][MB];
#pragma unroll
        for (int j = 0; j < MTW; ++j)
#pragma unroll
            for (int nbk = 0; nbk < MB; ++nbk) dw[j][nbk] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto accumulate = [&](int buf) {
            lds_barrier();          // da and [x ; h] of the position are complete in copy `buf`
            float xb[MB][4], ar[MTW][4];
#pragma unroll
            for (int nbk = 0; nbk < MB; ++nbk)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) xb[nbk][ks] = xh_lds[buf][(nbk * 16 + n) * kLdsPad + 4 * ks + g];
#pragma unroll
            for (int j = 0; j < MTW; ++j)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    ar[j][ks] = da_lds[buf][(((W - 1 - s) + W * j) * 16 + n) * kLdsPad + 4 * ks + g];
#pragma unroll
            for (int j = 0; j < MTW; ++j)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int nbk = 0; nbk < MB; ++nbk) dw[j][nbk] = mfma16(ar[j][ks], xb[nbk][ks], dw[j][nbk]);
        };
        for (int r0 = blockIdx.y; r0 < a.d && r0 < Pt; r0 += gridDim.y) {
            const int p_last = r0 + ((Pt - 1 - r0) / a.d) * a.d;
            __syncthreads();
            int buf = 0;
            for (int p = p_last; p >= a.d; p -= a.d) {
                accumulate(buf);
                buf ^= 1;
            }
            accumulate(buf);
        }
#pragma unroll
        for (int j = 0; j < MTW; ++j) {
            const int row = (W - 1 - s) + W * j;
#pragma unroll
            for (int nbk = 0; nbk < MB; ++nbk) {
                float *dst = a.dw_partial + (part * (HT * MB) + row * MB + nbk) * 256 + lane;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) dst[rr * 64] = dw[j][nbk][rr];
            }
        }
        return;
    }

    // ---- chain waves: steps A and B
    // W^T operands of the k-steps this wave owns: k-step 4*mt + gate, mt = s + 4j
    float wreg[MB][4 * MTW];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < MTW; ++j) {
            const int mt = s + W * j;
#pragma unroll
            for (int r = 0; r < 4; ++r) wreg[mb][4 * j + r] = a.wpack[((size_t)mb * 4 * HT + 4 * mt + r) * 64 + lane];
        }
    f32x4 dbacc[MTW];
#pragma unroll
    for (int j = 0; j < MTW; ++j) dbacc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const size_t xtile = (size_t)KXT * 64, htile = (size_t)HT * 64;

    // operands of one position, requested one position ahead.  Branch-free: a missing predecessor aliases p itself.
    float4 pf_gt[MTW];
    float pf_c[MTW], pf_cp[MTW], pf_g[MTW], pf_g2[MTW], pf_xh[XH_PER_THREAD];
    // The requests of a position go out piece by piece, each as soon as the registers it fills are free:
    // [x ; h] after it has gone to LDS, the operands of unit tile j after the elementwise step of tile j.
    auto fetch_xh = [&](int p) {
        const size_t pb = (size_t)p * a.NB + bt;
        const size_t pbd = (size_t)(p >= a.d ? p - a.d : p) * a.NB + bt;
#pragma unroll
        for (int i = 0; i < XH_PER_THREAD; ++i) {
            const int q = s + W * i;                       // unit tile of [x ; h]
            const float *src = q < KXT ? a.xsrc + pb * xtile + q * 64 : a.hid + pbd * htile + (q - KXT) * 64;
            pf_xh[i] = src[lane];
        }
    };
    auto fetch_tile = [&](int j, int p, bool first) {
        const size_t pb = (size_t)p * a.NB + bt;
        const size_t pbd = (size_t)(p >= a.d ? p - a.d : p) * a.NB + bt;
        // wave-uniform tile bases plus the lane index: scalar address arithmetic
        const int mt = s + W * j;
        const size_t tile = (pb * HT + mt) * 64;
        pf_gt[j] = (reinterpret_cast<const float4 *>(a.gates) + tile)[lane];
        pf_c[j] = first ? (a.c + tile)[lane] : pf_cp[j];
        pf_cp[j] = (a.c + (pbd * HT + mt) * 64)[lane];
        pf_g[j] = (a.gsrc[0] + tile)[lane];
        pf_g2[j] = (a.gsrc[1] + tile)[lane];    // gsrc[1] repeats gsrc[0] when there is one source (ignored then)
    };
    auto fetch = [&](int p, bool first) {
        fetch_xh(p);
#pragma unroll
        for (int j = 0; j < MTW; ++j) fetch_tile(j, p, first);
    };
    const float g2_scale = a.n_gsrc >= 2 ? 1.0f : 0.0f;
    int n_valid = 0;
    float pen = 0.0f;
    if constexpr (CP) {
        const int col = bt * kTileN + n;
        const int len = col < a.B ? min(max(a.lengths[col], 0), a.T) : 0;
        n_valid = len - a.I - a.H + 1;
        pen = a.two_lambda_cs * a.sc->inv_n_cs;
    }
    float dcreg[MTW], dhreg[MTW];
    float da[MTW][4];
    auto step_a_tile = [&](int j, bool has_prev, int p_cur, int buf) {
        const float4 gt = pf_gt[j];
        const float dh = pf_g[j] + g2_scale * pf_g2[j] + dhreg[j];
        const float tc = tanh_f(pf_c[j]);
        // (products shared between the terms are formed once: the vector ALU's cycles are the matrix pipe's)
        const float dh_o = dh * gt.w;
        float dc = dcreg[j] + dh_o * (1.0f - tc * tc);
        if constexpr (CP) dc += p_cur < n_valid ? pen * pf_c[j] : 0.0f;
        const float cp = has_prev ? pf_cp[j] : 0.0f;
        const float dc_i = dc * gt.x, dc_f = dc * gt.y;
        da[j][0] = dc_i * gt.z * (1.0f - gt.x);
        da[j][1] = dc_f * cp * (1.0f - gt.y);
        da[j][2] = dc_i * (1.0f - gt.z * gt.z);
        da[j][3] = dh_o * tc * (1.0f - gt.w);
        dcreg[j] = dc_f;
        float *dst = da_lds[buf] + ((s + W * j) * 16 + g) * kLdsPad + n;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            dst[r * 4 * kLdsPad] = da[j][r];
            dbacc[j][r] += da[j][r];
        }
    };
    auto store_xh = [&](bool has_prev, int buf) {
#pragma unroll
        for (int i = 0; i < XH_PER_THREAD; ++i) {
            const int e = threadIdx.x + i * NT;
            xh_lds[buf][(e >> 4) * kLdsPad + (e & 15)] = (e < KXT * 64 || has_prev) ? pf_xh[i] : 0.0f;
        }
    };
    auto step_b = [&](int buf) {
        f32x4 acc[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < MTW; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[mb] = mfma16(wreg[mb][4 * j + r], da[j][r], acc[mb]);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int r = 0; r < 4; ++r) part_lds[buf][s][mb * 4 + r][lane] = acc[mb][r];
    };
    float dxv[QXW];
    auto finish = [&](int buf) {
        lds_barrier();              // partials, da, [x ; h] of the position complete
        const float (*pt)[MB * 4][64] = part_lds[buf];
#pragma unroll
        for (int j = 0; j < MTW; ++j) {
            const int q = KXT + s + W * j;   // row of part_lds = unit tile of [x ; h]
            dhreg[j] = (pt[0][q][lane] + pt[1][q][lane]) + (pt[2][q][lane] + pt[3][q][lane]);
        }
#pragma unroll
        for (int j = 0; j < QXW; ++j) {
            const int q = s + W * j;
            dxv[j] = (pt[0][q][lane] + pt[1][q][lane]) + (pt[2][q][lane] + pt[3][q][lane]);
        }
    };
    auto store_dx = [&](int p) {
        const size_t pb = (size_t)p * a.NB + bt;
#pragma unroll
        for (int j = 0; j < QXW; ++j) (a.gdst + pb * xtile + (s + W * j) * 64)[lane] = dxv[j];
    };

    for (int r0 = blockIdx.y; r0 < a.d && r0 < Pt; r0 += gridDim.y) {
        const int p_last = r0 + ((Pt - 1 - r0) / a.d) * a.d;
#pragma unroll
        for (int j = 0; j < MTW; ++j) { dcreg[j] = 0.0f; dhreg[j] = 0.0f; }
        __syncthreads();            // LDS free (previous chain / initial clearing)
        int buf = 0;
        fetch(p_last, true);
        store_xh(p_last >= a.d, buf);
#pragma unroll
        for (int j = 0; j < MTW; ++j) step_a_tile(j, p_last >= a.d, p_last, buf);
        fetch(max(p_last - a.d, r0), false);
        step_b(buf);
        for (int p = p_last; p >= a.d; p -= a.d) {
            finish(buf);
            buf ^= 1;               // position p - d goes to the other copy
            store_dx(p);
            const bool has_prev = p >= 2 * a.d;
            const int p_next = max(p - 2 * a.d, r0);
            store_xh(has_prev, buf);
            fetch_xh(p_next);
#pragma unroll
            for (int j = 0; j < MTW; ++j) {
                step_a_tile(j, has_prev, p - a.d, buf);
                fetch_tile(j, p_next, false);
            }
            step_b(buf);
        }
        finish(buf);
        store_dx(r0);
    }
#pragma unroll
    for (int j = 0; j < MTW; ++j) {
        const int mt = s + W * j;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const float tot = group16_sum(dbacc[j][rr]);
            if (n == 0) a.db_partial[(part * HT + mt) * 16 + g * 4 + rr] = tot;
        }
    }
}

// out = a + b (+ c): gradient sources of a layer behind three or more residual blocks
__global__ void __launch_bounds__(256) sum_sources_kernel(const float4 *__restrict__ a, const float4 *__restrict__ b,
                                                           const float4 *__restrict__ c, float4 *__restrict__ out, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float4 v = a[i];
    const float4 w = b[i];
    v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
    if (c) {
        const float4 u = c[i];
        v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
    }
    out[i] = v;
}

template <int HT, int KXT>
hipError_t run_bwd(const LstmBwdArgs &a, int chains, hipStream_t st)
{
    if (a.sc) lstm_backward_split_kernel<HT, KXT, true><<<dim3(a.NB, chains), 128 * kLstmWaves, 0, st>>>(a);
    else lstm_backward_split_kernel<HT, KXT, false><<<dim3(a.NB, chains), 128 * kLstmWaves, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_lstm_backward(const Plan &pl, int layer, const int32_t *lengths, float *ws, hipStream_t st)
{
    const LayerPlan &lp = pl.layer[layer];
    LstmBwdSources src{{ws + lp.gsrc[0], ws + lp.gsrc[lp.n_gsrc >= 2 ? 1 : 0]}, std::min(lp.n_gsrc, 2)};
    if (lp.n_gsrc > 2) {
        // three or more residual blocks: the sources past the first are summed into a buffer of their
        // own first (they stay intact for the layers that consume them separately)
        const size_t n4 = (size_t)pl.P * pl.NB * pl.HT * 16;   // float4 elements of a TL(HP) array
        const float *s3 = lp.n_gsrc > 3 ? ws + lp.gsrc[3] : nullptr;
        sum_sources_kernel<<<(unsigned)((n4 + 255) / 256), 256, 0, st>>>(
            reinterpret_cast<const float4 *>(ws + lp.gsrc[1]), reinterpret_cast<const float4 *>(ws + lp.gsrc[2]),
            reinterpret_cast<const float4 *>(s3), reinterpret_cast<float4 *>(ws + pl.gsum), n4);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        src.g[1] = ws + pl.gsum;
    }
    if (lp.narrow_bwd) return launch_lstm_backward_narrow(pl, layer, lengths, ws, st);
    if (bwd_three_term(pl.HT)) return launch_lstm_backward_three_term(pl, layer, src, lengths, ws, st);
    LstmBwdArgs a{};
    const bool cp = lp.first_in_block && pl.cfg.lambda_cs != 0.0f;
    a.lengths = lengths;
    a.sc = cp ? reinterpret_cast<const Scalars *>(ws + pl.scalars) : nullptr;
    a.two_lambda_cs = 2.0f * pl.cfg.lambda_cs;
    a.B = pl.B; a.T = pl.T; a.I = pl.I; a.H = pl.H;
    a.wpack = ws + lp.wpack_bwd; a.xsrc = ws + lp.xsrc; a.gates = ws + lp.gates; a.c = ws + lp.c; a.hid = ws + lp.hid;
    a.n_gsrc = src.n;
    a.gsrc[0] = src.g[0];
    a.gsrc[1] = src.g[1];
    a.gdst = ws + lp.gdst; a.dw_partial = ws + lp.dw_partial; a.db_partial = ws + lp.db_partial;
    a.NB = pl.NB; a.d = lp.dil;
    a.pmax = reinterpret_cast<const int32_t *>(ws + pl.pmax);
#define X(HT_, KXT_) if constexpr (!bwd_three_term(HT_)) if (pl.HT == HT_ && lp.KXT == KXT_) return run_bwd<HT_, KXT_>(a, lp.chains_bwd, st);
    ESRNN_LSTM_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace esrnn
