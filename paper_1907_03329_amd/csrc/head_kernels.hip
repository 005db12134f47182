// Output stage of the network (Section 3.4: tanh layer, then linear layer), the
// pinball loss over unmasked outputs (Section 3.5) and the reverse pass of both
// in ONE kernel (the forecasts of Eq. (5) follow in a small kernel of their own,
// for callers that want them): the gradient of the loss
// with respect to an output depends only on that output, its target and the
// number of unmasked outputs (known from the lengths), so the reverse pass of
// this stage can run while the activations are still in registers.  Every
// (window position, 16-series) tile is independent: one wave processes one tile at a time.
//
// Row order.  "Unit-tile order" of a 16-row output tile m: row 4g+r is logical
// row 4(4m+r)+g, so that component r of lane (g, n) belongs to unit tile 4m+r
// in the one-float-per-lane layout and can be fed back, as it stands, into the
// next product.  Both forward products use it: the tanh layer's
// output feeds the linear layer, and the linear layer's output (hence the loss
// gradient) feeds the transposed products.
//
// All products run on the bf16 matrix pipe with fp32 accuracy (three_term.h).  A wave holds all units of its sixteen
// series, so the changing operands of the four contractions are split where they are computed and never leave its
// registers; only the weight gradients, which contract over the series, need both operands turned: their parts go through
// the wave's own corner of LDS and are read with the transpose load (the LDS home of lstm_backward.h).  Biases come last
// and products start from zero accumulators, largest terms first, for the reason given in lstm_forward.h.
//
// The forward operands stay in registers; the transposed ones, and those of the linear layer where they do not fit beside
// two waves per SIMD, are read from LDS, one copy per workgroup.  Waves of a workgroup add up their weight gradients at
// the end, so that a quarter (an eighth) as many partial blocks are written and reduced as with one per wave.
#include "device_utils.h"
#include "esrnn_internal.h"
#include "three_term.h"

namespace esrnn {

namespace {

struct HeadArgs {
    const u32x4 *WaF, *WoF, *WoT, *WaT;   // A operands [tile][quad][64], forward and transposed
    const float *baF, *boF;               // biases
    const float *R;         // TL(HP) top block output
    const float *Z;         // TL(OP) targets
    const int32_t *lengths;
    const int32_t *pmax;    // [NB] window positions the longest series of a tile has
    const Scalars *sc;
    float *O;               // TL(OP) outputs
    float *loss_partial;    // [gridDim.x]
    float *gO;              // TL(OP): dL/d(output); the target's gradient is its negative
    float *gTop;            // TL(HP): dL/d(top block output)
    float *partial;         // [gridDim.x][stride] weight-gradient partials of every workgroup
    int P, NB, B, T, I, H, stride;
    int orows;              // rows of the Z, O and gO tiles: 4 * ceil(H / 4)
    float tau;
    // forecasts at the end of the series (head_last_kernel)
    float *forecasts;       // [B][H]
    const float *u, *S1, *S2;
    int Bt, m1, m2;         // row stride of those; periods (0: no such seasonality)
};

// Parts of a lane's values of N unit tiles, in pairs of tiles: per pair hi, mid, lo; past N zero.  (Vectors: arrays of
// single words are read back as vectors before they are taken apart into registers, and stay in memory.)
template <int NP, int N>
__device__ __forceinline__ void split_all(const float (&v)[N], u32x4 (&p)[NP])
{
    static_for<0, NP>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (2 * i < N) {
            float second = 0.0f;
            if constexpr (2 * i + 1 < N) second = v[2 * i + 1];
            const Parts q = split_pair<true>(v[2 * i], second);
            p[i] = u32x4{q.hi, q.mid, q.lo, 0u};
        } else {
            p[i] = u32x4{0u, 0u, 0u, 0u};
        }
    });
}
// B operand of a contraction over the first NP pairs (three_term.h)
template <int NP, int N>
__device__ __forceinline__ void b_quads(const u32x4 (&p)[N], u32x4 (&b)[tt_b_quads(NP)])
{
    constexpr int full = tt_full(NP), rest = tt_rest(NP), base = 4 * full;
    static_for<0, 12 * full>([&](auto kc) {
        constexpr int k = decltype(kc)::value, i = 4 * (k / 12) + k % 4;
        if constexpr (i < NP) b[k / 4][k % 4] = p[i][k / 4 % 3];
        else b[k / 4][k % 4] = 0u;
    });
    if constexpr (rest == 1) b[3 * full] = u32x4{p[base][0], p[base][1], p[base][2], p[base][0]};
    if constexpr (rest == 2) {
        b[3 * full] = u32x4{p[base][0], p[base + 1][0], p[base][1], p[base + 1][1]};
        b[3 * full + 1] = u32x4{p[base][2], p[base + 1][2], p[base][0], p[base + 1][0]};
    }
}
// acc[m] = sum over the contraction; w(m, q): quad q of output tile m.
// LDS: the quads of one q at a time, the next ones requested ahead of the products (left to itself the compiler puts every
// read from LDS right before its use); the first ones by request(), as early as can be.
// Two sums: one of the instructions that hold leading terms, one of all others, so that the small terms do not round the
// large ones.  (The loss gradient has two values, so the few products of a contraction over the horizon repeat themselves
// and so do their rounding errors: with one sum the gradients of the tanh layer were off by 1.2 to 1.8 times as much as
// with fp32 products.)
template <int NP, int M, bool LDS>
struct Contraction {
    static constexpr int Q = tt_a_quads(NP);
    static constexpr bool leading(int i) { return i % 6 == 0; }     // (of a rest, the first one too)
    u32x4 quad[LDS ? 2 : 1][LDS ? M : 1];
    template <class W>
    __device__ __forceinline__ void request(W &&w, int q = 0)
    {
        if constexpr (LDS) {
#pragma unroll
            for (int m = 0; m < M; ++m) quad[q & 1][m] = w(m, q);
        }
    }
    template <class W>
    __device__ __forceinline__ void sum(W &&w, const u32x4 (&b)[tt_b_quads(NP)], f32x4 (&acc)[M])
    {
        f32x4 small[M];
#pragma unroll
        for (int m = 0; m < M; ++m) acc[m] = small[m] = f32x4{0.f, 0.f, 0.f, 0.f};
        static_for<0, Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            if constexpr (LDS) {
                if constexpr (q + 1 < Q) request(w, q + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            static_for<0, tt_mfmas(NP)>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                constexpr TtPair t = tt_mfma(NP, i);
                if constexpr (t.a == q) {
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        f32x4 &to = leading(i) ? acc[m] : small[m];
                        if constexpr (LDS) to = mfma_bf16(quad[q & 1][m], b[t.b], to);
                        else to = mfma_bf16(w(m, q), b[t.b], to);
                    }
                }
            });
        });
#pragma unroll
        for (int m = 0; m < M; ++m) acc[m] += small[m];
    }
};

// What a sum of the linear layer is multiplied by: infinite where a weight of its row is (whose operand is a finite number).
__device__ __forceinline__ float row_scale(unsigned long long infinite_rows, int row)
{
    return (infinite_rows >> row) & 1 ? __builtin_inff() : 1.0f;
}

template <int HT, int MO>
struct HeadShape {
    static constexpr int MA = (HT + 3) / 4;             // 16-row tiles of the hidden units
    static constexpr int OTMAX = 4 * MO;                // unit tiles that cover the outputs
    static constexpr int NPH = (HT + 1) / 2, NPO = 2 * MO;
    static constexpr int QH = tt_a_quads(NPH), QO = tt_a_quads(NPO);
    static constexpr int W = head_waves(HT, MO);
    // a wave's corner: the parts of the inputs, of the tanh layer's outputs and later of their gradient, of the loss gradient
    static constexpr int kTile = 3 * kPartBytes;
    static constexpr int kCorner = (2 * MA + MO) * kTile;
    // operands of the linear layer in LDS, where they do not fit the registers beside the rest but do fit there
    static constexpr int kLimit = 127 * 1024;
    static constexpr bool kWoLds = (W == 8 ? HT >= 10 : MO >= 3 || HT >= 13) && (MA * (QO + QH) + MO * QH) * 1024 + W * kCorner <= kLimit;
    static constexpr int kWeightQuads = MA * (QO + QH) + (kWoLds ? MO * QH : 0);
    static constexpr int kPartials = (MO * MA + MA * MA) * 4 + OTMAX + 4 * MA;      // per lane
    static constexpr int kAtOnce = std::min(kPartials, kLimit / (W * 256));         // of them added up together, at the end
    static constexpr int kBytes = std::max(kWeightQuads * 1024 + W * kCorner, W * kAtOnce * 256);
    static_assert(kBytes <= kLimit, "LDS budget of the output-stage kernel");
};

// What bounds it: issue and dependency stalls of the one or two waves a SIMD has room for.  Hidden 40, horizon 8, 4096 series,
// 61 positions: 44 - 47 us (fp32 products 64 - 67 us; 108 MB, 21 us at the rate of a large copy); matrix pipe 21 % busy,
// instructions issued 34 % of the time.  Hidden 50, horizon 18, 211 positions: 254 - 256 us (369 us); matrix pipe 33 %,
// issue 53 %.  Hidden 30: 32 us (42 us); hidden 40, horizon 48, 512 series: 98 us (131 - 135 us).  Hidden 50, 40 positions: horizon
// 40 74 us (100), 64 216 us (245), where registers spill.
// REVERSE: a reverse pass follows; without it outputs and loss are all.
template <int HT, int MO, bool REVERSE>
__global__ void __launch_bounds__(64 * head_waves(HT, MO)) head_kernel(HeadArgs a)
{
    using S = HeadShape<HT, MO>;
    constexpr int MA = S::MA, OTMAX = S::OTMAX, NPH = S::NPH, NPO = S::NPO, QH = S::QH, QO = S::QO, W = S::W;
    __shared__ __align__(16) char lds[S::kBytes];
    __shared__ float s_part[W];
    __shared__ __align__(16) float s_ba[16 * MA];               // [tile][lane group][component]
    __shared__ __align__(16) float s_out[16 * MO][2];           // likewise: scale of a sum, bias

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index, known to be uniform
    const int g = lane >> 4, n = lane & 15;
    u32x4 *s_WoT = reinterpret_cast<u32x4 *>(lds), *s_WaT = s_WoT + MA * QO * 64, *s_Wo = s_WaT + MA * QH * 64;
    char *corner = lds + S::kWeightQuads * 1024 + wv * S::kCorner;

    // Operands of one tile.  Those of the next one are requested into the same registers as soon as they are free.
    float br[HT], z[OTMAX];            // rows 4*q + g, 4*ks + g
    int raw_len;                       // length of this lane's series
    // Tiles are numbered p * NB + (series tile); a wave takes every stride-th one and keeps (p, series
    // tile) by increments.  All of it is wave-uniform, so tile bases live on the scalar unit and the
    // lanes only add their own index.
    const int n_tiles = a.P * a.NB;
    const int stride = gridDim.x * W;
    const int step_p = stride / a.NB, step_bt = stride % a.NB;
    auto load_inputs = [&](int t, int bt) {     // (past the end: the last tile again)
        if (t >= n_tiles) { t = n_tiles - 1; bt = a.NB - 1; }
        const int b = bt * 16 + n;
        const float *rt = a.R + (size_t)t * HT * 64;
#pragma unroll
        for (int q = 0; q < HT; ++q) br[q] = (rt + q * 64)[lane];
        raw_len = a.lengths[b < a.B ? b : a.B - 1];
    };
    auto load_targets = [&](int t) {
        const float *zt = a.Z + (size_t)min(t, n_tiles - 1) * a.orows * 16;
#pragma unroll
        for (int ks = 0; ks < OTMAX; ++ks) {
            const int j = 4 * ks + g;
            z[ks] = zt[(j < a.orows ? j : a.orows - 1) * 16 + n];
        }
    };
    // Ragged batches: a tile past the longest series of its 16 holds no window.  Nothing was computed for it upstream and
    // nothing downstream reads it.  The next tile is looked for before its operands are requested, so that the loop below has
    // one way through it, and the waits in it count exactly what has been issued since.
    auto advance = [&](int &t, int &p, int &bt) {
        do {
            t += stride; p += step_p; bt += step_bt;
            if (bt >= a.NB) { bt -= a.NB; ++p; }
        } while (t < n_tiles && p >= a.pmax[bt]);
    };
    int tile = blockIdx.x * W + wv;
    int p = tile / a.NB, bt = tile % a.NB;
    if (tile < n_tiles && p >= a.pmax[bt]) advance(tile, p, bt);
    load_inputs(tile, bt);
    load_targets(tile);
    {
        // (WaT follows WoT in the workspace too; all requests before the first of them is waited for)
        constexpr int kT = MA * (QO + QH) * 64, kAll = S::kWeightQuads * 64, kPer = (kAll + 64 * W - 1) / (64 * W);
        u32x4 v[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = min(k * 64 * W + (int)threadIdx.x, kAll - 1);
            v[k] = i < kT ? a.WoT[i] : a.WoF[i - kT];
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (k * 64 * W + (int)threadIdx.x < kAll) s_WoT[k * 64 * W + threadIdx.x] = v[k];
    }
    __builtin_amdgcn_sched_barrier(0);
    if ((int)threadIdx.x < 16 * MA) {
        s_ba[threadIdx.x] = a.baF[threadIdx.x];
    } else if (const int e = (int)threadIdx.x - 16 * MA; e < 16 * MO) {
        s_out[e][0] = row_scale(a.sc->infinite_rows, 4 * (4 * (e >> 4) + (e & 3)) + ((e >> 2) & 3));
        s_out[e][1] = a.boF[e];
    }
    u32x4 wa[MA][QH], wo[S::kWoLds ? 1 : MO][S::kWoLds ? 1 : QH];
#pragma unroll
    for (int m = 0; m < MA; ++m)
#pragma unroll
        for (int q = 0; q < QH; ++q) wa[m][q] = a.WaF[(m * QH + q) * 64 + lane];
    if constexpr (!S::kWoLds)
#pragma unroll
        for (int m = 0; m < MO; ++m)
#pragma unroll
            for (int q = 0; q < QH; ++q) wo[m][q] = a.WoF[(m * QH + q) * 64 + lane];
    __syncthreads();
    auto wa_op = [&](int m, int q) { return wa[m][q]; };
    auto wo_op = [&](int m, int q) { return S::kWoLds ? s_Wo[(m * QH + q) * 64 + lane] : wo[S::kWoLds ? 0 : m][S::kWoLds ? 0 : q]; };
    auto woT_op = [&](int m, int q) { return s_WoT[(m * QO + q) * 64 + lane]; };
    auto waT_op = [&](int m, int q) { return s_WaT[(m * QH + q) * 64 + lane]; };

    f32x4 dWo[MO][MA], dWa[MA][MA];
#pragma unroll
    for (int j = 0; j < MA; ++j) {
#pragma unroll
        for (int i = 0; i < MO; ++i) dWo[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < MA; ++i) dWa[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float dbo[OTMAX], dba[4 * MA];
#pragma unroll
    for (int i = 0; i < OTMAX; ++i) dbo[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < 4 * MA; ++i) dba[i] = 0.0f;

    // Turned operands of the weight gradients: parts of a tensor's tiles into the corner, the first one at tile `first`, and quads out of it (series along the
    // contraction; which parts meet in an instruction: lstm_backward.h).
    auto put = [&](int first, auto &parts, auto tiles) {
        static_for<0, decltype(tiles)::value>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            char *dst = corner + (first + m) * S::kTile + 8 * lane + 32 * (lane >> 5);
            static_for<0, 3>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                *reinterpret_cast<u32x2 *>(dst + q * kPartBytes) = u32x2{parts[2 * m][q], parts[2 * m + 1][q]};
            });
        });
    };
    constexpr std::integral_constant<int, MA> all_a;
    constexpr std::integral_constant<int, MO> all_o;
    const int tr = ((n & 3) * 16 + 8 * (g & 1) + (n >> 2)) * 8 + 32 * ((n & 3) >> 1);
    const int hl = tr + (g >= 2 ? 2 * kPartBytes : 0), hm = tr + (g >= 2 ? kPartBytes : 0), lh = tr + (g >= 2 ? 0 : 2 * kPartBytes);
    auto quad = [&](const char *at) {
        const u32x2 v0 = lds_read_transposed(at), v1 = lds_read_transposed(at + 32);
        return u32x4{v0[0], v0[1], v1[0], v1[1]};
    };
    // dw[i][j] += rows of tile row0 + i (x) rows of tile col0 + j
    auto outer = [&](auto rows, int row0, int col0, auto &dw) {
        u32x4 x[MA][2];
#pragma unroll
        for (int j = 0; j < MA; ++j) {
            const char *at = corner + (col0 + j) * S::kTile;
            x[j][0] = quad(at + hm);
            x[j][1] = quad(at + lh);
        }
        static_for<0, decltype(rows)::value>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const char *at = corner + (row0 + i) * S::kTile;
            const u32x4 hi = quad(at + tr), mid = quad(at + tr + kPartBytes), both = quad(at + hl);
#pragma unroll
            for (int j = 0; j < MA; ++j) dw[i][j] = mfma_bf16(both, x[j][1], dw[i][j]);
#pragma unroll
            for (int j = 0; j < MA; ++j) dw[i][j] = mfma_bf16(mid, x[j][0], dw[i][j]);
#pragma unroll
            for (int j = 0; j < MA; ++j) dw[i][j] = mfma_bf16(hi, x[j][0], dw[i][j]);
        });
    };

    const float inv_n = a.sc->inv_n_pin;
    float loss = 0.0f;
    for (; tile < n_tiles;) {
        const int this_tile = tile;
        int len = raw_len < 0 ? 0 : (raw_len > a.T ? a.T : raw_len);
        if (bt * 16 + n >= a.B) len = 0;
        const bool valid = p < len - a.I - a.H + 1;
        advance(tile, p, bt);

        // ---- forward: tanh layer, linear layer
        float av[4 * MA];
        f32x4 oc[MO];
        {
            Contraction<NPH, MA, false> tanh_layer;
            Contraction<NPH, MO, S::kWoLds && W == 4> linear_layer;
            u32x4 bq[tt_b_quads(NPH)], parts[2 * MA];
            split_all(br, parts);
            __builtin_amdgcn_sched_barrier(0);
            load_inputs(tile, bt);
            __builtin_amdgcn_sched_barrier(0);
            put(0, parts, all_a);
            b_quads<NPH>(parts, bq);
            f32x4 acc[MA];
            tanh_layer.sum(wa_op, bq, acc);
            linear_layer.request(wo_op);
#pragma unroll
            for (int m = 0; m < MA; ++m) {
                const f32x4 ba = *reinterpret_cast<const f32x4 *>(s_ba + (m * 4 + g) * 4);
#pragma unroll
                for (int r = 0; r < 4; ++r) av[4 * m + r] = (4 * m + r < HT) ? tanh_f(acc[m][r] + ba[r]) : 0.0f;
            }
            split_all(av, parts);
            put(MA, parts, all_a);
            b_quads<NPH>(parts, bq);
            linear_layer.sum(wo_op, bq, oc);
        }
        // ---- outputs, loss and the gradient of the pinball loss; unit tile ks holds rows 4ks..4ks+3
        float go[OTMAX];
        float *ot = a.O + (size_t)this_tile * a.orows * 16, *got = a.gO + (size_t)this_tile * a.orows * 16;
#pragma unroll
        for (int ks = 0; ks < OTMAX; ++ks) {
            go[ks] = 0.0f;
            if (4 * ks >= a.orows) continue;        // (uniform; the rows of a tile are whole unit tiles)
            const int j = 4 * ks + g;               // 0-based step of the horizon
            const float *of = s_out[((ks >> 2) * 4 + g) * 4 + (ks & 3)];
            const float o = fmaf(oc[ks >> 2][ks & 3], of[0], of[1]);
            const float d = z[ks] - o;
            const bool counted = valid && j < a.H;
            if (counted) loss += d >= 0.0f ? a.tau * d : (a.tau - 1.0f) * d;
            go[ks] = counted ? (d >= 0.0f ? -a.tau : 1.0f - a.tau) * inv_n : 0.0f;
            ot[j * 16 + n] = o;
            got[j * 16 + n] = go[ks];
            dbo[ks] += go[ks];
        }
        load_targets(tile);
        if constexpr (!REVERSE) continue;       // forward-only callers: nothing below is needed
        // ---- reverse: dA = Wo^T gO (unit-tile order), through the tanh; dR = Wa^T dpre
        f32x4 acc[MA];
        {
            Contraction<NPO, MA, W == 4> linear_layer;
            u32x4 bq[tt_b_quads(NPO)], parts[NPO];
            linear_layer.request(woT_op);
            split_all(go, parts);
            put(2 * MA, parts, all_o);
            b_quads<NPO>(parts, bq);
            linear_layer.sum(woT_op, bq, acc);
        }
        float dp[4 * MA];
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int q = 4 * m + r;
                dp[q] = acc[m][r] * (1.0f - av[q] * av[q]);
                dba[q] += dp[q];
            }
        outer(all_o, 2 * MA, MA, dWo);
        {
            Contraction<NPH, MA, W == 4> tanh_layer;
            tanh_layer.request(waT_op);
            u32x4 bq[tt_b_quads(NPH)], parts[2 * MA];
            split_all(dp, parts);
            // (LDS serves a wave's instructions in order: the place is free again)
            put(MA, parts, all_a);
            b_quads<NPH>(parts, bq);
            tanh_layer.sum(waT_op, bq, acc);
        }
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int q = 4 * m + r;
                if (q < HT) (a.gTop + (size_t)this_tile * HT * 64 + q * 64)[lane] = acc[m][r];
            }
        outer(all_a, MA, 0, dWa);
    }

    const float tot = wave_sum(loss);
    if (lane == 0) s_part[wv] = tot;
    if constexpr (REVERSE) {
        // The waves' sums meet in LDS, some at a time; every wave adds up and stores its share of them.
        float *slot = reinterpret_cast<float *>(lds), *dst = a.partial + (size_t)blockIdx.x * a.stride;
        constexpr int kTiles = (MO * MA + MA * MA) * 4;
        const int OT = (a.H + 3) / 4;
        static_for<0, (S::kPartials + S::kAtOnce - 1) / S::kAtOnce>([&](auto rc) {
            constexpr int first = decltype(rc)::value * S::kAtOnce, count = std::min(S::kAtOnce, S::kPartials - first);
            __syncthreads();
            static_for<0, count>([&](auto kc) {
                constexpr int k = first + decltype(kc)::value;
                float v;
                if constexpr (k < MO * MA * 4) v = dWo[k / 4 / MA][k / 4 % MA][k % 4];
                else if constexpr (k < kTiles) v = dWa[k / 4 / MA - MO][k / 4 % MA][k % 4];
                else if constexpr (k < kTiles + OTMAX) v = dbo[k - kTiles];
                else v = dba[k - kTiles - OTMAX];
                slot[(wv * count + decltype(kc)::value) * 64 + lane] = v;
            });
            __syncthreads();
            for (int i = wv; i < count; i += W) {
                float v = slot[i * 64 + lane];
#pragma unroll
                for (int w = 1; w < W; ++w) v += slot[(w * count + i) * 64 + lane];
                const int k = first + i;
                // the workgroup's block: dWo tiles, dWa tiles, dbo, dba
                if (k < kTiles) {
                    dst[k * 64 + lane] = v;
                } else {
                    v = group16_sum(v);
                    const int ks = k - kTiles, q = ks - OTMAX;
                    if (q < 0) { if (n == 0 && ks < OT) dst[kTiles * 64 + 4 * ks + g] = v; }
                    else if (n == 0 && q < HT) dst[kTiles * 64 + 4 * OT + 4 * q + g] = v;
                }
            }
        });
    } else {
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        float t = 0.0f;
#pragma unroll
        for (int i = 0; i < W; ++i) t += s_part[i];
        a.loss_partial[blockIdx.x] = t;
    }
}

// ---------------------------------------------------------------------------
// The output stage, forward, at the LAST window of every series only (out-of-sample forecasts).  One wave per 16-series
// tile: a column of the products is a series, so every lane reads the block output at its own series' position, and the
// arithmetic per column is that of head_kernel.  Replaces a pass over all positions (4096 quarterly series: 32 -> 5 us).
// The lane that has an output of step j turns it into the forecast (Eq. (4), (5); a launch of its own took 4 - 5 us):
// exp(output + ln l_t) * S1[t + (j mod m1) + 1] * S2[...], t the last observation, j from 0: the last m factors the
// recursion produced, repeated with their period.  Series that take no part (length 0) have zeros.
// ---------------------------------------------------------------------------
template <int HT, int MO>
__global__ void __launch_bounds__(256) head_last_kernel(HeadArgs a)
{
    using S = HeadShape<HT, MO>;
    constexpr int MA = S::MA, OTMAX = S::OTMAX, NPH = S::NPH, QH = S::QH;
    const int lane = threadIdx.x & 63;
    const int bt = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (bt >= a.NB) return;
    const int g = lane >> 4, n = lane & 15, b = bt * 16 + n;
    const int len = b < a.B ? min(max(a.lengths[b], 0), a.T) : 0;
    const int windows = len - a.I - a.H + 1;
    const size_t tile = (size_t)max(windows - 1, 0) * a.NB + bt;       // (a series without a window: any tile, nothing is stored)
    float br[HT];
#pragma unroll
    for (int q = 0; q < HT; ++q) br[q] = a.R[tile * HT * 64 + q * 64 + lane];
    const int t = max(len - a.H - 1, 0), col = min(b, a.B - 1);
    const float ut = a.u[(size_t)t * a.Bt + col];
    float seas[OTMAX];
#pragma unroll
    for (int ks = 0; ks < OTMAX; ++ks) {
        const int j = min(4 * ks + g, a.H - 1);
        float s1 = 1.0f, s2 = 1.0f;
        if (a.m1 > 0) s1 = a.S1[(size_t)min(t + j % a.m1 + 1, a.T - 1) * a.Bt + col];
        if (a.m2 > 0) s2 = a.S2[(size_t)min(t + j % a.m2 + 1, a.T - 1) * a.Bt + col];
        seas[ks] = s1 * s2;
    }
    f32x4 ba[MA], bo[MO], acc[MA], oc[MO];
#pragma unroll
    for (int m = 0; m < MA; ++m) ba[m] = *reinterpret_cast<const f32x4 *>(a.baF + (m * 4 + g) * 4);
#pragma unroll
    for (int m = 0; m < MO; ++m) bo[m] = *reinterpret_cast<const f32x4 *>(a.boF + (m * 4 + g) * 4);
    u32x4 ph[NPH];
    u32x4 bq[tt_b_quads(NPH)];
    split_all(br, ph);
    b_quads<NPH>(ph, bq);
    auto wa_op = [&](int m, int q) { return a.WaF[(m * QH + q) * 64 + lane]; };
    auto wo_op = [&](int m, int q) { return a.WoF[(m * QH + q) * 64 + lane]; };
    Contraction<NPH, MA, false>().sum(wa_op, bq, acc);
    float av[HT];
#pragma unroll
    for (int q = 0; q < HT; ++q) av[q] = tanh_f(acc[q >> 2][q & 3] + ba[q >> 2][q & 3]);
    split_all(av, ph);
    b_quads<NPH>(ph, bq);
    Contraction<NPH, MO, false>().sum(wo_op, bq, oc);
#pragma unroll
    for (int ks = 0; ks < OTMAX; ++ks) {
        const int j = 4 * ks + g;
        const float o = fmaf(oc[ks >> 2][ks & 3], row_scale(a.sc->infinite_rows, j), bo[ks >> 2][ks & 3]);
        if (windows >= 1 && j < a.orows) a.O[tile * a.orows * 16 + j * 16 + n] = o;
        if (b < a.B && j < a.H) a.forecasts[(size_t)b * a.H + j] = windows >= 1 ? __expf(o + ut) * seas[ks] : 0.0f;
    }
}

// ---------------------------------------------------------------------------
// Loss: sum of the per-workgroup partial sums in double, then
// loss = pinball_sum / n_pin + lambda * level_sum / n_lv + lambda_cs * cell_state_sum / n_cs.
// ---------------------------------------------------------------------------
struct LossArgs {
    const float *pin, *lv, *cs;
    int n_pin, n_lv, n_cs;
    const Scalars *sc;
    float lambda, lambda_cs;
    float *loss;
    TogetherWords words;        // of the reverse pass, in the place of operands that are not needed any more
};

// sum over the workgroup of a value per thread, in a fixed order
__device__ __forceinline__ double block_sum(double v, double *s_wave)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) s_wave[threadIdx.x >> 6] = v;
    __syncthreads();
    v = (s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]);
    __syncthreads();
    return v;
}

__device__ void loss_body(const LossArgs &a, double *s_wave)
{
    clear_words(a.words, kWordStride);
    double pin = 0.0, lv = 0.0, cs = 0.0;
    for (int i = threadIdx.x; i < a.n_pin; i += 256) pin += (double)a.pin[i];
    for (int i = threadIdx.x; i < a.n_lv; i += 256) lv += (double)a.lv[i];
    for (int i = threadIdx.x; i < a.n_cs; i += 256) cs += (double)a.cs[i];
    pin = block_sum(pin, s_wave);
    lv = block_sum(lv, s_wave);
    cs = block_sum(cs, s_wave);
    if (threadIdx.x == 0)
        *a.loss = (float)(pin * (double)a.sc->inv_n_pin + (double)a.lambda * lv * (double)a.sc->inv_n_lv +
                          (double)a.lambda_cs * cs * (double)a.sc->inv_n_cs);
}

// ---------------------------------------------------------------------------
// Forecasts of Eq. (5) at every window position: exp(output) * level * seasonal factors of the target
// time, zero where the window does not fit into the series.  One wave per (position, 16-series) tile.
// Lane (g, n) computes the steps j = g, g+4, ... of series n: the tile of outputs and the rows of the
// seasonal factors are read in their storage order.  The tile's 16 * H forecasts are contiguous in the
// [P][B][H] array but ordered [series][step]: they are turned through the wave's corner of LDS and written
// out in storage order as well.
//
// The first workgroup adds up the loss instead (a launch of its own took 4 - 5 us; done by the output-stage workgroup that
// finishes last, 256 counts of one counter and the cache write-backs that order them cost the same 4 us).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) forecast_kernel(const float *__restrict__ O, const float *__restrict__ u,
                                                        const float *__restrict__ S1, const float *__restrict__ S2,
                                                        const int32_t *__restrict__ lengths, const int32_t *__restrict__ pmax,
                                                        float *__restrict__ forecasts, int P, int NB, int B, int Bp, int T,
                                                        int I, int H, int orows, int n_seas, LossArgs loss)
{
    __shared__ __align__(16) float s_f[4][16 * ESRNN_MAX_WINDOW];
    const int lane = threadIdx.x & 63, g = lane >> 4, n = lane & 15;
    float *fl = s_f[threadIdx.x >> 6];
    if (blockIdx.x == 0) {
        loss_body(loss, reinterpret_cast<double *>(&s_f[0][0]));
        return;
    }
    const long long tile = (long long)(blockIdx.x - 1) * 4 + (threadIdx.x >> 6);
    if (tile >= (long long)P * NB) return;              // (no workgroup barrier below)
    const int p = (int)(tile / NB), bt = (int)(tile % NB);
    const int t = p + I - 1;
    const int b = bt * 16 + n;
    const int cols = min(16, B - bt * 16);              // series of this tile that exist
    const int len = b < B ? min(max(lengths[b], 0), T) : 0;
    const bool valid = p < pmax[bt] && p < len - I - H + 1;     // past pmax the tile of outputs holds nothing
    const float ut = valid ? u[(size_t)t * Bp + b] : 0.0f;
    const float *ot = O + (size_t)tile * orows * 16;
    // Several steps' operands at a time, in range by choice of address (behind a condition each, a lane waited for every one
    // of them: 50 us at 512 hourly series, 44 us at 4096 monthly ones; now 34 and 41 us, 128 and 124 MB).
    const int col = min(b, Bp - 1);
    auto steps = [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        for (int j0 = g; j0 < H; j0 += 4 * K) {
            float o[K], s1[K], s2[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int j = min(j0 + 4 * k, H - 1);
                const size_t at = (size_t)min(t + 1 + j, T - 1) * Bp + col;
                o[k] = ot[j * 16 + n];
                s1[k] = n_seas >= 1 ? S1[at] : 1.0f;
                s2[k] = n_seas >= 2 ? S2[at] : 1.0f;
            }
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (j0 + 4 * k < H) fl[n * H + j0 + 4 * k] = valid ? __expf(o[k] + ut) * (s1[k] * s2[k]) : 0.0f;
        }
    };
    if (H <= 8) steps(std::integral_constant<int, 2>{});
    else steps(std::integral_constant<int, 4>{});
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // same wave: LDS serves its instructions in order
    float *ft = forecasts + ((size_t)p * B + bt * 16) * H;
    for (int e = lane; e < cols * H; e += 64) ft[e] = fl[e];
}

#define ESRNN_HEAD_SHAPES(X) \
    X(2, 1) X(2, 2) X(2, 3) X(2, 4) X(8, 1) X(8, 2) X(8, 3) X(8, 4) X(10, 1) X(10, 2) X(10, 3) X(10, 4) \
    X(13, 1) X(13, 2) X(13, 3) X(13, 4) X(16, 1) X(16, 2) X(16, 3) X(16, 4)

}  // namespace

hipError_t launch_loss_and_forecasts(const Plan &pl, const int32_t *lengths, float *ws, float *loss, float *forecasts, hipStream_t st)
{
    const esrnn_config &c = pl.cfg;
    const LossArgs la{ws + pl.loss_partial, ws + pl.loss_partial + pl.head_blocks, ws + pl.cs_partial, pl.head_blocks, pl.es_blocks,
                      pl.n_cs_partial, reinterpret_cast<const Scalars *>(ws + pl.scalars), c.lambda_lv, c.lambda_cs, loss,
                      TogetherWords{reinterpret_cast<unsigned *>(ws + pl.together_words_bwd), pl.together_bwd ? 1 + pl.together_groups_bwd : 0}};
    const long long tiles = forecasts ? (long long)pl.P * pl.NB : 0;
    forecast_kernel<<<(unsigned)(1 + (tiles + 3) / 4), 256, 0, st>>>(
        ws + pl.O, ws + pl.u, ws + pl.S1, ws + pl.S2, lengths, reinterpret_cast<const int32_t *>(ws + pl.pmax), forecasts,
        pl.P, pl.NB, pl.B, pl.Bt, pl.T, pl.I, pl.H, pl.OP, pl.cfg.n_seas, la);
    return hipGetLastError();
}

namespace {
HeadArgs head_args(const Plan &pl, const int32_t *lengths, float *ws, float *forecasts)
{
    const esrnn_config &c = pl.cfg;
    const HeadPack hp = head_pack_layout(pl);
    const float *f = ws + pl.head_fwd_pack, *bk = ws + pl.head_bwd_pack;
    auto quads = [](const float *at) { return reinterpret_cast<const u32x4 *>(at); };
    return HeadArgs{quads(f + hp.WaF), quads(f + hp.WoF), quads(bk + hp.WoT), quads(bk + hp.WaT), f + hp.baF, f + hp.boF,
                    ws + pl.blk_out[pl.cfg.n_blocks - 1], ws + pl.Z, lengths,
                    reinterpret_cast<const int32_t *>(ws + pl.pmax), reinterpret_cast<const Scalars *>(ws + pl.scalars), ws + pl.O, ws + pl.loss_partial,
                    ws + pl.gO, ws + pl.gTop, ws + pl.head_dw_partial,
                    pl.P, pl.NB, pl.B, pl.T, pl.I, pl.H, pl.head_dw_stride, pl.OP, c.tau,
                    forecasts, ws + pl.u, ws + pl.S1, ws + pl.S2, pl.Bt,
                    c.n_seas >= 1 ? c.m1 : 0, c.n_seas >= 2 ? c.m2 : 0};
}
}  // namespace

hipError_t launch_head(const Plan &pl, const int32_t *lengths, float *ws, bool reverse, hipStream_t st)
{
    const int blocks = pl.head_blocks;
    const HeadArgs a = head_args(pl, lengths, ws, nullptr);
#define X(HT_, MO_)                                              \
    if (pl.HT == HT_ && pl.MO == MO_) {                          \
        if (reverse) head_kernel<HT_, MO_, true><<<blocks, 64 * head_waves(HT_, MO_), 0, st>>>(a); \
        else head_kernel<HT_, MO_, false><<<blocks, 64 * head_waves(HT_, MO_), 0, st>>>(a); \
        return hipGetLastError();                                \
    }
    ESRNN_HEAD_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_head_last(const Plan &pl, const int32_t *lengths, float *ws, float *forecasts, hipStream_t st)
{
    const HeadArgs a = head_args(pl, lengths, ws, forecasts);
#define X(HT_, MO_)                                                              \
    if (pl.HT == HT_ && pl.MO == MO_) {                                          \
        head_last_kernel<HT_, MO_><<<(pl.NB + 3) / 4, 256, 0, st>>>(a);          \
        return hipGetLastError();                                                \
    }
    ESRNN_HEAD_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace esrnn
