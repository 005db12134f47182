// Streaming kernels of the training step: loss normalisers, operand packing,
// exponential-smoothing recursions (forward and adjoint), window extraction
// (forward and adjoint), loss reduction and weight-gradient reduction.
#include <algorithm>
#include <mutex>
#include <numeric>
#include <type_traits>

#include "device_utils.h"
#include "esrnn_internal.h"
#include "three_term.h"

namespace esrnn {

namespace {

__device__ __forceinline__ int clamp_len(int len, int T) { return len < 0 ? 0 : (len > T ? T : len); }

// What the caller's lengths mean to a call.  Training: the observations there are.  Out-of-sample forecasts (extend = H):
// every series runs H steps further, so that the window that ends at its last observation counts as complete; a series too
// short for one window, or too long for H more rows, takes no part.
struct Lengths {
    const int32_t *of;
    int T, I, extend;
    __device__ int run(int len) const
    {
        if (extend == 0) return clamp_len(len, T);
        return len >= I && len <= T - extend ? len + extend : 0;
    }
    __device__ int at(int b) const { return run(of[b]); }
};

// ---------------------------------------------------------------------------
// Loss normalisers (Section 3.5: padded outputs are masked out of the loss).
// ---------------------------------------------------------------------------
struct PrepArgs {
    Lengths lengths;
    Scalars *sc;
    int32_t *pmax;       // [NB] window positions needed by the longest series of every 16-series tile
    int NB;
    int B, H;
    int cs_per_window;   // cell-state values per valid window in the cell-state penalty: hidden * blocks
    TogetherWords words; // of the forward pass
};

// One workgroup reads all lengths, eight requests in flight per thread, of four lengths each where the caller's array is
// aligned for that (65 536 series: 26 us a length at a time as a launch of its own; now beside the recursions, which take
// 18 us).  The counts are whole numbers: any order of adding them up gives the same sums.
__device__ __forceinline__ void prep_body(const PrepArgs &pa, float *scratch)
{
    const Lengths L = pa.lengths;
    clear_words(pa.words, kWordStride);
    unsigned long long *s_pin = reinterpret_cast<unsigned long long *>(scratch), *s_lv = s_pin + 256;
    unsigned long long np_ = 0, nl = 0;
    auto count = [&](int raw) {
        const int l = L.run(raw), windows = l - L.I - pa.H + 1;
        if (windows > 0) np_ += (unsigned)windows;
        if (l > 2) nl += (unsigned)(l - 2);
    };
    const bool aligned = (reinterpret_cast<size_t>(L.of) & 15) == 0;
    const int quads = aligned ? pa.B / 4 : 0;
    for (int q0 = threadIdx.x; q0 < quads; q0 += 8 * 256) {
        int4 len[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int q = q0 + k * 256;
            len[k] = reinterpret_cast<const int4 *>(L.of)[q < quads ? q : quads - 1];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (q0 + k * 256 < quads) { count(len[k].x); count(len[k].y); count(len[k].z); count(len[k].w); }
    }
    for (int b0 = 4 * quads + threadIdx.x; b0 < pa.B; b0 += 8 * 256) {
        int len[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) len[k] = L.of[min(b0 + k * 256, pa.B - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (b0 + k * 256 < pa.B) count(len[k]);
    }
    s_pin[threadIdx.x] = np_;
    s_lv[threadIdx.x] = nl;
    __syncthreads();
    for (int off = 128; off >= 1; off >>= 1) {
        if ((int)threadIdx.x < off) {
            s_pin[threadIdx.x] += s_pin[threadIdx.x + off];
            s_lv[threadIdx.x] += s_lv[threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double windows = (double)s_pin[0], n_pin = windows * pa.H, n_lv = (double)s_lv[0];
        pa.sc->inv_n_pin = n_pin > 0.0 ? (float)(1.0 / n_pin) : 0.0f;
        pa.sc->inv_n_lv = n_lv > 0.0 ? (float)(1.0 / n_lv) : 0.0f;
        const double n_cs = windows * (double)pa.cs_per_window;   // valid windows x hidden x blocks
        pa.sc->inv_n_cs = n_cs > 0.0 ? (float)(1.0 / n_cs) : 0.0f;
    }
}

// Ragged batches (Section 8.1: padding multiplies the iterations of the recursions): every later kernel
// stops a 16-series tile at the number of window positions its longest series has.  One thread per tile.
__device__ __forceinline__ void pmax_body(const PrepArgs &pa, int block, int n_blocks)
{
    for (int bt = block * 256 + threadIdx.x; bt < pa.NB; bt += n_blocks * 256) {
        int best = 0;
        for (int k = 0; k < kTileN; ++k) {
            const int b = bt * kTileN + k;
            if (b < pa.B) best = max(best, pa.lengths.at(b) - pa.lengths.I - pa.H + 1);
        }
        pa.pmax[bt] = best;
    }
}

// ---------------------------------------------------------------------------
// Operand packing: weights rearranged into the per-lane operand order of the
// 16x16x4 MFMA (lane l supplies A[l%16][l/16]) so that every wave loads its
// register-resident slice with coalesced reads.
// ---------------------------------------------------------------------------
struct PackLstmArgs {
    const float *W, *b;
    float *fwd, *bias, *bwd;
    int h, in_dim, HT, KXT;
    int narrow_fwd, narrow_bwd;   // operand orders of the 4-series kernels (4x4x1 MFMA) instead

    // element of W for gate `gate` of hidden unit `unit` and row `u` of the layer input or the recurrent state; zero
    // in the padding
    __device__ float at(int gate, int unit, bool in_x, int u) const
    {
        const bool exists = unit < h && u < (in_x ? in_dim : h);
        return exists ? W[(size_t)(gate * h + unit) * (in_dim + h) + (in_x ? u : in_dim + u)] : 0.0f;
    }
    // the same for a row of [x ; h] in whole unit tiles
    __device__ float at_row(int gate, int unit, int row) const
    {
        const int KX = 4 * KXT;
        return row < KX ? at(gate, unit, true, row) : row < KX + 4 * HT ? at(gate, unit, false, row - KX) : 0.0f;
    }
};

// Operands of the 4-series kernels.  v_mfma_f32_4x4x1: lane l supplies A[l%4] of block l/4.
//   forward  [wave][column k of h][lane]: gate l/16 of unit wave*HT + min(l%16, HT-1) (the lanes past HT
//            repeat the last unit, so that all lanes do the same work on the same addresses); then those of x
//            for v_mfma_f32_16x16x4, [wave][column tile][unit tile k of x][lane]: column c = 16*tile + l%16, gate c/HT of unit
//            wave*HT + c%HT, row 4*k + l/16 of x
//   reverse  [wave][group g][k-step 4*u + gate][lane]: W[gate, unit wave*HT + u][column 64*g + l]
__device__ __forceinline__ void pack_forward_narrow(const PackLstmArgs &a, int block, int n_blocks)
{
    const int HP = 4 * a.HT, n = 4 * HP * 64;
    for (int idx = block * 256 + threadIdx.x; idx < n; idx += n_blocks * 256) {
        const int lane = idx & 63, k = (idx >> 6) % HP, w = (idx >> 6) / HP;
        a.fwd[idx] = a.at(lane >> 4, w * a.HT + min(lane & 15, a.HT - 1), false, k);
    }
    const int tiles = (a.HT + 3) / 4, nx = 4 * tiles * a.KXT * 64;
    for (int idx = block * 256 + threadIdx.x; idx < nx; idx += n_blocks * 256) {
        const int lane = idx & 63, k = (idx >> 6) % a.KXT, t = (idx >> 6) / a.KXT % tiles, w = (idx >> 6) / (a.KXT * tiles);
        const int c = 16 * t + (lane & 15);
        a.fwd[n + idx] = c < HP ? a.at(c / a.HT, w * a.HT + c % a.HT, true, 4 * k + (lane >> 4)) : 0.0f;
    }
}
__device__ __forceinline__ void pack_backward_narrow(const PackLstmArgs &a, int block, int n_blocks)
{
    const int NG = (4 * (a.KXT + a.HT) + 63) / 64, n = 4 * NG * 4 * a.HT * 64;
    for (int idx = block * 256 + threadIdx.x; idx < n; idx += n_blocks * 256) {
        const int lane = idx & 63, ks = (idx >> 6) % (4 * a.HT), g = ((idx >> 6) / (4 * a.HT)) % NG, w = (idx >> 6) / (4 * a.HT * NG);
        a.bwd[idx] = a.at_row(ks & 3, w * a.HT + (ks >> 2), 64 * g + lane);
    }
}

// Operands of the 16-series forward kernel: three bf16 parts of W (three_term.h) as [unit tile][quads of x, then of
// h][lane][dword], and the bias as [unit tile][unit][gate].  Row 4g+r of unit tile mt is gate r of unit 4mt+g; lane
// group k of a pair of input tiles stands for unit k of each.
__device__ __forceinline__ void pack_forward(const PackLstmArgs &a, int block, int n_blocks)
{
    const int npx = (a.KXT + 1) / 2, nph = (a.HT + 1) / 2, qx = tt_a_quads(npx), quads = qx + tt_a_quads(nph);
    const int n = a.HT * quads * 256;
    for (int idx = block * 256 + threadIdx.x; idx < n; idx += n_blocks * 256) {
        const int d = idx & 3, lane = (idx >> 2) & 63, q = (idx >> 8) % quads, mt = (idx >> 8) / quads;
        const int i = lane & 15, k = lane >> 4, unit = 4 * mt + (i >> 2), gate = i & 3;
        const bool in_x = q < qx;
        const TtDword w = tt_a_dword(in_x ? npx : nph, in_x ? q : q - qx, d);
        const Parts p = split_pair(splittable(a.at(gate, unit, in_x, 8 * w.pair + k)), splittable(a.at(gate, unit, in_x, 8 * w.pair + 4 + k)));
        reinterpret_cast<unsigned *>(a.fwd)[idx] = part_of(p, w.part);
    }
    for (int j = block * 256 + threadIdx.x; j < a.HT * 16; j += n_blocks * 256) {
        const int gate = j & 3, unit = j >> 2;   // (mt*4+g)*4 + r  ->  unit = 4mt+g
        a.bias[j] = unit < a.h ? a.b[gate * a.h + unit] : 0.0f;
    }
}

// Operands of the 16-series reverse kernel: three bf16 parts of W^T as [row tile][unit tile][part][lane][dword].  Lane
// group k of unit tile t is unit 4t+k, its dwords are the gate pairs (0, 1) and (2, 3); row 4g+r of a row tile is unit
// g of its unit tile r.  The row tiles of x come first; the unit tiles of the others are those of h and then the
// merged ones of x (three_term.h).
__device__ __forceinline__ void pack_backward(const PackLstmArgs &a, int block, int n_blocks)
{
    const int rx = bwd_x_row_tiles(a.HT, a.KXT), ml = bwd_merged_tiles(a.HT, a.KXT), tiles = bwd_even_tiles(a.HT);
    const int n = bwd_pack_dwords(a.HT, a.KXT);
    for (int idx = block * 256 + threadIdx.x; idx < n; idx += n_blocks * 256) {
        const int d = idx & 1, lane = (idx >> 1) & 63, part = (idx >> 7) % 3, t = (idx / 384) % tiles, rt = idx / (384 * tiles);
        const int i = lane & 15, unit = 4 * t + (lane >> 4);
        const int slot = 4 * (rt < rx ? rt : rt - rx) + (i & 3);
        const bool merged = rt >= rx && slot >= a.HT, exists = !merged || slot < a.HT + ml;
        const bool in_x = rt < rx || merged;
        const int row = 4 * (merged ? 4 * rx + slot - a.HT : slot) + (i >> 2);
        const Parts p = split_pair(exists ? a.at(2 * d, unit, in_x, row) : 0.0f, exists ? a.at(2 * d + 1, unit, in_x, row) : 0.0f);
        reinterpret_cast<unsigned *>(a.bwd)[idx] = part_of(p, part);
    }
}

// The same for the fp32 kernel (hidden sizes above 52).  Transposed contraction: k-step 4mt+gate, lane group = unit within
// tile; output row 4g+r of tile mb is row g of input unit tile 4mb+r.
__device__ __forceinline__ void pack_backward_fp32(const PackLstmArgs &a, int block, int n_blocks)
{
    const int MB = (a.KXT + a.HT + 3) / 4, n = MB * 4 * a.HT * 64;
    for (int idx = block * 256 + threadIdx.x; idx < n; idx += n_blocks * 256) {
        const int lane = idx & 63, ks = (idx >> 6) % (4 * a.HT), mb = (idx >> 6) / (4 * a.HT);
        const int i = lane & 15;
        a.bwd[idx] = a.at_row(ks & 3, 4 * (ks >> 2) + (lane >> 4), 4 * (4 * mb + (i & 3)) + (i >> 2));
    }
}

__device__ __forceinline__ void pack_lstm_body(const PackLstmArgs &a, int block, int n_blocks)
{
    if (a.narrow_fwd) pack_forward_narrow(a, block, n_blocks);
    else pack_forward(a, block, n_blocks);
    if (a.narrow_bwd) pack_backward_narrow(a, block, n_blocks);
    else if (bwd_three_term(a.HT)) pack_backward(a, block, n_blocks);
    else pack_backward_fp32(a, block, n_blocks);
}

struct PackHeadArgs {
    const float *Wa, *ba, *Wo, *bo;
    float *WaF, *baF, *WoF, *boF, *WoT, *WaT;
    Scalars *sc;
    int h, H, HT, MA, MO;
};

// An infinity has no parts: inf, NaN, NaN.  Forward, the largest number that has three parts stands for it: in the tanh
// layer it saturates a unit, and the linear layer finds the rows that are to be infinite in Scalars::infinite_rows.
// Transposed, where an infinite weight meets a gradient that is zero (of a saturated unit, of a masked output) and others
// that are not, NaN does.  (A run that has diverged is to see it in its loss and its gradients, as with fp32 products.)
__device__ __forceinline__ float finite_parts(float x)
{
    return __builtin_fabsf(x) >= 0x1.ffp127f ? __builtin_copysignf(0x1.fep127f, x) : x;      // (halfway to 2^128)
}
__device__ __forceinline__ float nan_parts(float x) { return __builtin_isinf(x) ? __builtin_nanf("") : finite_parts(x); }

// One workgroup; `found`: 4 words of LDS
__device__ __forceinline__ void infinite_rows_body(const PackHeadArgs &a, unsigned long long *found)
{
    constexpr int per = ESRNN_MAX_WINDOW / 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float w[per];
#pragma unroll
    for (int k = 0; k < per; ++k) w[k] = a.Wo[min(4 * k + wave, a.H - 1) * a.h + min(lane, a.h - 1)];
    unsigned long long rows = 0;
#pragma unroll
    for (int k = 0; k < per; ++k)
        if (__ballot(__builtin_isinf(w[k])) != 0 && 4 * k + wave < a.H) rows |= 1ull << (4 * k + wave);
    if (lane == 0) found[wave] = rows;
    __syncthreads();
    if (threadIdx.x == 0) a.sc->infinite_rows = found[0] | found[1] | found[2] | found[3];
}

// Operands of the output stage (head_kernels.hip): three bf16 parts as [tile][quad][lane][dword], rows in unit-tile order:
// row 4g+r of tile m is row 4(4m+r)+g of the product.
__device__ __forceinline__ void pack_head_body(const PackHeadArgs &a, int block, int n_blocks, float *scratch)
{
    if (block == n_blocks - 1) infinite_rows_body(a, reinterpret_cast<unsigned long long *>(scratch));   // (has the least to pack)
    const int np_h = (a.HT + 1) / 2, np_o = 2 * a.MO, qh = tt_a_quads(np_h), qo = tt_a_quads(np_o);
    auto pack = [&](float *dst, int tiles, int quads, int np, auto &&at) {      // at(row, column), zero outside
        for (int idx = block * 256 + threadIdx.x; idx < tiles * quads * 256; idx += n_blocks * 256) {
            const int d = idx & 3, lane = (idx >> 2) & 63, q = (idx >> 8) % quads, m = (idx >> 8) / quads;
            const int i = lane & 15, k = lane >> 4, row = 4 * (4 * m + (i & 3)) + (i >> 2);
            const TtDword w = tt_a_dword(np, q, d);
            const Parts p = split_pair(at(row, 8 * w.pair + k), at(row, 8 * w.pair + 4 + k));
            reinterpret_cast<unsigned *>(dst)[idx] = part_of(p, w.part);
        }
    };
    auto wa = [&](int out, int in) { return out < a.h && in < a.h ? a.Wa[out * a.h + in] : 0.0f; };
    auto wo = [&](int out, int in) { return out < a.H && in < a.h ? a.Wo[out * a.h + in] : 0.0f; };
    pack(a.WaF, a.MA, qh, np_h, [&](int unit, int in) { return finite_parts(wa(unit, in)); });
    pack(a.WoF, a.MO, qh, np_h, [&](int out, int in) { return finite_parts(wo(out, in)); });
    pack(a.WoT, a.MA, qo, np_o, [&](int unit, int out) { return nan_parts(wo(out, unit)); });
    pack(a.WaT, a.MA, qh, np_h, [&](int unit, int out) { return nan_parts(wa(out, unit)); });
    for (int j = block * 256 + threadIdx.x; j < 16 * (a.MA + a.MO); j += n_blocks * 256) {
        const bool second = j >= 16 * a.MA;
        const int e = second ? j - 16 * a.MA : j;
        const int row = 4 * (4 * (e >> 4) + (e & 3)) + ((e >> 2) & 3);
        if (second) a.boF[e] = row < a.H ? a.bo[row] : 0.0f;
        else a.baF[e] = row < a.h ? a.ba[row] : 0.0f;
    }
}

// Out-of-sample forecasts, Section 3.4 with Eq. (4) and (5): the forward pass is run with every length extended by H (the
// rows past a series never reach its forecast: the network is causal in the window position).  The later kernels read the
// extended lengths from `ext`.
//
// The same workgroups find what those outputs depend on: per 16-series tile and layer, the residue classes of the dilation
// that the forward kernels have to walk (ForwardMode::need).  Top layer: the classes of the last windows.  Below: a layer is
// read at the positions of the classes above it, which fall into every class congruent to one of those modulo the common
// divisor g of the two dilations.  (Where every position is a class of its own, any multiple of the other dilation stands
// for this one: g is that other dilation.)  One thread per series, sixteen of a tile next to each other.
struct ClassArgs {
    Lengths lengths;
    int32_t *ext;        // [B]
    unsigned *need;      // [L][NB][kNeedWords]; null: not wanted
    int L, NB, B;
    int dil[kMaxLayers], gcd_above[kMaxLayers];   // gcd_above[l]: g of layers l and l + 1
};
__device__ __forceinline__ void extend_body(const ClassArgs &a, int block, unsigned *masks)
{
    // masks: [this layer, the one above][tile][word]
    const int b = block * 256 + threadIdx.x;
    const int len = b < a.B ? a.lengths.at(b) : 0;      // (a series that takes no part has length 0)
    if (b < a.B) a.ext[b] = len;
    if (!a.need) return;
    const int last = len - a.lengths.extend - a.lengths.I;      // its last window
    const int grp = threadIdx.x >> 4, k = threadIdx.x & 15, bt = b >> 4;
    for (int l = a.L - 1; l >= 0; --l) {
        const int d = a.dil[l];
        unsigned *mine = masks + ((l & 1) * 16 + grp) * kNeedWords;
        const unsigned *over = masks + (((l + 1) & 1) * 16 + grp) * kNeedWords;
        __syncthreads();
        if (k < kNeedWords) mine[k] = 0u;
        __syncthreads();
        if (d <= kNeedMost) {                           // (more classes than bits: the mask is not read)
            if (l == a.L - 1) {
                if (len > 0) atomicOr(&mine[last % d >> 5], 1u << (last % d & 31));
            } else {
                const int above = a.dil[l + 1], g = a.gcd_above[l];
                for (int r = k; r < g; r += 16) {
                    bool any = above > kNeedMost;
                    for (int q = r; q < above && !any; q += g) any = (over[q >> 5] >> (q & 31)) & 1;
                    if (any)
                        for (int q = r; q < d; q += g) atomicOr(&mine[q >> 5], 1u << (q & 31));
                }
            }
        }
        __syncthreads();
        if (k < kNeedWords && bt < a.NB) a.need[((size_t)l * a.NB + bt) * kNeedWords + k] = mine[k];
    }
}

// Everything that only depends on the weights and the lengths, by workgroup: the loss normalisers, the position bounds,
// the extended lengths, the operands of every layer and of the output stage.  `scratch`: kSetupScratch floats of LDS.
constexpr int kSetupScratch = 1024;
struct SetupArgs {
    PackLstmArgs lstm[kMaxLayers];
    PackHeadArgs head;
    PrepArgs prep;
    ClassArgs classes;
    int L, pmax_blocks, extend_blocks, pack_blocks;     // pack_blocks: per layer (0: nothing is packed)
    int blocks() const { return 1 + pmax_blocks + extend_blocks + (pack_blocks ? (L + 1) * pack_blocks : 0); }
};
__device__ __forceinline__ void setup_body(const SetupArgs &a, int block, float *scratch)
{
    if (block == 0) { prep_body(a.prep, scratch); return; }
    block -= 1;
    if (block < a.pmax_blocks) { pmax_body(a.prep, block, a.pmax_blocks); return; }
    block -= a.pmax_blocks;
    if (block < a.extend_blocks) { extend_body(a.classes, block, reinterpret_cast<unsigned *>(scratch)); return; }
    block -= a.extend_blocks;
    const int z = block / a.pack_blocks, k = block % a.pack_blocks;
    if (z < a.L) pack_lstm_body(a.lstm[z], k, a.pack_blocks);
    else pack_head_body(a.head, k, a.pack_blocks, scratch);
}

// ---------------------------------------------------------------------------
// Exponential-smoothing recursions, Section 3.1 Eq. (1) and (3) without trend;
// Section 8.2 variants (two seasonalities, none).  One lane per series, time
// sequential; every load and store is one contiguous row segment of a
// time-major array.  The seasonal factors that will apply m steps ahead live
// in a per-lane ring in LDS (slot t mod m holds the factor for time t until
// step t has used it, then the factor for time t + m).
// ---------------------------------------------------------------------------
struct EsArgs {
    const float *y;           // [T][B]
    Lengths lengths;
    const float *es;          // [K][B]
    float *lvl, *S1, *S2, *u, *v;   // [T][Bp], one column per lane of every wave
    float *lv_partial;        // [blocks]
    int blocks;               // workgroups of the recursions; the launch's others do the set-up
    int B, Bp, T, n_seas, m1, m2, logit;   // Bp: row stride of the time-major arrays (batch padded to 64)
    int row_gamma1, row_gamma2, row_s1, row_s2;
};

// CS: how many consecutive time steps take their seasonal factors out of the ring together (and put the
// new ones back together): a divisor of 8 not larger than the shorter period, so that no factor a group
// reads is produced inside the group.  Within a group the steps are then plain register arithmetic whose
// only chain is the level (one multiply-add per step); divisions and seasonal updates of the other steps
// overlap with it.
//
// Division of labour.  A workgroup serves 64 series with three or four waves.  Wave 0 runs the recursion and
// nothing else: it reads observations (several chunks ahead), keeps the rings, and leaves level,
// de-seasonalised value and factors of every step in an LDS staging buffer; it issues no global store and
// computes no logarithm.  Of the previous chunk, wave 1 forms the level penalty, wave 2 turns the staged level into
// lvl and u = ln(level) and the staged value into v, and wave 3 (seasonal shapes) stores the factors.  A lone
// wave issues one instruction every few cycles whatever the instruction is; with the chain, five stores and two
// logarithms per step on the same wave a step took about three times as long as the chain alone.
constexpr int kEsChunk = 8;                 // steps per staging buffer
constexpr int kEsAhead = 4;                 // chunks between the request of a row and its use
// staged per step: level, de-seasonalised value, and one factor per seasonality
constexpr int es_stage_floats(int n_seas) { return 2 * kEsChunk * (2 + n_seas) * 64; }


// Storing of staged rows, four steps and four series a lane: a quarter of the stores (a wave has at most 63 under way) and of
// the instructions around them.  501 monthly series 24.0 -> 23.4 us, 65 536 quarterly ones 27.4 -> 26.7 us, 16 9.7 -> 9.3 us;
// with long periods, below, 0.55 -> 0.47 us a chunk.
struct ChunkRows {
    int row, col, t_end, lens[4];       // this lane's step of four, its first series, and the lengths of its series
    size_t base, Bp;
    __device__ ChunkRows(int Bp_, int t_end_, int len) : row((threadIdx.x & 63) >> 4), col(4 * (threadIdx.x & 15)), t_end(t_end_), Bp(Bp_)
    {
        base = (size_t)blockIdx.x * 64 + col;
#pragma unroll
        for (int e = 0; e < 4; ++e) lens[e] = __shfl(len, col + e, 64);
    }
    // of a row of 64 series staged every `stride` floats from `at` on
    __device__ f32x4 quad(const float *at, int stride) const { return *reinterpret_cast<const f32x4 *>(at + row * stride + col); }
    __device__ f32x4 logs(const f32x4 &v) const { return f32x4{fast_log(v[0]), fast_log(v[1]), fast_log(v[2]), fast_log(v[3])}; }
    // row t (if the wave's series go that far), the padding value past a series' end
    __device__ void put(float *to, int t, const f32x4 &v, float pad) const
    {
        f32x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = t < lens[e] ? v[e] : pad;
        if (t < t_end) *reinterpret_cast<f32x4 *>(to + (size_t)t * Bp + base) = r;
    }
};

// The set-up work needs nothing of the recursions and they nothing of it, and neither fills the chip: one launch has both
// (as two launches: 11 + 6.5 us at 4096 quarterly series, 9.9 + 4.8 us at 16; a forecast had a third one for the lengths).
template <int NS, int CS>
__global__ void __launch_bounds__(256) es_forward_kernel(EsArgs a, SetupArgs setup)
{
    extern __shared__ __align__(16) float ring[];   // [m1 + m2][64] rings, then [2][kEsChunk][2 + NS][64] staging
    if ((int)blockIdx.x >= a.blocks) {
        setup_body(setup, blockIdx.x - a.blocks, ring);
        return;
    }
    constexpr int CH = kEsChunk, NF = 2 + NS;
    static_assert(CH % CS == 0, "groups tile a chunk");
    const int role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (NS == 0 && role == 3) return;       // (no seasonal factors to store)
    const int lane = threadIdx.x & 63;
    const int b = blockIdx.x * 64 + lane;
    const bool in_batch = b < a.B;
    const int len = in_batch ? a.lengths.at(b) : 0;
    float *ring1 = ring, *ring2 = ring + (size_t)a.m1 * 64;
    float *stage = ring + (size_t)(a.m1 + a.m2) * 64;       // [buffer][step][lt, q, s1, s2][lane]
    // Ragged batches (Section 8.1): the sweep ends at the longest series of the wave.  Rows between a
    // series' own length and that bound get the defined padding values; rows beyond it are neither written
    // here nor read by any later kernel (their bounds are those of 16-series tiles, never larger).
    // (every wave of the workgroup holds the same 64 series, so the bound is the same in all of them)
    const int t_end = wave_max_int(len);
    const int n_chunks = (t_end + CH - 1) / CH;
    // Every lane owns a column of the time-major arrays (their rows are padded to whole waves), so no store
    // is ever skipped and a row address is a wave-uniform base plus the lane: scalar address arithmetic.
    const unsigned ub = b;

    // Initial seasonal factors into the rings (ring 2 follows ring 1): all waves of the workgroup share the
    // rows, eight requests in flight each - read one after the other by a single wave, the m1 + m2 rows of a
    // long-period shape took longer than the whole recursion.
    {
        constexpr int NWV = NS == 0 ? 3 : 4;
        const int rows = a.m1 + a.m2;
        for (int k0 = role * 8; k0 < rows; k0 += NWV * 8) {
            float sv[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = min(k0 + j, rows - 1);
                const int row = k < a.m1 ? a.row_s1 + k : a.row_s2 + (k - a.m1);
                sv[j] = in_batch ? a.es[(size_t)row * a.B + b] : 1.0f;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (k0 + j < rows) ring[(k0 + j) * 64 + lane] = (a.logit && in_batch) ? expf(sv[j]) : sv[j];
        }
        __syncthreads();
    }
    if (role == 0) {
        float alpha = 0.5f, g1 = 0.0f, g2 = 0.0f;
        if (in_batch) {
            alpha = a.es[b];
            if (NS >= 1) g1 = a.es[(size_t)a.row_gamma1 * a.B + b];
            if (NS >= 2) g2 = a.es[(size_t)a.row_gamma2 * a.B + b];
            if (a.logit) {
                alpha = 1.0f / (1.0f + expf(-alpha));
                g1 = 1.0f / (1.0f + expf(-g1));
                g2 = 1.0f / (1.0f + expf(-g2));
            }
        }
        float l_prev = 1.0f;
        int i1 = 0, i2 = 0;           // ring slot of the current time: t mod m
        const float one_m_alpha = 1.0f - alpha;

        // CS consecutive steps t0 .. t0+CS-1, staged at `out`.  WRAP: whether a ring index may pass the end of
        // its ring inside the group; if not, the group's slots are consecutive and every LDS address is one
        // per-lane base plus a constant.  (Always inlined: in a call, as the compiler makes them for short groups, the
        // observations lie in scratch; 240 steps with a period of 1 of two took 82 us, now 33.)
        auto steps = [&](auto wrap, int t0, const float *yv, float *out) __attribute__((always_inline)) {
            constexpr bool WRAP = decltype(wrap)::value;
            float s1v[CS], s2v[CS], w1v[CS], w2v[CS];
            float *r1 = ring1 + i1 * 64 + lane, *r2 = ring2 + i2 * 64 + lane;
            auto slot1 = [&](int k) { return WRAP ? ring1 + (i1 + k < a.m1 ? i1 + k : i1 + k - a.m1) * 64 + lane : r1 + k * 64; };
            auto slot2 = [&](int k) { return WRAP ? ring2 + (i2 + k < a.m2 ? i2 + k : i2 + k - a.m2) * 64 + lane : r2 + k * 64; };
#pragma unroll
            for (int k = 0; k < CS; ++k) {
                s1v[k] = NS >= 1 ? *slot1(k) : 1.0f;             // CS <= m: at most one wrap
                s2v[k] = NS >= 2 ? *slot2(k) : 1.0f;
            }
#pragma unroll
            for (int k = 0; k < CS; ++k) {
                const int t = t0 + k;
                // Past the end of a series the observation is replaced by 1: levels and factors stay finite,
                // the storing waves replace what they write there by the padding values.
                const float yt = t < len ? yv[k] : 1.0f;
                const float s1 = s1v[k], s2 = s2v[k];
                const float r12 = fast_rcp(s1 * s2);         // one reciprocal serves 1/(s1 s2), 1/s1 and 1/s2
                const float q = yt * r12;
                // reading for the state before the first observation: l_{-1} = y_0 / S[0]
                const float lt = (t == 0) ? q : alpha * q + one_m_alpha * l_prev;
                // Eq. (3): divide by the previous level (and the other factor); at t = 0 the produced factor
                // equals the initial one
                const float ry = yt * fast_rcp(l_prev);
                w1v[k] = (NS >= 1 && t >= 1) ? g1 * ry * (NS >= 2 ? r12 * s1 : 1.0f) + (1.0f - g1) * s1 : s1;
                w2v[k] = (NS >= 2 && t >= 1) ? g2 * ry * (r12 * s2) + (1.0f - g2) * s2 : s2;
                float *o = out + k * NF * 64 + lane;
                o[0] = lt;
                o[64] = q;
                if (NS >= 1) o[128] = s1;
                if (NS >= 2) o[192] = s2;
                l_prev = t < len ? lt : l_prev;
            }
#pragma unroll
            for (int k = 0; k < CS; ++k) {
                if (NS >= 1) *slot1(k) = w1v[k];     // the factor for time t + m
                if (NS >= 2) *slot2(k) = w2v[k];
            }
            if (NS >= 1) { i1 += CS; if (i1 >= a.m1) i1 -= a.m1; }
            if (NS >= 2) { i2 += CS; if (i2 >= a.m2) i2 -= a.m2; }
        };
        // Observations are requested kEsAhead chunks ahead: a request takes about as long as a chunk of steps,
        // and one chunk of lead made every chunk wait for memory.  The register sets rotate through a loop
        // unrolled kEsAhead times, so that their indices are constants.  Row offsets in 32 bits (B * T is at
        // most 2^30): one scalar multiply per request instead of a 64-bit product.
        float ybuf[kEsAhead][CH];
        const unsigned ycol = in_batch ? ub : 0u;
        auto load_chunk = [&](int c, float *dst) {
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                // raw value of a wave-uniform row (the last row again past the end); the step replaces what
                // lies past the series' length
                const unsigned t = (unsigned)min(c * CH + k, a.T - 1);
                dst[k] = a.y[t * (unsigned)a.B + ycol];
            }
        };
        static_for<0, kEsAhead>([&](auto d) { load_chunk(decltype(d)::value, ybuf[decltype(d)::value]); });
        rotate_while<kEsAhead>([&](auto dd, int c) {
            constexpr int d = decltype(dd)::value;
            if (c >= n_chunks) return false;                // (wave-uniform)
            float *out = stage + (c & 1) * (CH * NF * 64);
#pragma unroll
            for (int k = 0; k < CH; k += CS) {
                // (wave-uniform; a group of one step never wraps)
                const bool wraps = CS > 1 && ((NS >= 1 && i1 + CS > a.m1) || (NS >= 2 && i2 + CS > a.m2));
                if (wraps) steps(std::true_type{}, c * CH + k, ybuf[d] + k, out + k * NF * 64);
                else steps(std::false_type{}, c * CH + k, ybuf[d] + k, out + k * NF * 64);
            }
            load_chunk(c + kEsAhead, ybuf[d]);
            // chunk c is staged; the other waves have finished with chunk c - 1, whose buffer chunk
            // c + 1 reuses
            lds_barrier();
            return true;
        });
        return;
    }

    // ---- the other waves: chunk c after the barrier that publishes it, the staged values of a whole chunk read together
    if (role == 1) {                            // Section 8.4: squared second difference of the log level
        float u1 = 0.0f, u2 = 0.0f, lv_sum = 0.0f;
        for (int c = 0; c < n_chunks; ++c) {
            lds_barrier();
            const float *in = stage + (c & 1) * (CH * NF * 64) + lane;
            float lt[CH];
#pragma unroll
            for (int k = 0; k < CH; ++k) lt[k] = in[k * NF * 64];
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int t = c * CH + k;
                const float ut = fast_log(lt[k]), e = ut - 2.0f * u1 + u2;
                lv_sum += t < len && t >= 2 ? e * e : 0.0f;
                u2 = u1; u1 = ut;
            }
        }
        const float tot = wave_sum(lv_sum);
        if (lane == 0) a.lv_partial[blockIdx.x] = tot;
        return;
    }
    const ChunkRows rows(a.Bp, t_end, len);
    for (int c = 0; c < n_chunks; ++c) {
        lds_barrier();
        const float *in = stage + (c & 1) * (CH * NF * 64);
#pragma unroll
        for (int k0 = 0; k0 < CH; k0 += 4) {
            const int t = c * CH + k0 + rows.row;
            auto staged = [&](int f) { return rows.quad(in + (k0 * NF + f) * 64, NF * 64); };
            if (role == 2) {
                const f32x4 l = staged(0);
                rows.put(a.lvl, t, l, 1.0f);
                rows.put(a.u, t, rows.logs(l), 0.0f);
                rows.put(a.v, t, rows.logs(staged(1)), 0.0f);              // ln y - ln(S1 S2)
            } else {
                if constexpr (NS >= 1) rows.put(a.S1, t, staged(2), 1.0f);
                if constexpr (NS >= 2) rows.put(a.S2, t, staged(3), 1.0f);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The same recursions for long periods and few series.  With factors that were produced three chunks of steps ago or
// earlier, only the level is a chain: per step one multiply-add.  Three stages, a chunk each, run side by side on waves of
// their own, one barrier per chunk:
//   A (two waves)  de-seasonalised values q and what they add to the level, from the factors in the rings;
//   B (one wave)   the level;
//   C (two waves)  the new factors, from the level, into the rings; beside it a wave for the level penalty and two that
//                  store what A and B have left of the chunk.
// Interval j runs A on chunk j, B on chunk j - 1, C and the stores on chunk j - 2.  A reads factors that C has left at
// least one barrier earlier, and touches none that C is writing, if no period is shorter than three chunks.
// 512 hourly series: 77 -> 50 us (333 for a forecast: 76 -> 47 us).  An interval takes 0.47 us; B alone takes 0.13, A or C
// alone 0.33; four waves each for A and C: no change.
// ---------------------------------------------------------------------------
constexpr int kEsLongChunk = 8, kEsLongShares = 2, kEsLongAhead = 8, kEsLongSlots = 4;      // shares: waves of A, and of C
constexpr int kEsLongWaves = 4 + 2 * kEsLongShares;
constexpr int es_long_fields(int n_seas) { return 4 + n_seas; }     // add, q, y, level, factors
constexpr int es_long_stage_floats(int n_seas) { return kEsLongSlots * kEsLongChunk * es_long_fields(n_seas) * 64; }

template <int NS>
__global__ void __launch_bounds__(64 * kEsLongWaves) es_forward_long_kernel(EsArgs a, SetupArgs setup)
{
    extern __shared__ __align__(16) float ring[];   // [m1 + m2][64] rings, then [slot][CH][fields][64]
    constexpr int CH = kEsLongChunk;
    static_assert(NS >= 1 && CH % 4 == 0, "waves share a chunk, and store four steps at a time");
    constexpr int NF = es_long_fields(NS), SHARES = kEsLongShares, PER = CH / SHARES, AHEAD = kEsLongAhead;
    if ((int)blockIdx.x >= a.blocks) {
        if (threadIdx.x < 256) setup_body(setup, blockIdx.x - a.blocks, ring);
        return;
    }
    const int role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int b = blockIdx.x * 64 + lane;
    const bool in_batch = b < a.B;
    const int len = in_batch ? a.lengths.at(b) : 0;
    float *ring1 = ring + lane, *ring2 = ring + (size_t)a.m1 * 64 + lane;
    float *stage = ring + (size_t)(a.m1 + a.m2) * 64 + lane;
    auto field = [&](int c, int k, int f) -> float & { return stage[(((c & (kEsLongSlots - 1)) * CH + k) * NF + f) * 64]; };
    enum { kAdd, kQ, kY, kLevel, kS1, kS2 };
    const int t_end = wave_max_int(len);            // (the same in all waves)
    const int n = (t_end + CH - 1) / CH;
    // Whole rounds of A's request buffers: behind any condition the wait for the observations would cover the newest request.
    // (The last intervals of A stage chunks that nobody takes.)
    const int intervals = (n + 2 + AHEAD - 1) / AHEAD * AHEAD;
    // Chunks in which every series goes on (and not the first one) need no choice per step.
    const int t_all = -wave_max_int(-len);
    auto by_chunk = [&](int c, auto &&f) {
        if (c > 0 && (c + 1) * CH <= t_all) f(std::true_type{});
        else f(std::false_type{});
    };
    const unsigned ub = b;
    {
        const int rows = a.m1 + a.m2;
        for (int k0 = role * 8; k0 < rows; k0 += kEsLongWaves * 8) {
            float sv[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = min(k0 + j, rows - 1);
                const int row = k < a.m1 ? a.row_s1 + k : a.row_s2 + (k - a.m1);
                sv[j] = in_batch ? a.es[(size_t)row * a.B + b] : 1.0f;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (k0 + j < rows) ring[(k0 + j) * 64 + lane] = (a.logit && in_batch) ? expf(sv[j]) : sv[j];
        }
    }
    auto parameter = [&](int row) {
        float v = in_batch ? a.es[(size_t)row * a.B + b] : 0.0f;
        if (a.logit) v = 1.0f / (1.0f + expf(-v));
        return v;
    };
    __syncthreads();
    auto wrapped = [](int i, int m) { return i < m ? i : i - m; };
    // f(k, slot) for PER consecutive slots of a ring of m from slot i on (no period is shorter than a chunk): one base and
    // constant offsets unless the ring ends among them
    auto factors = [&](float *at, int i, int m, auto &&f) {
        if (i + PER <= m) {
            float *first = at + i * 64;
#pragma unroll
            for (int k = 0; k < PER; ++k) f(k, first[k * 64]);
        } else {
#pragma unroll
            for (int k = 0; k < PER; ++k) f(k, at[wrapped(i + k, m) * 64]);
        }
    };

    if (role == 0) {                                // ---- B
        const float keep = in_batch ? 1.0f - parameter(0) : 0.5f;
        float level = 1.0f;
        for (int j = 0; j < intervals; ++j) {
            const int c = j - 1;
            if (c >= 0 && c < n) {
                float add[CH];
#pragma unroll
                for (int k = 0; k < CH; ++k) add[k] = field(c, k, kAdd);
                by_chunk(c, [&](auto whole) {
#pragma unroll
                    for (int k = 0; k < CH; ++k) {
                        const int t = c * CH + k;
                        // reading for the state before the first observation: l_0 = y_0 / S[0]; past the end the level stays
                        const float f = decltype(whole)::value ? keep : t == 0 ? 0.0f : t < len ? keep : 1.0f;
                        level = f * level + add[k];
                        field(c, k, kLevel) = level;
                    }
                });
            }
            lds_barrier();
        }
    } else if (role <= SHARES) {                    // ---- A
        const float alpha = in_batch ? parameter(0) : 0.5f;
        const unsigned ycol = 4u * (in_batch ? ub : 0u), stride = 4u * a.B;
        auto run = [&](auto hc) {
            constexpr int h = decltype(hc)::value;  // this wave's steps of a chunk: h .. h + PER - 1
            float y[AHEAD][PER];
            auto request = [&](int c, float (&v)[PER]) {
                // (rows past the last one: the last one again)
                const int t0 = min(c * CH + h, a.T - 1), rest = a.T - 1 - t0;
                const buf_rsrc rows = make_rsrc(a.y + (size_t)t0 * a.B);
#pragma unroll
                for (int k = 0; k < PER; ++k) v[k] = buf_load(rows, ycol, min(k, rest) * stride);
            };
            static_for<0, AHEAD>([&](auto d) { request(decltype(d)::value, y[decltype(d)::value]); });
            int i1 = h, i2 = h;
            for (int j0 = 0; j0 < intervals; j0 += AHEAD) {
                static_for<0, AHEAD>([&](auto dc) {
                    constexpr int d = decltype(dc)::value;
                    const int c = j0 + d;
                    float s1[PER], s2[PER];
                    factors(ring1, i1, a.m1, [&](int k, float &at) { s1[k] = at; });
                    if constexpr (NS >= 2) factors(ring2, i2, a.m2, [&](int k, float &at) { s2[k] = at; });
                    by_chunk(c, [&](auto whole) {
                        constexpr bool W = decltype(whole)::value;
#pragma unroll
                        for (int k = 0; k < PER; ++k) {
                            const int t = c * CH + h + k;
                            const float yt = W || t < len ? y[d][k] : 1.0f;     // (levels and factors stay finite)
                            const float q = yt * fast_rcp(NS >= 2 ? s1[k] * s2[k] : s1[k]);
                            field(c, h + k, kAdd) = !W && t == 0 ? q : W || t < len ? alpha * q : 0.0f;
                            field(c, h + k, kQ) = q;
                            field(c, h + k, kY) = yt;
                            field(c, h + k, kS1) = s1[k];
                            if constexpr (NS >= 2) field(c, h + k, kS2) = s2[k];
                        }
                    });
                    i1 = wrapped(i1 + CH, a.m1);
                    if constexpr (NS >= 2) i2 = wrapped(i2 + CH, a.m2);
                    request(c + AHEAD, y[d]);
                    lds_barrier();
                });
            }
        };
        static_for<0, SHARES>([&](auto sc) {
            if (role == 1 + decltype(sc)::value) run(std::integral_constant<int, PER * decltype(sc)::value>{});
        });
    } else if (role <= 2 * SHARES) {                // ---- C
        const float g1 = parameter(a.row_gamma1), g2 = NS >= 2 ? parameter(a.row_gamma2) : 0.0f;
        auto run = [&](auto hc) {
            constexpr int h = decltype(hc)::value;
            int i1 = h, i2 = h;
            for (int j = 0; j < intervals; ++j) {
                const int c = j - 2;
                if (c >= 0 && c < n) {
                    float before[PER], y[PER], s1[PER], s2[PER], w1[PER], w2[PER];
#pragma unroll
                    for (int k = 0; k < PER; ++k) {
                        constexpr int last = CH - 1;
                        before[k] = h + k > 0 ? field(c, h + k > 0 ? h + k - 1 : 0, kLevel) : field(c + kEsLongSlots - 1, last, kLevel);
                        y[k] = field(c, h + k, kY);
                        s1[k] = field(c, h + k, kS1);
                        s2[k] = NS >= 2 ? field(c, h + k, kS2) : 1.0f;
                    }
#pragma unroll
                    for (int k = 0; k < PER; ++k) {
                        // Eq. (3): divide by the previous level (and the other factor); at t = 0 the produced factor
                        // equals the initial one
                        const bool first = h + k == 0 && c == 0;
                        const float ry = y[k] * fast_rcp(before[k]), r12 = NS >= 2 ? fast_rcp(s1[k] * s2[k]) : 1.0f;
                        w1[k] = g1 * ry * (NS >= 2 ? r12 * s1[k] : 1.0f) + (1.0f - g1) * s1[k];
                        w2[k] = g2 * ry * (r12 * s2[k]) + (1.0f - g2) * s2[k];
                        if (first) { w1[k] = s1[k]; w2[k] = s2[k]; }
                    }
                    factors(ring1, i1, a.m1, [&](int k, float &at) { at = w1[k]; });
                    if constexpr (NS >= 2) factors(ring2, i2, a.m2, [&](int k, float &at) { at = w2[k]; });
                    i1 = wrapped(i1 + CH, a.m1);
                    if constexpr (NS >= 2) i2 = wrapped(i2 + CH, a.m2);
                }
                lds_barrier();
            }
        };
        static_for<0, SHARES>([&](auto sc) {
            if (role == 1 + SHARES + decltype(sc)::value) run(std::integral_constant<int, PER * decltype(sc)::value>{});
        });
    } else if (role == 2 * SHARES + 1) {            // ---- level penalty: squared second difference of the log level (Section 8.4)
        float u1 = 0.0f, u2 = 0.0f, lv_sum = 0.0f;
        for (int j = 0; j < intervals; ++j) {
            const int c = j - 2;
            if (c >= 0 && c < n) {
                float l[CH];
#pragma unroll
                for (int k = 0; k < CH; ++k) l[k] = field(c, k, kLevel);
#pragma unroll
                for (int k = 0; k < CH; ++k) {
                    const int t = c * CH + k;
                    const float ut = fast_log(l[k]), e = ut - 2.0f * u1 + u2;
                    lv_sum += t < len && t >= 2 ? e * e : 0.0f;
                    u2 = u1; u1 = ut;
                }
            }
            lds_barrier();
        }
        const float tot = wave_sum(lv_sum);
        if (lane == 0) a.lv_partial[blockIdx.x] = tot;
    } else {                                        // ---- stores
        const ChunkRows rows(a.Bp, t_end, len);
        for (int j = 0; j < intervals; ++j) {
            const int c = j - 2;
            if (c >= 0 && c < n) {
#pragma unroll
                for (int k0 = 0; k0 < CH; k0 += 4) {
                    const int t = c * CH + k0 + rows.row;
                    auto staged = [&](int f) { return rows.quad(&field(c, k0, f) - lane, NF * 64); };
                    if (role == 2 * SHARES + 2) {
                        const f32x4 l = staged(kLevel);
                        rows.put(a.lvl, t, l, 1.0f);
                        rows.put(a.u, t, rows.logs(l), 0.0f);
                    } else {
                        rows.put(a.v, t, rows.logs(staged(kQ)), 0.0f);              // ln y - ln(S1 S2)
                        rows.put(a.S1, t, staged(kS1), 1.0f);
                        if constexpr (NS >= 2) rows.put(a.S2, t, staged(kS2), 1.0f);
                    }
                }
            }
            lds_barrier();
        }
    }
}

// ---------------------------------------------------------------------------
// Windows, Section 5.3 and Eq. (6): with u = ln(level), v = ln y - ln(seasonal
// factors), input x[p][i] = v[p+i] - u[t], target z[p][j] = v[t+j] - u[t],
// t = p + I - 1.  One wave writes one (p, 16-series) tile; every store
// instruction covers 4 rows x 16 series = 256 contiguous bytes.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) window_forward_kernel(const float *__restrict__ u, const float *__restrict__ v,
                                                              float *__restrict__ X, float *__restrict__ Z,
                                                              int P, int NB, int Bp, int I, int H, int xrows, int zrows,
                                                              int p_per_wave, const int32_t *__restrict__ categories,
                                                              int n_cat, int B, const int32_t *__restrict__ pmax)
{
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4, n = lane & 15;
    // the four waves of a workgroup take four adjacent series tiles at the same positions, so that the
    // workgroup writes 1 KB (X, I = 4) and 2 KB (Z, H = 8) contiguous per position
    const int bt = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (bt >= NB) return;
    const int p0 = blockIdx.y * p_per_wave;
    const int col = bt * 16 + n;
    // Section 5.3: the one-hot block of the series' category follows the window (rows I .. I+n_cat-1)
    const int hot = (n_cat > 0 && col < B) ? I + categories[col] : -1;
    const int Pt = min(P, pmax[bt]);     // windows past the tile's longest series are not needed by any later kernel
    for (int p = p0; p < p0 + p_per_wave && p < Pt; ++p) {
        const size_t tile = (size_t)p * NB + bt;
        const int t = p + I - 1;
        const float ut = u[(size_t)t * Bp + col];
        float *xo = X + tile * xrows * 16 + lane;
        // streaming stores: the tiles are consumed by later kernels, not by this one
        for (int r = g; r < xrows; r += 4)
            __builtin_nontemporal_store((r < I) ? v[(size_t)(p + r) * Bp + col] - ut : (r == hot ? 1.0f : 0.0f),
                                        xo + (r - g) * 16);
        float *zo = Z + tile * zrows * 16 + lane;
        for (int r = g; r < zrows; r += 4)
            __builtin_nontemporal_store((r < H) ? v[(size_t)(t + 1 + r) * Bp + col] - ut : 0.0f, zo + (r - g) * 16);
    }
}

// Gradient of the level penalty (Section 8.4) with respect to u[t] of one series, times `scale`:
// e[k] = u[k] - 2u[k-1] + u[k-2] for 2 <= k < len; d/du[t] of sum e^2 = 2(e[t] - 2e[t+1] + e[t+2]).
__device__ __forceinline__ float level_penalty_grad(const float *__restrict__ u, int Bp, int col, int t, int len, float scale)
{
    float acc = 0.0f;
#pragma unroll
    for (int dk = 0; dk <= 2; ++dk) {
        const int k = t + dk;
        if (k >= 2 && k < len) {
            const float e = u[(size_t)k * Bp + col] - 2.0f * u[(size_t)(k - 1) * Bp + col] + u[(size_t)(k - 2) * Bp + col];
            acc += (dk == 1 ? -2.0f : 1.0f) * e;
        }
    }
    return scale * acc;
}

// ---------------------------------------------------------------------------
// Weight-gradient reduction: sums the per-workgroup partial tiles in a fixed order and writes the caller's packing.
// ---------------------------------------------------------------------------
// Stage 1: every job (one block of partial results per producer
// workgroup) is cut into `splits` interleaved subsets of the producers; a thread sums
// one element over one subset.  Stage 2 (the kernels below) sums the subsets and
// writes the caller's packing.  Both orders are fixed.
//
// Neither stage has anything to do with the smoothing part of the reverse pass: the first is in the launch of the window
// adjoint, the second in that of the recursions' adjoint, whose few workgroups are one long chain (as launches of their
// own: 19 + 5 us at 4096 quarterly series, 5 + 4.6 us at 16).
struct ReduceJob {
    const float *src;
    float *dst;          // [splits][n_elems]
    unsigned stride;     // floats between consecutive partial blocks
    int n_part, n_elems, splits;
    int end;             // workgroups of this job and those before it
};
constexpr int kMaxReduceJobs = 2 * kMaxLayers + 1;
struct ReduceJobs {
    ReduceJob job[kMaxReduceJobs];
    int blocks;          // 0: nothing to reduce
};

__device__ __forceinline__ void reduce_stage1_body(const ReduceJobs &jobs, int block)
{
    int i = 0;
    while (block >= jobs.job[i].end) ++i;
    const ReduceJob &j = jobs.job[i];
    if (i > 0) block -= jobs.job[i - 1].end;
    const int chunks = (j.n_elems + 255) / 256;
    const int e = block % chunks * 256 + threadIdx.x, sp = block / chunks;
    if (e >= j.n_elems) return;
    const float *src = j.src + e;
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
    int w = sp;
    for (; w + 3 * j.splits < j.n_part; w += 4 * j.splits) {
        a0 += src[(size_t)w * j.stride];
        a1 += src[(size_t)(w + j.splits) * j.stride];
        a2 += src[(size_t)(w + 2 * j.splits) * j.stride];
        a3 += src[(size_t)(w + 3 * j.splits) * j.stride];
    }
    for (; w < j.n_part; w += j.splits) a0 += src[(size_t)w * j.stride];
    j.dst[(size_t)sp * j.n_elems + e] = (a0 + a1) + (a2 + a3);
}

struct ReduceLstmArgs {
    const float *dw_partial, *db_partial;
    float *gW, *gb;
    int NB, h, in_dim, HT, KXT;
};

// Sums `n_part` partial blocks for 64 consecutive elements per workgroup: the
// four waves take interleaved quarters of the partials (each load instruction
// reads 256 contiguous bytes of one partial), then combine in a fixed order.
__device__ __forceinline__ float reduce_partials(const float *__restrict__ base, size_t stride, int n_part, int elem,
                                                 bool active, float (*s_red)[64])
{
    const int e = threadIdx.x & 63, sl = threadIdx.x >> 6;
    float acc = 0.0f;
    if (active) {
        const float *src = base + elem;
        int w = sl;
        for (; w + 12 < n_part; w += 16) {
            const float a0 = src[(size_t)w * stride], a1 = src[(size_t)(w + 4) * stride];
            const float a2 = src[(size_t)(w + 8) * stride], a3 = src[(size_t)(w + 12) * stride];
            acc += (a0 + a1) + (a2 + a3);
        }
        for (; w < n_part; w += 4) acc += src[(size_t)w * stride];
    }
    s_red[sl][e] = acc;
    __syncthreads();
    return (s_red[0][e] + s_red[1][e]) + (s_red[2][e] + s_red[3][e]);
}

__device__ __forceinline__ void reduce_lstm_body(const ReduceLstmArgs &a, int block, float (*s_red)[64])
{
    const int KT = a.KXT + a.HT, MB = (KT + 3) / 4, ld = a.in_dim + a.h;
    const int n_dw = a.HT * MB * 256, n_db = a.HT * 16;
    const int n_dw_blocks = (n_dw + 63) / 64;
    const int e = threadIdx.x & 63;
    if (block < n_dw_blocks) {
        const int idx = block * 64 + e;                  // element of the tile block: [tile][component][lane]
        const float tot = reduce_partials(a.dw_partial, (size_t)n_dw, a.NB, idx, idx < n_dw, s_red);
        if (threadIdx.x < 64 && idx < n_dw) {
            const int lane = idx & 63, comp = (idx >> 6) & 3, tix = idx >> 8;
            const int mt = tix / MB, nbk = tix % MB;
            // tile row 4*gate + unit-in-tile sits in lane group `gate`, component `unit-in-tile`
            const int gate = lane >> 4, unit = 4 * mt + comp;
            const int xr = 16 * nbk + (lane & 15);
            int col = -1;
            if (xr < 4 * a.KXT) { if (xr < a.in_dim) col = xr; }
            else if (xr - 4 * a.KXT < a.h) col = a.in_dim + xr - 4 * a.KXT;
            if (unit < a.h && col >= 0) a.gW[(size_t)(gate * a.h + unit) * ld + col] = tot;
        }
    } else {
        const int idx = (block - n_dw_blocks) * 64 + e;   // [unit tile][unit][gate]
        const float tot = reduce_partials(a.db_partial, (size_t)n_db, a.NB, idx, idx < n_db, s_red);
        if (threadIdx.x < 64 && idx < n_db) {
            const int gate = idx & 3, unit = idx >> 2;
            if (unit < a.h) a.gb[gate * a.h + unit] = tot;
        }
    }
}

struct ReduceHeadArgs {
    const float *partial;
    float *gWa, *gba, *gWo, *gbo;
    int n_part, stride, h, H, HT, MA, MO, OT;
};

__device__ __forceinline__ void reduce_head_body(const ReduceHeadArgs &a, int block, float (*s_red)[64])
{
    // partial block: dWo tiles [MO*MA][4][64], dWa tiles [MA*MA][4][64], dbo [4*OT], dba [4*HT]
    const int offWa = a.MO * a.MA * 256, offbo = offWa + a.MA * a.MA * 256, offba = offbo + 4 * a.OT;
    const int n = offba + 4 * a.HT;
    const int idx = block * 64 + (threadIdx.x & 63);
    const float tot = reduce_partials(a.partial, (size_t)a.stride, a.n_part, idx, idx < n, s_red);
    if (threadIdx.x >= 64 || idx >= n) return;
    if (idx < offbo) {
        const bool isWa = idx >= offWa;
        const int j = isWa ? idx - offWa : idx;
        const int lane = j & 63, comp = (j >> 6) & 3, tix = j >> 8;
        const int mt = tix / a.MA, nt = tix % a.MA;
        // (rows and columns of a tile in unit-tile order)
        const int row = 4 * (4 * mt + comp) + (lane >> 4), col = 4 * (4 * nt + (lane & 3)) + ((lane & 15) >> 2);
        if (col < a.h) {
            if (isWa) { if (row < a.h) a.gWa[row * a.h + col] = tot; }
            else if (row < a.H) a.gWo[row * a.h + col] = tot;
        }
    } else if (idx < offba) {
        const int j = idx - offbo;
        if (j < a.H) a.gbo[j] = tot;
    } else {
        const int j = idx - offba;
        if (j < a.h) a.gba[j] = tot;
    }
}

struct ReduceStage2Args {
    ReduceLstmArgs lstm[kMaxLayers];
    ReduceHeadArgs head;
    int end[kMaxLayers + 1];    // workgroups of this layer (the last one: of the output stage) and those before it
    int L;
    TogetherWords words;        // of the reverse pass, for the next one
    int blocks() const { return end[kMaxLayers]; }      // 0: nothing to reduce
};

__device__ __forceinline__ void reduce_stage2_body(const ReduceStage2Args &a, int block, float *scratch)
{
    float (*s_red)[64] = reinterpret_cast<float (*)[64]>(scratch);
    if (block == 0) clear_words(a.words, kWordStride);
    int z = 0;
    while (z < a.L && block >= a.end[z]) ++z;
    if (z > 0) block -= a.end[z - 1];
    if (z < a.L) reduce_lstm_body(a.lstm[z], block, s_red);
    else reduce_head_body(a.head, block, s_red);
}

// ---------------------------------------------------------------------------
// Window adjoint in gather form (no atomics): every x and z is v[.] - u[t], so
//   gv[k] = sum_i gX[k-i][i] + sum_j gZ[k-(I-1)-j][j],  gu[t] = -(sum of row p = t-I+1),
// with gZ = -gO, plus the gradient of the level penalty (Section 8.4).
// One thread per (t, series); a workgroup takes 64 series at four consecutive t.
//
// Every 128-byte line of gX / gO holds two rows of a tile and is read for two neighbouring t and once
// more for the row sum, by different workgroups.  The workgroups that touch the tiles of one group of 64
// series therefore all run on the same XCD (workgroups go to the XCDs in turn), one after the other in
// time order: the line is then fetched from memory once and found in that XCD's L2 afterwards.
// ---------------------------------------------------------------------------
struct WindowBwdArgs {
    const float *gX, *gO, *u;
    const int32_t *lengths;
    const Scalars *sc;
    float lambda;
    float *gu, *gv;
    int P, NB, B, Bp, T, I, H, xrows, zrows;    // Bp: row stride of the time-major arrays (the batch padded to 64)
    const int32_t *pmax;
    int t_chunks;        // gather: groups of four time steps
    int R;               // streaming: slots of the ring
    int blocks;          // workgroups of the window adjoint; the launch's others reduce weight gradients
};

__global__ void __launch_bounds__(256) window_backward_kernel(WindowBwdArgs a, ReduceJobs jobs)
{
    if ((int)blockIdx.x >= a.blocks) {
        reduce_stage1_body(jobs, blockIdx.x - a.blocks);
        return;
    }
    const float *__restrict__ gX = a.gX, *__restrict__ gO = a.gO;
    const int NB = a.NB, Bp = a.Bp, T = a.T, I = a.I, H = a.H, xrows = a.xrows, zrows = a.zrows;
    // (columns past the 16 * NB series of the tiles have no windows)
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int cg = (slot / a.t_chunks) * 8 + xcd;               // group of 64 series
    const int t = (slot % a.t_chunks) * 4 + (threadIdx.x >> 6);
    if (cg * 64 >= Bp || t >= T) return;
    const int col = cg * 64 + (threadIdx.x & 63);
    const size_t idx = (size_t)t * Bp + col;
    if (col >= 16 * NB) {
        a.gu[idx] = 0.0f;
        a.gv[idx] = 0.0f;
        return;
    }
    const int bt = col >> 4, n = col & 15;
    const int P = min(a.P, a.pmax[bt]);      // window gradients past the tile's longest series do not exist
    float sv = 0.0f, su = 0.0f;
    // Eight independent requests at a time, in range by choice of address, not behind a condition each.  (One after the
    // other, a thread was a chain of 2 (I + H) round trips.)
    auto sum8 = [&](int rows, auto &&at, auto &&counts) {
        float total = 0.0f;
        for (int r0 = 0; r0 < rows; r0 += 8) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = at(min(r0 + k, rows - 1));
#pragma unroll
            for (int k = 0; k < 8; ++k) total += r0 + k < rows && counts(r0 + k) ? v[k] : 0.0f;
        }
        return total;
    };
    if (P > 0) {
        const int last = P - 1, p_u = t - I + 1, p_row = min(max(p_u, 0), last);
        sv = sum8(I, [&](int i) { return gX[((size_t)(min(max(t - i, 0), last) * NB + bt) * xrows + i) * 16 + n]; },
                  [&](int i) { return t - i >= 0 && t - i <= last; }) -
             sum8(H, [&](int j) { return gO[((size_t)(min(max(t - I - j, 0), last) * NB + bt) * zrows + j) * 16 + n]; },
                  [&](int j) { return t - I - j >= 0 && t - I - j <= last; });
        if (p_u >= 0 && p_u <= last)
            su = sum8(H, [&](int j) { return gO[((size_t)(p_row * NB + bt) * zrows + j) * 16 + n]; }, [](int) { return true; }) -
                 sum8(I, [&](int i) { return gX[((size_t)(p_row * NB + bt) * xrows + i) * 16 + n]; }, [](int) { return true; });
    }
    if (a.lambda != 0.0f)
        su += level_penalty_grad(a.u, Bp, col, t, col < a.B ? clamp_len(a.lengths[col], T) : 0, a.lambda * 2.0f * a.sc->inv_n_lv);
    a.gu[idx] = su;
    a.gv[idx] = sv;
}

// ---------------------------------------------------------------------------
// Window adjoint in streaming form, for batches with many series tiles.  One wave owns a series tile and
// walks over the positions in time order.  Every row group of gX and gO (four rows of 16 series, 256
// contiguous bytes) is loaded exactly once, by one full-width instruction; lane (g, n) adds its element of
// row c of position p to slot (p + c) mod R of a ring of R >= I + H + 4 anti-diagonal sums in LDS (plain read, add,
// write: the lanes of one instruction hit different slots, and the LDS unit serves a wave's instructions in
// order, so no atomic is needed and the sums are formed in a fixed order).  After a block of four positions the four oldest slots are complete:
// lane group g writes gv[s + g] and clears its slot, and writes gu[s + g + I - 1] from the row sum of its
// position.  The gather kernel above reads every element twice in 64-byte pieces; this one is the faster
// of the two once there are enough tiles for the waves to hide each other's memory latency.
// ---------------------------------------------------------------------------
// NQ: row groups that hold window elements (0: any number, one block at a time, nothing requested ahead).
template <int NQ>
__global__ void __launch_bounds__(256, NQ > 0 ? 4 : 1) window_backward_stream_kernel(WindowBwdArgs a, ReduceJobs jobs)
{
    if ((int)blockIdx.x >= a.blocks) {
        reduce_stage1_body(jobs, blockIdx.x - a.blocks);
        return;
    }
    const float *__restrict__ gX = a.gX, *__restrict__ gO = a.gO;
    const float lambda = a.lambda;
    const int NB = a.NB, Bp = a.Bp, T = a.T, I = a.I, H = a.H, xrows = a.xrows, zrows = a.zrows, R = a.R;
    extern __shared__ float ring_all[];                     // [wave][R][16]
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int g = lane >> 4, n = lane & 15;
    const int bt = blockIdx.x * 4 + wave;
    if (bt >= NB) return;                                   // (no workgroup barrier below)
    float *ring = ring_all + wave * R * 16;
    for (int e = lane; e < R * 16; e += 64) ring[e] = 0.0f;
    const int mask = R - 1;
    const int Pt = min(a.P, a.pmax[bt]);
    const int col = bt * 16 + n;
    const int len = col < a.B ? clamp_len(a.lengths[col], T) : 0;
    const float pen = lambda * 2.0f * a.sc->inv_n_lv;
    const int QX = (I + 3) >> 2, Q = QX + ((H + 3) >> 2);   // row groups that hold window elements
    // columns between the last tile and the padded batch: the wave of the last tile clears them
    const int pad_col = 16 * NB + lane;
    const bool pads = bt == NB - 1 && 16 * NB < Bp;         // (wave-uniform)

    // Blocks whose four positions exist and whose outputs are all in range: the next block's requests travel while this one's are added
    // up.  Straight runs without conditions around requests and stores, two blocks each (a block's registers are the next one's otherwise,
    // and a copy waits).  65 536 quarterly series: 75 -> 57 us, 230 MB at 4.0 TB/s.
    auto streamed = [&]() {
        constexpr int N = NQ > 0 ? NQ : 1;
        struct Request { float w[4][N], u[5]; };
        auto request = [&](int s0, Request &q) {
            const int p0 = min(s0, (Pt & ~3) - 4);                      // (past the last block: that one again)
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                const int t = p0 + g + I - 3 + k;
                q.u[k] = a.u[(size_t)min(max(t, 0), T - 1) * Bp + col];
            }
#pragma unroll
            for (int sp = 0; sp < 4; ++sp) {
                const size_t tile = (size_t)(p0 + sp) * NB + bt;
#pragma unroll
                for (int e = 0; e < N; ++e) q.w[sp][e] = (e < QX ? gX + (tile * xrows + 4 * e) * 16 : gO + (tile * zrows + 4 * (e - QX)) * 16)[lane];
            }
        };
        auto block = [&](int s0, const Request &q) {
            float mine = 0.0f;
#pragma unroll
            for (int sp = 0; sp < 4; ++sp) {
                float su = 0.0f;
                bool ok[N];
                int at[N];
                float val[N], old[N];
#pragma unroll
                for (int e = 0; e < N; ++e) {
                    const bool is_x = e < QX;
                    const int r = 4 * (is_x ? e : e - QX) + g;
                    ok[e] = r < (is_x ? I : H);
                    // (the address of a row that does not count, which is not accessed: that of the window's first one)
                    at[e] = ((s0 + sp + (ok[e] ? (is_x ? r : I + r) : 0)) & mask) * 16 + n;
                    val[e] = is_x ? q.w[sp][e] : -q.w[sp][e];
                }
#pragma unroll
                for (int e = 0; e < N; ++e)
                    if (ok[e]) old[e] = ring[at[e]];
#pragma unroll
                for (int e = 0; e < N; ++e)
                    if (ok[e]) {
                        ring[at[e]] = old[e] + val[e];
                        su -= val[e];
                    }
                su += __shfl_xor(su, 16, 64);
                su += __shfl_xor(su, 32, 64);
                mine = g == sp ? su : mine;
            }
            const int s = s0 + g, t = s + I - 1;
            float acc = 0.0f;
#pragma unroll
            for (int dk = 0; dk <= 2; ++dk) {
                const float e = q.u[dk + 2] - 2.0f * q.u[dk + 1] + q.u[dk];
                acc += t + dk >= 2 && t + dk < len ? (dk == 1 ? -2.0f : 1.0f) * e : 0.0f;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            float *slot = &ring[(s & mask) * 16 + n];
            a.gv[(size_t)s * Bp + col] = *slot;
            *slot = 0.0f;
            a.gu[(size_t)t * Bp + col] = mine + (lambda != 0.0f ? pen * acc : 0.0f);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        };
        Request q0, q1;
        const int blocks = Pt >> 2;
        request(0, q0);
        int s0 = 0;
        if (int pairs = blocks >> 1) do {
            request(s0 + 4, q1);
            __builtin_amdgcn_sched_barrier(0);
            block(s0, q0);
            request(s0 + 8, q0);
            __builtin_amdgcn_sched_barrier(0);
            block(s0 + 4, q1);
            s0 += 8;
        } while (--pairs);
        if (blocks & 1) block(s0, q0);
    };

    for (int s0 = -((I + 2) & ~3); s0 < T; s0 += 4) {      // output block: gv[s0 .. s0+3], gu[s0+I-1 .. s0+I+2]
        if constexpr (NQ > 0)
            if (s0 == 0 && Pt >= 4) {
                streamed();
                if (pads && pad_col < Bp)
                    for (int s = 0; s < (Pt & ~3); ++s) {
                        a.gv[(size_t)s * Bp + pad_col] = 0.0f;
                        a.gu[(size_t)(s + I - 1) * Bp + pad_col] = 0.0f;
                    }
                s0 = Pt & ~3;
                if (s0 >= T) break;
            }
        float su[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        // the penalty term of this lane's gu row, requested ahead of the gradient tiles: its five loads then
        // travel together with theirs instead of being a second round trip at the end of the block
        const int t_pen = s0 + g + I - 1;
        const float pen_grad = (lambda != 0.0f && t_pen >= 0 && t_pen < T) ? level_penalty_grad(a.u, Bp, col, t_pen, len, pen) : 0.0f;
        if (s0 + 3 >= 0 && s0 < Pt) {
            for (int e0 = 0; e0 < Q; e0 += 4) {
                float w[4][4];
                // sixteen independent loads in flight, then sixteen LDS additions
#pragma unroll
                for (int sp = 0; sp < 4; ++sp) {
                    const int p = min(max(s0 + sp, 0), Pt - 1);
                    const size_t tile = (size_t)p * NB + bt;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int e = min(e0 + j, Q - 1);
                        const float *src = e < QX ? gX + (tile * xrows + 4 * e) * 16 : gO + (tile * zrows + 4 * (e - QX)) * 16;
                        w[sp][j] = src[lane];
                    }
                }
#pragma unroll
                for (int sp = 0; sp < 4; ++sp) {
                    const int p = s0 + sp;
                    if (p < 0 || p >= Pt) continue;                     // (wave-uniform)
                    // The row groups of one position go to different slots in every lane (row c of the window
                    // part is below I, row c of the horizon part is I or more), so their four read-add-write
                    // sequences are independent: all reads, then all writes.  Two positions do share slots.
                    bool ok[4];
                    int at[4];
                    float val[4], old[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int e = e0 + j;
                        const bool is_x = e < QX;
                        const int r = 4 * (is_x ? e : e - QX) + g;
                        // gX rows past the window (categories, padding) and gO rows past the horizon do not count
                        ok[j] = e < Q && r < (is_x ? I : H);
                        at[j] = ((p + (is_x ? r : I + r)) & mask) * 16 + n;
                        val[j] = is_x ? w[sp][j] : -w[sp][j];           // dL/dz = -dL/do
                        if (ok[j]) old[j] = ring[at[j]];
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (ok[j]) {
                            ring[at[j]] = old[j] + val[j];
                            su[sp] -= val[j];
                        }
                    }
                }
            }
        }
        // row sums over the four lane groups; lane group g keeps the one of position s0 + g
        float mine = 0.0f;
#pragma unroll
        for (int sp = 0; sp < 4; ++sp) {
            float v = su[sp];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            mine = g == sp ? v : mine;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int s = s0 + g;
        if (s >= 0 && s < T) {
            float *slot = &ring[(s & mask) * 16 + n];
            a.gv[(size_t)s * Bp + col] = *slot;
            *slot = 0.0f;
        }
        const int t = s + I - 1;
        if (t >= 0 && t < T) {
            a.gu[(size_t)t * Bp + col] = mine + pen_grad;
        }
        if (pads && pad_col < Bp) {
            for (int k = 0; k < 4; ++k) {
                if (s0 + k >= 0 && s0 + k < T) a.gv[(size_t)(s0 + k) * Bp + pad_col] = 0.0f;
                if (s0 + k + I - 1 >= 0 && s0 + k + I - 1 < T) a.gu[(size_t)(s0 + k + I - 1) * Bp + pad_col] = 0.0f;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// ---------------------------------------------------------------------------
// Adjoint of the smoothing recursions: reverse sweep over time, one lane per
// series.  Lb is the adjoint of the level; the adjoints of the seasonal factors
// sit in a per-lane LDS ring (slot t mod m holds the adjoint of the factor for
// time t + m when step t starts, and that of time t when it ends).
// ---------------------------------------------------------------------------
struct EsBwdArgs {
    const float *y;
    const int32_t *lengths;
    const float *es;
    const float *lvl, *S1, *S2, *gu, *gv;   // [T][Bp]
    float *grad_es;                          // [K][B]
    int blocks;                              // workgroups of the recursions; the launch's others reduce weight gradients
    int B, Bp, T, n_seas, m1, m2, logit;
    int row_gamma1, row_gamma2, row_s1, row_s2;
};

// Division of labour, as in the forward recursion.  The reverse recursion is linear in the adjoints: at step t
//   Lb   = gu[t] / l[t] + (carry),            x = Lb * alpha * q,   z1 = A1 * g1 * r1,   z2 = A2 * g2 * r2,
//   S1b  = -gv[t] / s1 + A1 (1 - g1) - (z2 + x) / s1,        S2b likewise with the indices exchanged,
//   Lb'  = Lb (1 - alpha) - (z1 + z2) / l[t-1]               (carried to step t-1),
// with q = y / (s1 s2), r1 = y / (l[t-1] s2), r2 = y / (l[t-1] s1): every coefficient depends on the forward
// pass only.  Three helper waves read the rows of a chunk of steps (a chunk ahead), form the twelve
// coefficients of every step - all the divisions - and stage them in LDS; wave 0 carries the adjoints through
// them: a dozen multiply-adds, the ring accesses and nothing else.
constexpr int kEsBwdChunk = 6;                // steps per staging buffer
constexpr int kEsBwdHelpers = 3;              // waves that form coefficients, each every third step
// coefficients per step: four, and four more per seasonality
constexpr int es_bwd_coefs(int n_seas) { return 4 + 4 * n_seas; }
constexpr int es_bwd_stage_floats(int n_seas) { return 2 * kEsBwdChunk * es_bwd_coefs(n_seas) * 64; }

template <int NS>
__global__ void __launch_bounds__(64 * (1 + kEsBwdHelpers)) es_backward_kernel(EsBwdArgs a, ReduceStage2Args reduce)
{
    extern __shared__ __align__(16) float ring[];   // [m1 + m2][64] rings, then [2][kEsBwdChunk][4 + 4 NS][64] staging
    static_assert(kEsBwdHelpers == 3 && es_bwd_stage_floats(0) >= 256, "the reduction has 256 threads and works in the same LDS");
    if ((int)blockIdx.x >= a.blocks) {
        reduce_stage2_body(reduce, blockIdx.x - a.blocks, ring);
        return;
    }
    constexpr int CH = kEsBwdChunk, NC = es_bwd_coefs(NS);
    const int role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int b = blockIdx.x * 64 + lane;     // column of the time-major arrays (their rows are padded to whole waves)
    const bool in_batch = b < a.B;
    const int bc = in_batch ? b : a.B - 1;    // column of the arrays with B columns
    const int len = in_batch ? clamp_len(a.lengths[b], a.T) : 0;
    // the sweep starts at the last observation of the wave's longest series (rows beyond were not produced);
    // both waves hold the same 64 series, so the bound is the same in both
    const int t_top = max(wave_max_int(len), 1) - 1;
    float *ring1 = ring, *ring2 = ring + (size_t)a.m1 * 64;
    float *stage = ring + (size_t)(a.m1 + a.m2) * 64;
    float alpha = a.es[bc], g1 = 0.0f, g2 = 0.0f;
    if (NS >= 1) g1 = a.es[(size_t)a.row_gamma1 * a.B + bc];
    if (NS >= 2) g2 = a.es[(size_t)a.row_gamma2 * a.B + bc];
    if (a.logit) {
        alpha = 1.0f / (1.0f + expf(-alpha));
        g1 = 1.0f / (1.0f + expf(-g1));
        g2 = 1.0f / (1.0f + expf(-g2));
    }
    for (int e = threadIdx.x; e < (a.m1 + a.m2) * 64; e += 64 * (1 + kEsBwdHelpers)) ring[e] = 0.0f;
    __syncthreads();
    // The sweep runs over the same times t_top ... 1 in every lane; a lane takes part from its own last
    // observation on (its state updates are switched off before that).  Time, ring slots and row addresses
    // are then wave-uniform.  Rows past a series' length hold defined values (level 1, factors 1, zero
    // adjoints).  Chunk c holds the steps t = t_top - c CH - k, k = 0 .. CH-1, as far as t >= 1.
    const int n_chunks = (t_top + CH - 1) / CH;
    float ab = 0.0f, g1b = 0.0f, g2b = 0.0f;
    float Lb_carry = 0.0f;      // contributions to the adjoint of l[t] from later steps

    // All waves run the same loop and meet at its one barrier: in interval j the helper waves stage chunk j
    // (helper h the steps k = h, h + 3, ...) while wave 0 consumes chunk j - 1 from the other buffer.
    if (role >= 1) {
        constexpr int NK = CH / kEsBwdHelpers;      // steps of a chunk per helper
        static_assert(CH % kEsBwdHelpers == 0, "helpers share a chunk evenly");
        struct Raw { float gu, gv, y, lt, lp, s1, s2; };
        Raw raw[kEsAhead][NK];
        const unsigned ub = b, ubc = bc;
        auto load_chunk = [&](int c, Raw *r) {
#pragma unroll
            for (int i = 0; i < NK; ++i) {
                const int k = (role - 1) + i * kEsBwdHelpers;
                const unsigned tc = (unsigned)max(t_top - c * CH - k, 1);      // steps below 1 are not executed
                // element offsets in 32 bits (B * T is at most 2^30): one scalar multiply per row
                const unsigned at = tc * (unsigned)a.Bp + ub;
                r[i].gu = a.gu[at];
                r[i].gv = a.gv[at];
                r[i].y = a.y[tc * (unsigned)a.B + ubc];
                r[i].lt = a.lvl[at];
                r[i].lp = a.lvl[at - (unsigned)a.Bp];
                r[i].s1 = NS >= 1 ? a.S1[at] : 1.0f;
                r[i].s2 = NS >= 2 ? a.S2[at] : 1.0f;
            }
        };
        // rows are requested kEsAhead chunks ahead (register sets rotating through an unrolled loop, as in the
        // forward recursion)
        static_for<0, kEsAhead>([&](auto d) { load_chunk(decltype(d)::value, raw[decltype(d)::value]); });
        // (the last interval stages a chunk that nobody takes: one way through the loop)
        rotate_while<kEsAhead>([&](auto dd, int j) {
            constexpr int d = decltype(dd)::value;
            if (j > n_chunks) return false;                 // (wave-uniform)
            float *out = stage + (j & 1) * (CH * NC * 64) + lane;
#pragma unroll
            for (int i = 0; i < NK; ++i) {
                const int k = (role - 1) + i * kEsBwdHelpers;
                const Raw &r = raw[d][i];
                const float ilp = fast_rcp(r.lp);
                const float is1 = NS >= 1 ? fast_rcp(r.s1) : 1.0f, is2 = NS >= 2 ? fast_rcp(r.s2) : 1.0f;
                const float ry = r.y * ilp;
                const float r1 = ry * is2, r2 = ry * is1;
                const float q = r.y * (is1 * is2);
                float *o = out + k * NC * 64;
                o[0 * 64] = r.gu * fast_rcp(r.lt);
                o[1 * 64] = ilp;
                o[2 * 64] = alpha * q;
                o[3 * 64] = q - r.lp;
                if (NS >= 1) {
                    o[4 * 64] = -r.gv * is1;
                    o[5 * 64] = is1;
                    o[6 * 64] = g1 * r1;
                    o[7 * 64] = r1 - r.s1;
                }
                if (NS >= 2) {
                    o[8 * 64] = -r.gv * is2;
                    o[9 * 64] = is2;
                    o[10 * 64] = g2 * r2;
                    o[11 * 64] = r2 - r.s2;
                }
            }
            load_chunk(j + kEsAhead, raw[d]);
            lds_barrier();
            return true;
        });
        return;
    }

    int i1 = NS >= 1 ? t_top % a.m1 : 0, i2 = NS >= 2 ? t_top % a.m2 : 0;   // ring slot of time t: t mod m
    // adjoint of the factor for time t + m, requested one step ahead of its use
    float A1 = 0.0f, A2 = 0.0f;
    const float one_m_alpha = 1.0f - alpha, one_m_g1 = 1.0f - g1, one_m_g2 = 1.0f - g2;
    auto step = [&](int t, const float (&cf)[NC]) {
        const bool active = t <= len - 1;
        // slot of the next step (time t-1): last written m-1 steps ago unless m = 1
        const int j1 = i1 == 0 ? a.m1 - 1 : i1 - 1, j2 = i2 == 0 ? a.m2 - 1 : i2 - 1;
        float A1n = 0.0f, A2n = 0.0f;
        if (NS >= 1) A1n = ring1[j1 * 64 + lane];
        if (NS >= 2) A2n = ring2[j2 * 64 + lane];
        const float Lb = cf[0] + Lb_carry;
        const float ilp = cf[1];
        const float x = Lb * cf[2];
        ab += active ? Lb * cf[3] : 0.0f;
        const float z1 = NS >= 1 ? A1 * cf[NS >= 1 ? 6 : 0] : 0.0f;
        const float z2 = NS >= 2 ? A2 * cf[NS >= 2 ? 10 : 0] : 0.0f;
        if (NS >= 1) {
            const float S1b = cf[NS >= 1 ? 4 : 0] + A1 * one_m_g1 - (z2 + x) * cf[NS >= 1 ? 5 : 0];
            g1b += active ? A1 * cf[NS >= 1 ? 7 : 0] : 0.0f;
            // an inactive lane leaves the slot as it is (zero)
            ring1[i1 * 64 + lane] = active ? S1b : A1;
            A1 = (a.m1 == 1 && active) ? S1b : A1n;
            i1 = j1;
        }
        if (NS >= 2) {
            const float S2b = cf[NS >= 2 ? 8 : 0] + A2 * one_m_g2 - (z1 + x) * cf[NS >= 2 ? 9 : 0];
            g2b += active ? A2 * cf[NS >= 2 ? 11 : 0] : 0.0f;
            ring2[i2 * 64 + lane] = active ? S2b : A2;
            A2 = (a.m2 == 1 && active) ? S2b : A2n;
            i2 = j2;
        }
        const float Lb_prev = Lb * one_m_alpha - (z1 + z2) * ilp;
        Lb_carry = active ? Lb_prev : 0.0f;
    };
    if (NS >= 1) A1 = ring1[i1 * 64 + lane];
    if (NS >= 2) A2 = ring2[i2 * 64 + lane];
    for (int j = 0; j <= n_chunks; ++j) {
        if (j >= 1) {
            const int c = j - 1;
            const float *in = stage + (c & 1) * (CH * NC * 64) + lane;
            const int t_hi = t_top - c * CH;
            // the coefficients of the whole chunk, read together: one LDS round trip per chunk
            float cf[CH][NC];
#pragma unroll
            for (int k = 0; k < CH; ++k)
#pragma unroll
                for (int i = 0; i < NC; ++i) cf[k][i] = in[(k * NC + i) * 64];
            if (t_hi - CH >= 0) {                   // a whole chunk: no branch inside
#pragma unroll
                for (int k = 0; k < CH; ++k) step(t_hi - k, cf[k]);
            } else {
#pragma unroll
                for (int k = 0; k < CH; ++k)
                    if (t_hi - k >= 1) step(t_hi - k, cf[k]);
            }
        }
        lds_barrier();
    }
    if (!in_batch) return;      // (no barrier below)
    if (len >= 1) {
        // t = 0: l[0] = y0 / (S1[0] S2[0]); the first produced factors equal the initial ones
        const size_t o = b;
        const float l0 = a.lvl[o];
        const float Lb = a.gu[o] / l0 + Lb_carry;
        const float gv0 = a.gv[o];
        if (NS >= 1) {
            const float s1 = a.S1[o];
            const float A = (a.m1 <= len - 1) ? ring1[lane] : 0.0f;
            ring1[lane] = -gv0 / s1 + A - Lb * l0 / s1;
        }
        if (NS >= 2) {
            const float s2 = a.S2[o];
            const float A = (a.m2 <= len - 1) ? ring2[lane] : 0.0f;
            ring2[lane] = -gv0 / s2 + A - Lb * l0 / s2;
        }
    }
    a.grad_es[b] = a.logit ? ab * alpha * (1.0f - alpha) : ab;
    if (NS >= 1) {
        a.grad_es[(size_t)a.row_gamma1 * a.B + b] = a.logit ? g1b * g1 * (1.0f - g1) : g1b;
        for (int k = 0; k < a.m1; ++k) {
            float gs = (k < len) ? ring1[k * 64 + lane] : 0.0f;
            if (a.logit) gs *= (k < len) ? a.S1[(size_t)k * a.Bp + b] : 0.0f;
            a.grad_es[(size_t)(a.row_s1 + k) * a.B + b] = gs;
        }
    }
    if (NS >= 2) {
        a.grad_es[(size_t)a.row_gamma2 * a.B + b] = a.logit ? g2b * g2 * (1.0f - g2) : g2b;
        for (int k = 0; k < a.m2; ++k) {
            float gs = (k < len) ? ring2[k * 64 + lane] : 0.0f;
            if (a.logit) gs *= (k < len) ? a.S2[(size_t)k * a.Bp + b] : 0.0f;
            a.grad_es[(size_t)(a.row_s2 + k) * a.B + b] = gs;
        }
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {
// Dynamic LDS above 64 KB has to be allowed per kernel.  Done once per kernel and device for the whole
// 160 KB, on the first launch that needs it (not on every launch: the call is not a stream operation).
hipError_t allow_large_lds(const void *kernel, size_t lds)
{
    if (lds <= 64 * 1024) return hipSuccess;
    constexpr int kMaxKernels = 32, kMaxDevices = 64;
    static std::mutex mu;
    static const void *known[kMaxKernels];
    static bool done[kMaxKernels][kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    int slot = -1;
    for (int i = 0; i < kMaxKernels && slot < 0; ++i)
        if (known[i] == kernel || known[i] == nullptr) { known[i] = kernel; slot = i; }
    if (slot >= 0 && dev >= 0 && dev < kMaxDevices && done[slot][dev]) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess && slot >= 0 && dev >= 0 && dev < kMaxDevices) done[slot][dev] = true;
    return e;
}
}  // namespace

namespace {
// Up to this many workgroups the kernel that keeps only the level in its chain: 16 384 hourly series 105 -> 68 us with the
// set-up, at 512 75 -> 51 us.  (Measured no further: four times that batch no longer fits the memory.)  It needs three chunks
// of eight steps in the shorter period; with chunks of four, for the periods from 12 on, it was no faster (240 monthly steps
// at 512 to 16 384 series: 22 - 26 us either way, at 65 536 71 against 60 us).
constexpr int kEsLongMostBlocks = 256;

SetupArgs setup_args(const Plan &pl, const Lengths &len, const float *weights, unsigned *need, float *ws)
{
    SetupArgs a{};
    a.L = pl.L;
    a.prep = PrepArgs{len, reinterpret_cast<Scalars *>(ws + pl.scalars), reinterpret_cast<int32_t *>(ws + pl.pmax), pl.NB,
                      pl.B, pl.H, pl.h * pl.cfg.n_blocks, TogetherWords{reinterpret_cast<unsigned *>(ws + pl.together_words), weights && pl.together_fwd ? 1 + pl.together_groups : 0}};
    a.pmax_blocks = std::min((pl.NB + 255) / 256, 63);
    if (len.extend) {
        ClassArgs &c = a.classes;
        c.lengths = len;
        c.ext = reinterpret_cast<int32_t *>(ws + pl.len_ext);
        c.need = need;
        c.L = pl.L; c.NB = pl.NB; c.B = pl.B;
        for (int l = 0; l < pl.L; ++l) {
            const int d = c.dil[l] = pl.layer[l].dil, above = l + 1 < pl.L ? pl.layer[l + 1].dil : 0;
            c.gcd_above[l] = above == pl.P ? d : d == pl.P ? above : std::gcd(d, above);
        }
        a.extend_blocks = (pl.B + 255) / 256;
    }
    if (!weights) return a;
    int max_total = 256;
    for (int l = 0; l < pl.L; ++l) {
        const LayerPlan &lp = pl.layer[l];
        a.lstm[l] = PackLstmArgs{weights + lp.w_off, weights + lp.b_off, ws + lp.wpack_fwd, ws + lp.bias_pack,
                                 ws + lp.wpack_bwd, pl.h, lp.in_dim, pl.HT, lp.KXT, lp.narrow_fwd, lp.narrow_bwd};
        max_total = std::max(max_total, 4 * pl.HT * 64 * (lp.KXT + pl.HT));     // (about the larger of the two operands)
    }
    const HeadPack hp = head_pack_layout(pl);
    float *f = ws + pl.head_fwd_pack, *b = ws + pl.head_bwd_pack;
    a.head = PackHeadArgs{weights + pl.Wa_off, weights + pl.ba_off, weights + pl.Wo_off, weights + pl.bo_off,
                          f + hp.WaF, f + hp.baF, f + hp.WoF, f + hp.boF, b + hp.WoT, b + hp.WaT, a.prep.sc,
                          pl.h, pl.H, pl.HT, pl.MA, pl.MO};
    a.pack_blocks = std::min((max_total + 255) / 256, 64);      // (the bodies loop over their elements)
    return a;
}
}  // namespace

hipError_t launch_es_forward(const Plan &pl, const float *y, const int32_t *lengths, const float *es, const float *weights,
                             float *ws, const ForwardMode &mode, hipStream_t st)
{
    const esrnn_config &c = pl.cfg;
    const Lengths len{lengths, pl.T, pl.I, mode.out_of_sample ? pl.H : 0};
    const SetupArgs setup = setup_args(pl, len, weights, mode.need, ws);
    EsArgs a{y, len, es, ws + pl.lvl, ws + pl.S1, ws + pl.S2, ws + pl.u, ws + pl.v,
             ws + pl.loss_partial + (pl.n_loss_partial - pl.es_blocks), pl.es_blocks,
             pl.B, pl.Bt, pl.T, c.n_seas, c.n_seas >= 1 ? c.m1 : 0, c.n_seas >= 2 ? c.m2 : 0,
             c.param_space == ESRNN_PARAMS_LOGIT, pl.row_gamma1, pl.row_gamma2, pl.row_s1, pl.row_s2};
    static_assert(es_stage_floats(0) >= kSetupScratch, "the set-up works in the same LDS");
    const size_t lds = ((size_t)(a.m1 + a.m2) * 64 + es_stage_floats(c.n_seas)) * sizeof(float);
    auto run = [&](auto kernel) {
        hipError_t e = allow_large_lds(reinterpret_cast<const void *>(kernel), lds);
        if (e != hipSuccess) return e;
        kernel<<<pl.es_blocks + setup.blocks(), 256, lds, st>>>(a, setup);
        return hipGetLastError();
    };
    int m_min = c.n_seas >= 1 ? c.m1 : 8;
    if (c.n_seas >= 2) m_min = std::min(m_min, c.m2);
    const size_t long_lds = ((size_t)(a.m1 + a.m2) * 64 + es_long_stage_floats(c.n_seas)) * sizeof(float);
    if (c.n_seas >= 1 && m_min >= 3 * kEsLongChunk && pl.es_blocks <= kEsLongMostBlocks && long_lds <= 152 * 1024) {
        auto run_long = [&](auto kernel) {
            hipError_t e = allow_large_lds(reinterpret_cast<const void *>(kernel), long_lds);
            if (e != hipSuccess) return e;
            kernel<<<pl.es_blocks + setup.blocks(), 64 * kEsLongWaves, long_lds, st>>>(a, setup);
            return hipGetLastError();
        };
        return c.n_seas == 1 ? run_long(es_forward_long_kernel<1>) : run_long(es_forward_long_kernel<2>);
    }
    // steps per group: the largest divisor of 8 that no period is shorter than
    const int cs = m_min >= 8 ? 8 : (m_min >= 4 ? 4 : (m_min >= 2 ? 2 : 1));
    if (c.n_seas == 0) return run(es_forward_kernel<0, 8>);
    if (c.n_seas == 1) {
        if (cs == 8) return run(es_forward_kernel<1, 8>);
        if (cs == 4) return run(es_forward_kernel<1, 4>);
        if (cs == 2) return run(es_forward_kernel<1, 2>);
        return run(es_forward_kernel<1, 1>);
    }
    if (cs == 8) return run(es_forward_kernel<2, 8>);
    if (cs == 4) return run(es_forward_kernel<2, 4>);
    if (cs == 2) return run(es_forward_kernel<2, 2>);
    return run(es_forward_kernel<2, 1>);
}

hipError_t launch_window_forward(const Plan &pl, const int32_t *categories, float *ws, hipStream_t st)
{
    // few positions per wave at small batches (enough waves), more at large ones (less per-wave overhead)
    const int p_per_wave = pl.NB >= 2048 ? 8 : (pl.NB >= 512 ? 4 : 1);
    window_forward_kernel<<<dim3((pl.NB + 3) / 4, (pl.P + p_per_wave - 1) / p_per_wave), 256, 0, st>>>(ws + pl.u, ws + pl.v, ws + pl.X, ws + pl.Z,
                                                                         pl.P, pl.NB, pl.Bt, pl.I, pl.H, 4 * pl.IT,
                                                                         pl.OP, p_per_wave, categories, pl.C, pl.B,
                                                                         reinterpret_cast<const int32_t *>(ws + pl.pmax));
    return hipGetLastError();
}

namespace {
int reduce_splits(int n_part) { return std::min(n_part, kReduceSplits); }

ReduceJobs reduce_jobs(const Plan &pl, float *ws)
{
    ReduceJobs jobs{};
    int nj = 0;
    auto add = [&](size_t src, size_t dst, size_t stride, int n_part, int n_elems) {
        const int splits = reduce_splits(n_part);
        jobs.blocks += (n_elems + 255) / 256 * splits;
        jobs.job[nj++] = ReduceJob{ws + src, ws + dst, (unsigned)stride, n_part, n_elems, splits, jobs.blocks};
    };
    for (int l = 0; l < pl.L; ++l) {
        const LayerPlan &lp = pl.layer[l];
        const int MB = (lp.KXT + pl.HT + 3) / 4;
        const int n_dw = pl.HT * MB * 256, n_db = pl.HT * 16;
        add(lp.dw_partial, lp.dw_reduced, n_dw, pl.partial_groups(lp), n_dw);
        add(lp.db_partial, lp.db_reduced, n_db, pl.partial_groups(lp), n_db);
    }
    const int n_head = (pl.MO * pl.MA + pl.MA * pl.MA) * 256 + 4 * pl.OT + 4 * pl.HT;
    add(pl.head_dw_partial, pl.head_dw_reduced, pl.head_dw_stride, pl.head_blocks, n_head);
    return jobs;
}

ReduceStage2Args reduce_stage2_args(const Plan &pl, float *ws, float *grad_weights)
{
    ReduceStage2Args r{};
    r.L = pl.L;
    r.words = TogetherWords{reinterpret_cast<unsigned *>(ws + pl.together_words_bwd), pl.together_bwd ? 1 + pl.together_groups_bwd : 0};
    int blocks = 0;
    for (int l = 0; l < pl.L; ++l) {
        const LayerPlan &lp = pl.layer[l];
        r.lstm[l] = ReduceLstmArgs{ws + lp.dw_reduced, ws + lp.db_reduced, grad_weights + lp.w_off,
                                   grad_weights + lp.b_off, reduce_splits(pl.partial_groups(lp)), pl.h, lp.in_dim, pl.HT, lp.KXT};
        const int MB = (lp.KXT + pl.HT + 3) / 4;
        r.end[l] = blocks += (pl.HT * MB * 256 + 63) / 64 + (pl.HT * 16 + 63) / 64;
    }
    const int n_head = (pl.MO * pl.MA + pl.MA * pl.MA) * 256 + 4 * pl.OT + 4 * pl.HT;
    r.head = ReduceHeadArgs{ws + pl.head_dw_reduced, grad_weights + pl.Wa_off, grad_weights + pl.ba_off,
                            grad_weights + pl.Wo_off, grad_weights + pl.bo_off,
                            reduce_splits(pl.head_blocks), n_head, pl.h, pl.H, pl.HT, pl.MA, pl.MO, pl.OT};
    r.end[kMaxLayers] = blocks + (n_head + 63) / 64;
    return r;
}
}  // namespace

hipError_t launch_window_backward(const Plan &pl, const int32_t *lengths, float *ws, bool reduce, hipStream_t st)
{
    const ReduceJobs jobs = reduce ? reduce_jobs(pl, ws) : ReduceJobs{};
    WindowBwdArgs a{ws + pl.gX, ws + pl.gO, ws + pl.u, lengths, reinterpret_cast<const Scalars *>(ws + pl.scalars),
                    pl.cfg.lambda_lv, ws + pl.gu, ws + pl.gv, pl.P, pl.NB, pl.B, pl.Bt, pl.T, pl.I, pl.H, 4 * pl.IT, pl.OP,
                    reinterpret_cast<const int32_t *>(ws + pl.pmax), 0, 0, 0};
    if (pl.window_stream) {
        a.R = 16;
        while (a.R < pl.I + pl.H + 4) a.R *= 2;             // ring of anti-diagonal sums, a power of two
        a.blocks = (pl.NB + 3) / 4;
        const unsigned grid = (unsigned)(a.blocks + jobs.blocks);
        const size_t lds = (size_t)4 * a.R * 16 * sizeof(float);
        if (pl.window_ahead) window_backward_stream_kernel<3><<<grid, 256, lds, st>>>(a, jobs);
        else window_backward_stream_kernel<0><<<grid, 256, lds, st>>>(a, jobs);
        return hipGetLastError();
    }
    a.t_chunks = (pl.T + 3) / 4;                            // four time steps per workgroup
    const int col_slots = (pl.Bt / 64 + 7) / 8;             // groups of 64 series per XCD
    a.blocks = 8 * col_slots * a.t_chunks;
    window_backward_kernel<<<(unsigned)(a.blocks + jobs.blocks), 256, 0, st>>>(a, jobs);
    return hipGetLastError();
}

hipError_t launch_es_backward(const Plan &pl, const float *y, const int32_t *lengths, const float *es, float *ws,
                              float *grad_es, float *grad_weights, hipStream_t st)
{
    const esrnn_config &c = pl.cfg;
    const ReduceStage2Args reduce = grad_weights ? reduce_stage2_args(pl, ws, grad_weights) : ReduceStage2Args{};
    EsBwdArgs a{y, lengths, es, ws + pl.lvl, ws + pl.S1, ws + pl.S2, ws + pl.gu, ws + pl.gv, grad_es, (pl.B + 63) / 64,
                pl.B, pl.Bt, pl.T, c.n_seas, c.n_seas >= 1 ? c.m1 : 0, c.n_seas >= 2 ? c.m2 : 0,
                c.param_space == ESRNN_PARAMS_LOGIT, pl.row_gamma1, pl.row_gamma2, pl.row_s1, pl.row_s2};
    const size_t lds = ((size_t)(a.m1 + a.m2) * 64 + es_bwd_stage_floats(c.n_seas)) * sizeof(float);
    auto run = [&](auto kernel) {
        hipError_t e = allow_large_lds(reinterpret_cast<const void *>(kernel), lds);
        if (e != hipSuccess) return e;
        kernel<<<(unsigned)(a.blocks + reduce.blocks()), 64 * (1 + kEsBwdHelpers), lds, st>>>(a, reduce);
        return hipGetLastError();
    };
    if (c.n_seas == 0) return run(es_backward_kernel<0>);
    if (c.n_seas == 1) return run(es_backward_kernel<1>);
    return run(es_backward_kernel<2>);
}

// ---------------------------------------------------------------------------
// Accuracy of forecasts against actual values, per series (Section 3.5 names the two metrics of the
// M4 competition): sMAPE = mean_h 200 |a - f| / (|a| + |f|); MASE = mean_h |a - f| divided by the
// in-sample mean of |y_t - y_{t-m}|, t = m .. len-1 (seasonal naive forecast of period m).
__global__ void __launch_bounds__(256) forecast_metrics_kernel(const float *__restrict__ f, const float *__restrict__ a,
                                                                const float *__restrict__ y, const int32_t *__restrict__ lengths,
                                                                float *__restrict__ smape, float *__restrict__ mase,
                                                                int B, int T, int H, int m)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= B) return;
    float s_sym = 0.0f, s_abs = 0.0f;
    for (int j = 0; j < H; ++j) {
        const float fv = f[(size_t)b * H + j], av = a[(size_t)b * H + j];
        const float d = fabsf(av - fv);
        s_sym += 200.0f * d / (fabsf(av) + fabsf(fv));
        s_abs += d;
    }
    const int len = clamp_len(lengths[b], T);
    float s_naive = 0.0f;
    for (int t = m; t < len; ++t) s_naive += fabsf(y[(size_t)t * B + b] - y[(size_t)(t - m) * B + b]);
    smape[b] = s_sym / (float)H;
    mase[b] = (s_abs / (float)H) / (s_naive / (float)(len - m));
}

hipError_t launch_forecast_metrics(const Plan &pl, const float *forecasts, const float *actuals, const float *y,
                                   const int32_t *lengths, int m, float *smape, float *mase, hipStream_t st)
{
    forecast_metrics_kernel<<<(pl.B + 255) / 256, 256, 0, st>>>(forecasts, actuals, y, lengths, smape, mase,
                                                                 pl.B, pl.T, pl.H, m);
    return hipGetLastError();
}

}  // namespace esrnn
