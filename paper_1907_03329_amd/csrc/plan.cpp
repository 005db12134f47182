// Host-side launch plan: validates a configuration, lays out the workspace and
// the packed operand blocks.  No device work happens here.
#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "esrnn_internal.h"
#include "three_term.h"

namespace esrnn {

namespace {

struct Bump {
    size_t at = 0;
    size_t take(size_t n_floats)
    {
        size_t r = at;
        at += (n_floats + 63) & ~size_t(63);   // keep every block 256-byte aligned
        return r;
    }
};

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Layers whose 16-series grid has fewer workgroups than this run on the 4-series kernels, separately for the two
// directions: with four times the workgroups a chip that is not full carries a quarter of the memory traffic on each.
// Measured on two layers of the same dilation, 61 positions (window 4) and 151 (window 12), in us with the events around a launch (16-series
// kernel against 4-series kernel, second layer, 61 positions unless stated; at 64 and less the 4-series kernels are the faster
// ones):
//   hidden   groups 68 (dilation 2)                72 (dilation 1)                    128 (dilation 1)
//      8     forward 13 / 16, reverse 16 / 22      21 / 26,  27 / 38                  22 / 27,  28 / 39
//     30     23 / 25,  32 / 38                     39 / 43,  55 / 65                  39 / 44,  56 / 68
//     40     31 / 32,  43 / 56                     54 / 51,  74 / 99                  55 / 60,  75 / 102
//     50     40 / 38,  68 / 92                     72 / 67,  122 / 167                73 / 71,  123 / 172
//     60     43 / 44,  188 / 104                   77 / 79,  364 / 189                80 / 82,  372 / 194
// and with 151 positions alike (hidden 40, 72 groups: 124 / 114, 172 / 229).  The line is where the first 4-series kernels lost in both
// directions; now their forward pass is up to 10 % faster at 68 and 72 groups of hidden 40 and 50 and slower at 128, and first layers of hidden 50
// are faster in reverse (72 groups, 151 positions 224 / 184).  Above hidden 52 the reverse pass of 16 series is the fp32 kernel, which
// loses up to 176 groups of dilation one (160: 372 / 289 us, 200: 374 / 376); at 160 it depends on the dilation (eight: 57 / 60, and
// 121 / 108 with 151 positions).
constexpr int kNarrowForwardBelow = 65, kNarrowBackwardBelow = 65, kNarrowBackwardBelowFp32 = 160;
// Series tiles from which the window adjoint streams (one wave per tile) instead of gathering (one thread per
// time step and series).  Gather against streaming in us: quarterly shape at 1024 / 2048 / 4096 / 8192 tiles 21 / 35 / 77 / 157
// and 52 / 58 / 77 / 155, yearly 14 / 22 / 37 / 81 and 28 / 33 / 40 / 85, monthly 131 / 257 / 497 / 979 and 274 / 324 / 440 / 949;
// a wave of the streaming kernel is a chain of dependent memory round trips and needs about sixteen waves per SIMD to
// hide them.  (Of the kernel that requests nothing ahead.)
constexpr int kWindowStreamFromDefault = 4096;

// Row groups of four that hold the elements of a window position.
int window_row_groups(int I, int H) { return ceil_div(I, 4) + ceil_div(H, 4); }

// Series tiles from which windows of three row groups take the streaming kernel that requests a block ahead; with four groups
// (yearly) two blocks are more registers than there are (97 and 198 us at 4096 and 8192 tiles: 4 to 6 us slower); fewer were not measured.  Reverse pass of smoothing and windows in us, gathered /
// streamed / with a block ahead, quarterly shape: 3072 tiles 59 / 75 / 55, 3333 66 / 86 / 65, 3584 74 / 85 / 64, 4096 92 / 93 / 72, 4375
// 100 / 105 / 98, 5120 115 / 105 / 105, 8192 188 / 184 / 157, 12 289 273 / 274 / 236, 32 768 734 / 643 / 584; with 40 steps instead of 72 3333 40 / 50 /
// 42, 3584 42 / 48 / 40, 4375 49 / 56 / 55; windows of 3 + 5 and of 6 + 4 alike.
constexpr int kWindowAheadFrom = 3600;
bool window_ahead_pays(int tiles, int I, int H) { return window_row_groups(I, H) == 3 && tiles >= kWindowAheadFrom; }

// Chains of the 16-series reverse kernels, which have one workgroup per compute unit: the fewest that take the least
// time, counted in rounds of 256 workgroups times classes each walks (80 groups, four classes: 320 workgroups with
// four chains are two rounds, 49 us; with two chains one round of two classes, 44 us).  No more than fill the chip
// once: every workgroup leaves a block of weight-gradient partials to be reduced.
int wide_reverse_chains(int groups, int classes)
{
    int best = 1;
    long long best_cost = -1;
    for (int c = 1; c <= classes && (c == 1 || groups * c <= 256); ++c) {
        const long long cost = (long long)ceil_div(groups * c, 256) * ceil_div(classes, c);
        if (best_cost < 0 || cost < best_cost) { best = c; best_cost = cost; }
    }
    return best;
}

// hidden sizes are padded to one of the instantiated unit-tile counts
int pick_ht(int hidden)
{
    const int need = ceil_div(hidden, 4);
    const int avail[] = {2, 8, 10, 13, 16};
    for (int v : avail)
        if (need <= v) return v;
    return -1;
}

}  // namespace

bool lstm_shape_supported(int HT, int KXT)
{
#define X(HT_, KXT_) if (HT == HT_ && KXT == KXT_) return true;
    ESRNN_LSTM_SHAPES(X)
#undef X
    return false;
}

HeadPack head_pack_layout(const Plan &pl)
{
    HeadPack hp{};
    Bump b;
    const size_t qh = (size_t)tt_a_quads((pl.HT + 1) / 2) * 256, qo = (size_t)tt_a_quads(2 * pl.MO) * 256;
    hp.WaF = b.take(pl.MA * qh);
    hp.baF = b.take((size_t)pl.MA * 16);
    hp.WoF = b.take(pl.MO * qh);
    hp.boF = b.take((size_t)pl.MO * 16);
    hp.fwd_total = b.at;
    Bump c;
    hp.WoT = c.take(pl.MA * qo);
    hp.WaT = c.take(pl.MA * qh);
    hp.bwd_total = c.at;
    return hp;
}

esrnn_status build_plan(const esrnn_config &cfg, Plan &pl)
{
    std::memset(&pl, 0, sizeof(pl));
    // ESRNN_NARROW_BELOW overrides both thresholds (0: never, a large number: always), for measurements.
    int narrow_fwd_below = kNarrowForwardBelow;
    int narrow_bwd_below = bwd_three_term(pick_ht(cfg.hidden)) ? kNarrowBackwardBelow : kNarrowBackwardBelowFp32;
    if (const char *env = std::getenv("ESRNN_NARROW_BELOW")) narrow_fwd_below = narrow_bwd_below = std::atoi(env);
    // The window adjoint streams tile by tile from this many series tiles on (one wave per tile needs enough
    // tiles to hide memory latency); ESRNN_WINDOW_STREAM_FROM overrides, for measurements.
    int window_stream_from = kWindowStreamFromDefault;
    bool default_stream = true;
    if (const char *env = std::getenv("ESRNN_WINDOW_STREAM_FROM")) {
        window_stream_from = std::atoi(env);
        default_stream = false;
    }
    // At most so many workgroups in a launch of several layers; ESRNN_TOGETHER overrides (0: every layer in a launch of its own),
    // for measurements.
    int together_groups = kTogetherGroups;
    if (const char *env = std::getenv("ESRNN_TOGETHER")) together_groups = std::min(std::atoi(env), kTogetherGroups);
    pl.cfg = cfg;
    if (cfg.B < 1 || cfg.T < 1 || cfg.I < 1 || cfg.H < 1 || cfg.hidden < 1) return ESRNN_ERR_CONFIG;
    if (cfg.hidden > ESRNN_MAX_HIDDEN || cfg.I > ESRNN_MAX_WINDOW || cfg.H > ESRNN_MAX_WINDOW) return ESRNN_ERR_CONFIG;
    if (cfg.n_seas < 0 || cfg.n_seas > 2) return ESRNN_ERR_CONFIG;
    if (cfg.n_seas >= 1 && (cfg.m1 < 1 || cfg.m1 > cfg.T)) return ESRNN_ERR_CONFIG;
    if (cfg.n_seas >= 2 && (cfg.m2 < 1 || cfg.m2 > cfg.T)) return ESRNN_ERR_CONFIG;
    // the smoothing kernels keep the seasonal rings of 64 series in LDS: (m1 + m2) * 64 floats, which with the
    // 36 KB staging buffer of the reverse recursion must fit into 160 KB
    if ((long long)(cfg.n_seas >= 1 ? cfg.m1 : 0) + (cfg.n_seas >= 2 ? cfg.m2 : 0) > 448) return ESRNN_ERR_CONFIG;
    if ((long long)cfg.I + cfg.H > cfg.T) return ESRNN_ERR_CONFIG;
    if (cfg.n_blocks < 1 || cfg.n_blocks > ESRNN_MAX_BLOCKS) return ESRNN_ERR_CONFIG;
    if (!(cfg.tau > 0.0f && cfg.tau < 1.0f)) return ESRNN_ERR_CONFIG;
    if (!(cfg.lambda_lv >= 0.0f)) return ESRNN_ERR_CONFIG;
    if (!(cfg.lambda_cs >= 0.0f)) return ESRNN_ERR_CONFIG;
    if (cfg.param_space != ESRNN_PARAMS_DIRECT && cfg.param_space != ESRNN_PARAMS_LOGIT) return ESRNN_ERR_CONFIG;
    if ((long long)cfg.B * cfg.T > (1LL << 30)) return ESRNN_ERR_CONFIG;
    if (cfg.n_categories < 0 || cfg.n_categories > ESRNN_MAX_CATEGORIES) return ESRNN_ERR_CONFIG;
    if (cfg.I + cfg.n_categories > ESRNN_MAX_WINDOW) return ESRNN_ERR_CONFIG;

    pl.B = cfg.B; pl.T = cfg.T; pl.I = cfg.I; pl.H = cfg.H; pl.h = cfg.hidden; pl.C = cfg.n_categories;
    pl.P = cfg.T - cfg.I - cfg.H + 1;
    pl.NB = ceil_div(cfg.B, kTileN);
    bool ahead = window_ahead_pays(pl.NB, pl.I, pl.H);
    pl.window_stream = pl.NB >= window_stream_from || (default_stream && ahead) ? 1 : 0;
    // ESRNN_WINDOW_AHEAD overrides where the adjoint streams (0: never, 1: wherever there are three row groups), for measurements.
    if (const char *env = std::getenv("ESRNN_WINDOW_AHEAD")) ahead = std::atoi(env) && window_row_groups(pl.I, pl.H) == 3;
    pl.window_ahead = pl.window_stream && ahead ? 1 : 0;
    pl.Bp = pl.NB * kTileN;
    pl.Bt = ceil_div(cfg.B, 64) * 64;
    pl.HT = pick_ht(cfg.hidden);
    if (pl.HT < 0) return ESRNN_ERR_CONFIG;
    pl.HP = 4 * pl.HT;
    pl.OT = ceil_div(cfg.H, 4);
    pl.MO = ceil_div(cfg.H, 16);
    pl.OP = 4 * pl.OT;
    pl.MA = ceil_div(pl.HT, 4);
    // layer 0 input tiles: exact if that kernel shape is instantiated, else padded to HT
    pl.IT = ceil_div(cfg.I + pl.C, 4);
    if (!lstm_shape_supported(pl.HT, pl.IT)) {
        if (cfg.I + pl.C > pl.HP) return ESRNN_ERR_CONFIG;
        pl.IT = pl.HT;
    }

    int r = 1;
    pl.row_gamma1 = pl.row_gamma2 = pl.row_s1 = pl.row_s2 = -1;
    if (cfg.n_seas >= 1) pl.row_gamma1 = r++;
    if (cfg.n_seas >= 2) pl.row_gamma2 = r++;
    if (cfg.n_seas >= 1) { pl.row_s1 = r; r += cfg.m1; }
    if (cfg.n_seas >= 2) { pl.row_s2 = r; r += cfg.m2; }
    pl.K = r;

    // user weight offsets
    size_t off = 0;
    int L = 0;
    const int h = cfg.hidden;
    for (int k = 0; k < cfg.n_blocks; ++k) {
        const int nl = cfg.layers_in_block[k];
        if (nl < 1 || nl > ESRNN_MAX_LAYERS_PER_BLOCK) return ESRNN_ERR_CONFIG;
        for (int j = 0; j < nl; ++j) {
            LayerPlan &lp = pl.layer[L];
            if (cfg.dilation[k][j] < 1) return ESRNN_ERR_CONFIG;
            // (a dilation past the last position leaves every position a chain of its own, like one of P; the kernels
            // form positions a few dilations ahead in 32 bits)
            lp.dil = std::min(cfg.dilation[k][j], pl.P);
            lp.block = k;
            lp.first_in_block = (j == 0);
            lp.last_in_block = (j == nl - 1);
            lp.in_dim = (L == 0) ? cfg.I + pl.C : h;
            lp.KXT = (L == 0) ? pl.IT : pl.HT;
            lp.w_off = off; off += (size_t)4 * h * (lp.in_dim + h);
            lp.b_off = off; off += (size_t)4 * h;
            ++L;
        }
    }
    pl.L = L;
    pl.Wa_off = off; off += (size_t)h * h;
    pl.ba_off = off; off += h;
    pl.Wo_off = off; off += (size_t)cfg.H * h;
    pl.bo_off = off; off += cfg.H;
    pl.n_weights = off;

    // workspace
    Bump ws;
    const size_t TB = (size_t)pl.T * pl.Bt;
    const size_t PN = (size_t)pl.P * pl.NB;
    const size_t tileH = (size_t)pl.HT * 64;         // floats of one (p, series-tile) block with HP rows
    // output stage: a tile per wave, no more workgroups than compute units
    const int head_w = head_waves(pl.HT, pl.MO);
    const int head_blocks = (int)std::min<size_t>((PN + head_w - 1) / head_w, 256);
    pl.head_blocks = head_blocks;
    pl.es_blocks = pl.Bt / 64;
    // first everything the smoothing and window stages touch (their own entry points need only this prefix)
    pl.scalars = ws.take(64);
    pl.len_ext = ws.take((size_t)pl.B);
    pl.pmax = ws.take((size_t)pl.NB);
    pl.opt_partial = ws.take(512);
    pl.n_loss_partial = head_blocks + pl.es_blocks;
    pl.loss_partial = ws.take((size_t)pl.n_loss_partial);
    pl.lvl = ws.take(TB); pl.S1 = ws.take(TB); pl.S2 = ws.take(TB);
    pl.u = ws.take(TB); pl.v = ws.take(TB); pl.gu = ws.take(TB); pl.gv = ws.take(TB);
    pl.X = ws.take(PN * (size_t)pl.IT * 64);
    pl.Z = ws.take(PN * (size_t)pl.OP * 16);
    pl.gX = ws.take(PN * (size_t)pl.IT * 64);
    pl.gO = ws.take(PN * (size_t)pl.OP * 16);
    pl.es_window_floats = ws.at;
    pl.O = ws.take(PN * (size_t)pl.OP * 16);
    pl.gTop = ws.take(PN * tileH);
    for (int l = 0; l < L; ++l) {
        LayerPlan &lp = pl.layer[l];
        const int KT = lp.KXT + pl.HT;
        const int MB = ceil_div(KT, 4);
        // Few workgroups (small batch, small dilation): four series per workgroup instead of sixteen.
        // Enough workgroups to put several on every compute unit, without more weight-gradient partials than
        // the reduction can read cheaply.
        const int most_chains = std::min(lp.dil, pl.P);
        auto chains_for = [&](int groups, int fill) { return std::min(most_chains, std::max(1, ceil_div(fill, groups))); };
        const int wide_groups = pl.NB * chains_for(pl.NB, 512);
        lp.narrow_fwd = wide_groups < narrow_fwd_below ? 1 : 0;
        lp.narrow_bwd = wide_groups < narrow_bwd_below ? 1 : 0;
        lp.chains = chains_for(lp.narrow_fwd ? 4 * pl.NB : pl.NB, 512);
        const int groups = lp.narrow_bwd ? 4 * pl.NB : pl.NB;
        // The 4-series reverse kernel has two workgroups per compute unit, or one of twelve waves, staging and weight gradient
        // on waves of their own: the faster kind where the grid has no more than that.
        lp.chains_bwd = lp.narrow_bwd ? chains_for(groups, 512) : wide_reverse_chains(groups, most_chains);
        lp.split_bwd = lp.narrow_bwd && groups * lp.chains_bwd <= 256 ? 1 : 0;
        // The forward operands lie where the first reduction stage of the weight gradient comes at the end of the reverse
        // pass, which does not need them any more and packs none for the next forward pass.
        const size_t fwd_pack = lp.narrow_fwd ? (size_t)4 * (4 * pl.HT + ceil_div(pl.HT, 4) * lp.KXT) * 64
                                              : (size_t)pl.HT * (tt_a_quads((lp.KXT + 1) / 2) + tt_a_quads((pl.HT + 1) / 2)) * 256;
        lp.wpack_fwd = lp.dw_reduced = ws.take(std::max((size_t)kReduceSplits * pl.HT * MB * 256, fwd_pack));
        lp.bias_pack = lp.narrow_fwd ? lp.wpack_fwd : ws.take((size_t)pl.HT * 16);   // (unused by the 4-series kernel)
        lp.wpack_bwd = lp.narrow_bwd ? ws.take((size_t)4 * ceil_div(4 * KT, 64) * 4 * pl.HT * 64)
                       : bwd_three_term(pl.HT) ? ws.take((size_t)bwd_pack_dwords(pl.HT, lp.KXT))
                                               : ws.take((size_t)MB * 4 * pl.HT * 64);
        lp.gates = ws.take(PN * tileH * 4);
        lp.c = ws.take(PN * tileH);
        lp.hid = ws.take(PN * tileH);
        lp.dw_partial = ws.take((size_t)groups * lp.chains_bwd * pl.HT * MB * 256);
        lp.db_partial = ws.take((size_t)groups * lp.chains_bwd * pl.HT * 16);
        lp.db_reduced = ws.take((size_t)kReduceSplits * pl.HT * 16);
        pl.dx[l] = l > 0 ? ws.take(PN * tileH) : pl.gX;
    }
    // First layers in one launch: every workgroup has one class, so that positions rise in all of them, there is a compute unit for
    // each, and a lane for every word that a workgroup looks at.  16-series layers count no positions: one can only be the last.
    // Steps in us, launches of one layer / this rule: quarterly 40 series 188 / 134, 100 192 / 151, 300 218 / 196, 700 264 / 264, 1024 298 / 299;
    // yearly 100 111 / 99, 500 123 / 124; monthly 40 519 / 387, 100 527 / 448, 250 606 / 547, 700 981 / 983; hourly 20 1026 / 819, 100
    // 1054 / 939, 250 1204 / 1198.  Up to 512 workgroups, with the kernels of eight waves before these: faster for 40 monthly series alone (475 /
    // 443, whose fourth forward layer then joins: 264 workgroups), else level or up to 8 % slower.  (One limit for both directions; they
    // were not measured apart.)
    {
        int n = 0, total = 0;
        for (; n < std::min(L, kTogetherMost); ++n) {
            const LayerPlan &lp = pl.layer[n];
            const int here = pl.forward_groups(lp);
            if (lp.chains < lp.dil || total + here > together_groups) break;
            if (n == 0 && !lp.narrow_fwd) break;
            if (n > 0 && (!pl.layer[n - 1].narrow_fwd || pl.layer[n - 1].dil * (lp.narrow_fwd ? 1 : 4) > 64)) break;
            // (in front of the words lie the masks of a forecast)
            if ((size_t)L * pl.NB * 8 + (size_t)(1 + total + here) * kWordStride > PN * (size_t)pl.OP * 16) break;
            total += here;
        }
        pl.together_fwd = n > 1 ? n : 0;
        pl.together_groups = n > 1 ? total : 0;
        pl.together_words = pl.O + (size_t)L * pl.NB * 8;
    }
    // cell-state penalty: one partial sum per forward workgroup of every block's first layer, contiguous
    pl.cs_partial = ws.at;
    pl.n_cs_partial = 0;
    if (cfg.lambda_cs != 0.0f)
        for (int l = 0; l < L; ++l) {
            LayerPlan &lp = pl.layer[l];
            if (!lp.first_in_block) continue;
            lp.cs_partial = pl.cs_partial + pl.n_cs_partial;
            pl.n_cs_partial += pl.forward_groups(lp);
        }
    ws.take((size_t)pl.n_cs_partial);
    // block outputs: block 0's is the hidden state of its last layer
    for (int l = 0; l < L; ++l) {
        LayerPlan &lp = pl.layer[l];
        if (lp.last_in_block) {
            if (lp.block == 0) pl.blk_out[0] = lp.hid;
            else pl.blk_out[lp.block] = ws.take(PN * tileH);
        }
    }
    for (int l = 0; l < L; ++l) {
        LayerPlan &lp = pl.layer[l];
        // forward wiring
        if (l == 0) lp.xsrc = pl.X;
        else if (lp.first_in_block) lp.xsrc = pl.blk_out[lp.block - 1];
        else lp.xsrc = pl.layer[l - 1].hid;
        if (lp.last_in_block && lp.block >= 1) { lp.resid = pl.blk_out[lp.block - 1]; lp.out = pl.blk_out[lp.block]; }
        // backward wiring.  The output of block k feeds the first layer of every
        // later block through the residual sums, and the head: the gradient
        // arriving at its last layer is the sum of those input gradients.
        lp.gdst = pl.dx[l];
        lp.n_gsrc = 0;
        if (lp.last_in_block) {
            lp.gsrc[lp.n_gsrc++] = pl.gTop;
            for (int m = l + 1; m < L; ++m)
                if (pl.layer[m].first_in_block) lp.gsrc[lp.n_gsrc++] = pl.dx[m];
        } else {
            lp.gsrc[lp.n_gsrc++] = pl.dx[l + 1];
        }
    }
    if (cfg.n_blocks >= 3) pl.gsum = ws.take(PN * tileH);
    const HeadPack hp = head_pack_layout(pl);
    pl.head_fwd_pack = ws.take(hp.fwd_total);
    pl.head_bwd_pack = ws.take(hp.bwd_total);
    // Layers of the reverse pass in one launch, likewise.  (With three or more blocks a launch of its own sums gradients.)
    {
        int n = 0, total = 0;
        for (; cfg.n_blocks < 3 && n < std::min(L, kTogetherMost); ++n) {
            const LayerPlan &lp = pl.layer[n];
            const int here = pl.partial_groups(lp);
            if (!lp.split_bwd || lp.chains_bwd < lp.dil || lp.dil > 64 || total + here > together_groups) break;
            if ((size_t)(1 + total + here) * kWordStride > pl.head_bwd_pack - pl.head_fwd_pack + hp.bwd_total) break;
            total += here;
        }
        pl.together_bwd = n > 1 ? n : 0;
        pl.together_groups_bwd = n > 1 ? total : 0;
        pl.together_words_bwd = pl.head_fwd_pack;
    }
    pl.head_dw_stride = (pl.MO * pl.MA + pl.MA * pl.MA) * 256 + 4 * pl.OT + 4 * pl.HT;
    pl.head_dw_stride = (pl.head_dw_stride + 63) & ~63;
    pl.head_dw_partial = ws.take((size_t)pl.head_blocks * pl.head_dw_stride);
    pl.head_dw_reduced = ws.take((size_t)std::min(kReduceSplits, head_blocks) * pl.head_dw_stride);
    pl.total_floats = ws.at;
    return ESRNN_OK;
}

}  // namespace esrnn
