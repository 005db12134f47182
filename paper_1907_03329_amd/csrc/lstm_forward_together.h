// First layers of the network in one launch, each behind the one below (see lstm_together.h): 4-series layers, the last one
// possibly a 16-series one.  The kernel template and its launcher, included by one translation unit per kind of last layer.
//
// What it gives (a launch a layer -> one launch), steps: at the rule in plan.cpp; the first two layers of 512 hourly series 400 -> 333 us, of 501 monthly
// ones 171 -> 136, forecasts of 512 hourly ones 470 -> 382.  What bounds it is the first layer's chain; at the end every layer adds what a
// store, a look and a load past the caches take and a few positions of its own, some 5 us.  A first layer alone in this launch, without
// counts, takes 105 us for 512 monthly series and 90 in a launch of its own (quarters of a tile on the same XCD there), 275 for 512 hourly ones;
// beside it the 16-series layer's stores cost another 30 and 50 us.
#pragma once

#include "lstm_forward.h"
#include "lstm_narrow_fwd.h"

namespace esrnn {

namespace {

struct FwdTogetherArgs {
    NarrowFwdArgs narrow[kTogetherMost];
    LstmFwdArgs wide;                   // of the last layer, if that is a 16-series one
    Places places;
};

// kind of the last layer
enum { kAllNarrow, kWideStash, kWideNoStash };

template <int HT, int KXT, bool CP, int KIND>
__global__ void __launch_bounds__(2 * kNT, KIND == kAllNarrow ? 4 : 2) lstm_forward_together_kernel(FwdTogetherArgs t)
{
    __shared__ unsigned ticket;
    const Place at = draw_place(t.places, &ticket);
    const int l = at.layer, d = t.places.d[l], bt = at.bt, q = at.q, chain = at.chain;
    const bool wide = KIND != kAllNarrow && l == t.places.layers - 1;
    const Progress progress = progress_of(t.places, at, l - 1);
    // A count is a store past the caches to a line that others look at, and the next request of x waits behind it.  Every fourth
    // position where a 16-series layer follows (forward pass of 512 hourly series 713 -> 699 us, 501 monthly 304 -> 300), every one
    // where 4-series layers do (64 monthly series 172.6 us, 179.3 with every fourth).
    constexpr int kCounted = KIND == kAllNarrow ? 1 : kInputGroup;
    if (l == 0) {
        lstm_forward_narrow_body<HT, KXT, CP, false, kFirst, kCounted>(t.narrow[0], bt, q, chain, d, progress);
    } else if (wide) {
        if constexpr (KIND != kAllNarrow) {
            constexpr bool stash = KIND == kWideStash;
            if (t.wide.out) lstm_forward_body<HT, HT, 8, CP, true, stash, true>(t.wide, bt, chain, d, progress);
            else lstm_forward_body<HT, HT, 8, CP, false, stash, true>(t.wide, bt, chain, d, progress);
        }
    } else if (t.narrow[l].out) {
        lstm_forward_narrow_body<HT, HT, CP, true, kLater>(t.narrow[l], bt, q, chain, d, progress);
    } else {
        lstm_forward_narrow_body<HT, HT, CP, false, kLater>(t.narrow[l], bt, q, chain, d, progress);
    }
}

template <int KIND>
hipError_t launch_together(const Plan &pl, const int32_t *lengths, const float *weights, float *ws, const ForwardMode &mode, hipStream_t st)
{
    FwdTogetherArgs t{};
    Places &places = t.places;
    places.layers = pl.together_fwd;
    places.NB = pl.NB;
    places.words = reinterpret_cast<unsigned *>(ws + pl.together_words);
    for (int l = 0; l < places.layers; ++l) {
        const LayerPlan &lp = pl.layer[l];
        places.d[l] = lp.dil;
        places.quarters[l] = lp.narrow_fwd ? 4 : 1;
        places.first[l + 1] = places.first[l] + pl.forward_groups(lp);
        if (lp.narrow_fwd) t.narrow[l] = narrow_forward_args(pl, l, lengths, weights, ws);
        else t.wide = forward_args(pl, l, lengths, ws, mode);
    }
    const bool cp = pl.cfg.lambda_cs != 0.0f;
    const int blocks = places.first[places.layers];
#define X(HT_, KXT_)                                                                                                            \
    if (pl.HT == HT_ && pl.layer[0].KXT == KXT_) {                                                                              \
        if (cp && KIND != kWideNoStash) lstm_forward_together_kernel<HT_, KXT_, KIND != kWideNoStash, KIND><<<blocks, 2 * kNT, 0, st>>>(t);        \
        else lstm_forward_together_kernel<HT_, KXT_, false, KIND><<<blocks, 2 * kNT, 0, st>>>(t);                               \
        return hipGetLastError();                                                                                               \
    }
    ESRNN_LSTM_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace esrnn
