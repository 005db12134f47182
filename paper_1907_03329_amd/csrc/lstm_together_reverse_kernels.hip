// Last layers of the reverse pass, the first ones of the network, in one launch, each behind the one above (see
// lstm_together.h): 4-series layers with twelve waves a workgroup.
//
// What it gives (a launch a layer -> one launch): 16 quarterly series, four layers 103 us and three gaps between launches -> 69 us,
// now 50 us.  What bounds it is the first layer's chain, 31 us, and per layer the positions between an input
// gradient and its count, a store, a look and a load past the caches.

#include "lstm_narrow_bwd.h"

namespace esrnn {

namespace {

struct BwdTogetherArgs {
    NarrowBwdArgs narrow[kTogetherMost];    // in the order in which they run: the network's first layer comes last
    Places places;
};

template <int HT, int KXT, bool CP>
__global__ void __launch_bounds__(narrow_bwd_threads(true)) lstm_backward_together_kernel(BwdTogetherArgs t)
{
    using Last = NarrowBwdLds<HT, KXT, true, kLast>;
    using Later = NarrowBwdLds<HT, HT, true, kLater>;
    // (arrays next to each other for both kinds of layers do not fit)
    constexpr size_t bytes = std::max(Last::bytes, Later::bytes);
    __shared__ __align__(16) char lds[bytes];
    __shared__ unsigned ticket;
    alone_on_compute_unit<(int)bytes>();
    const Place at = draw_place(t.places, &ticket);
    const Progress progress = progress_of(t.places, at, at.layer - 1);
    const int d = t.places.d[at.layer];
    if (at.layer == t.places.layers - 1)
        lstm_backward_narrow_body<HT, KXT, CP, true, kLast>(t.narrow[at.layer], Last::in(lds), at.bt, at.q, at.chain, d, progress);
    else
        lstm_backward_narrow_body<HT, HT, CP, true, kLater>(t.narrow[at.layer], Later::in(lds), at.bt, at.q, at.chain, d, progress);
}

}  // namespace

hipError_t launch_lstm_backward_together(const Plan &pl, const int32_t *lengths, float *ws, hipStream_t st)
{
    BwdTogetherArgs t{};
    Places &places = t.places;
    places.layers = pl.together_bwd;
    places.NB = pl.NB;
    places.words = reinterpret_cast<unsigned *>(ws + pl.together_words_bwd);
    for (int i = 0; i < places.layers; ++i) {
        const int l = places.layers - 1 - i;
        const LayerPlan &lp = pl.layer[l];
        places.d[i] = lp.dil;
        places.quarters[i] = 4;
        places.first[i + 1] = places.first[i] + pl.partial_groups(lp);
        t.narrow[i] = narrow_backward_args(pl, l, lengths, ws);
    }
    const int blocks = places.first[places.layers];
    const bool cp = pl.cfg.lambda_cs != 0.0f;
#define X(HT_, KXT_)                                                                                                            \
    if (pl.HT == HT_ && pl.layer[0].KXT == KXT_) {                                                                              \
        if (cp) lstm_backward_together_kernel<HT_, KXT_, true><<<blocks, narrow_bwd_threads(true), 0, st>>>(t);                                  \
        else lstm_backward_together_kernel<HT_, KXT_, false><<<blocks, narrow_bwd_threads(true), 0, st>>>(t);                                    \
        return hipGetLastError();                                                                                               \
    }
    ESRNN_LSTM_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace esrnn
