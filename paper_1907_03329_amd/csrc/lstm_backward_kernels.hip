// 16-series reverse LSTM kernel, hidden sizes up to 40 (see lstm_backward.h).
#include "lstm_backward.h"

namespace esrnn {

hipError_t launch_lstm_backward_three_term(const Plan &pl, int layer, const LstmBwdSources &src, const int32_t *lengths,
                                           float *ws, hipStream_t st)
{
    const LayerPlan &lp = pl.layer[layer];
    if (pl.HT > 10) return launch_lstm_backward_three_term_large(pl, layer, src, lengths, ws, st);
    const LstmBwdArgs a = backward_args(pl, layer, src, lengths, ws);
#define X(HT_, KXT_) if constexpr (HT_ <= 10) if (pl.HT == HT_ && lp.KXT == KXT_) return run_bwd<HT_, KXT_>(a, lp.chains_bwd, st);
    ESRNN_LSTM_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace esrnn
