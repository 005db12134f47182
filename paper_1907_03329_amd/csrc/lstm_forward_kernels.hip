// 16-series forward LSTM kernel, layers without a residual output (see lstm_forward.h).
#include "lstm_forward.h"

namespace esrnn {

hipError_t launch_lstm_forward(const Plan &pl, int layer, const int32_t *lengths, const float *weights, float *ws,
                               const ForwardMode &mode, hipStream_t st)
{
    const LayerPlan &lp = pl.layer[layer];
    if (lp.narrow_fwd) return launch_lstm_forward_narrow(pl, layer, lengths, weights, ws, st);
    if (lp.out) return launch_lstm_forward_residual(pl, layer, lengths, ws, mode, st);
    const LstmFwdArgs a = forward_args(pl, layer, lengths, ws, mode);
#define X(HT_, KXT_) if (pl.HT == HT_ && lp.KXT == KXT_) return run_fwd<HT_, KXT_, false>(a, lp.chains, st);
    ESRNN_LSTM_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace esrnn
