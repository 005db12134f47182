// 16-series forward LSTM kernel, last layer of a residual block: also writes block input + hidden state (see
// lstm_forward.h).
#include "lstm_forward.h"

namespace esrnn {

hipError_t launch_lstm_forward_residual(const Plan &pl, int layer, const int32_t *lengths, float *ws, const ForwardMode &mode,
                                        hipStream_t st)
{
    const LayerPlan &lp = pl.layer[layer];
    const LstmFwdArgs a = forward_args(pl, layer, lengths, ws, mode);
    // (every layer but the first one takes the hidden state of another layer as its input)
#define X(HT_) if (pl.HT == HT_ && lp.KXT == HT_) return run_fwd<HT_, HT_, true>(a, lp.chains, st);
    X(2) X(8) X(10) X(13) X(16)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace esrnn
