// First layers of the forward pass in one launch, 4-series layers only (see lstm_forward_together.h).
#include "lstm_forward_together.h"

namespace esrnn {

hipError_t launch_lstm_forward_together(const Plan &pl, const int32_t *lengths, const float *weights, float *ws, const ForwardMode &mode,
                                        hipStream_t st)
{
    if (pl.layer[pl.together_fwd - 1].narrow_fwd) return launch_together<kAllNarrow>(pl, lengths, weights, ws, mode, st);
    // (with the cell-state penalty there is only the general kernel: it writes the stash and computes every class)
    if (mode.stash || pl.cfg.lambda_cs != 0.0f) return launch_lstm_forward_together_wide(pl, lengths, weights, ws, mode, st);
    return launch_lstm_forward_together_forecast(pl, lengths, weights, ws, mode, st);
}

}  // namespace esrnn
