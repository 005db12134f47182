// First layers of the forward pass in one launch, the last one a 16-series layer, no reverse pass to come (see lstm_forward_together.h).
#include "lstm_forward_together.h"

namespace esrnn {

hipError_t launch_lstm_forward_together_forecast(const Plan &pl, const int32_t *lengths, const float *weights, float *ws,
                                             const ForwardMode &mode, hipStream_t st)
{
    return launch_together<kWideNoStash>(pl, lengths, weights, ws, mode, st);
}

}  // namespace esrnn
