// First layers of the forward pass in one launch, the last one a 16-series layer (see lstm_forward_together.h).
#include "lstm_forward_together.h"

namespace esrnn {

hipError_t launch_lstm_forward_together_wide(const Plan &pl, const int32_t *lengths, const float *weights, float *ws,
                                             const ForwardMode &mode, hipStream_t st)
{
    return launch_together<kWideStash>(pl, lengths, weights, ws, mode, st);
}

}  // namespace esrnn
