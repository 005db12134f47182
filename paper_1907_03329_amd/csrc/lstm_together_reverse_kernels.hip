// Last layers of the reverse pass in one launch (see lstm_backward_together.h).
#include "lstm_backward_together.h"
