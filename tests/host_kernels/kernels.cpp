// The 16-series LSTM kernels as host functions (instrumented: every load and store is reported to host_kernels.cpp), in
// two parts that compile side by side.
#include <hip/hip_runtime.h>
void host_launch(void (*thread)(const void *), const void *args, dim3 grid, int threads);
#ifdef REVERSE
#include "lstm_backward_kernels.hip"
#include "lstm_backward_large_kernels.hip"
#else
#include "lstm_forward_kernels.hip"
#include "lstm_forward_residual_kernels.hip"
#endif
