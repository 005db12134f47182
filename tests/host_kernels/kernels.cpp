// The kernels as host functions (instrumented: every load and store is reported to host_kernels.cpp), in parts that compile
// side by side.
#include <hip/hip_runtime.h>
#include PART
