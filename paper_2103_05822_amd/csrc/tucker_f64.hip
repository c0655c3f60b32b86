// The streaming kernels of tucker.hip for complex128.
#define TUCKFMM_STREAM_F64
#include "tucker.hip"
