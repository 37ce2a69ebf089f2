// The complex forward kernels for float32 inputs, in an object of their own (they take as long to compile as those for bfloat16).
#define LRNNX_CFWD_F32
#include "selective_cplx_fwd.hip"
