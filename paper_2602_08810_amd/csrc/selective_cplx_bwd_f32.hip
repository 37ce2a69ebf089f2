// The complex backward kernels for float32 inputs, in an object of their own (they take as long to compile as those for bfloat16).
#define LRNNX_CBWD_F32
#include "selective_cplx_bwd.hip"
