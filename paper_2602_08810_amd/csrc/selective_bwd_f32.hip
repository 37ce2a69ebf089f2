// The backward kernels for float32 inputs, in an object of their own (they take as long to compile as those for bfloat16).
#define LRNNX_BWD_F32
#include "selective_bwd.hip"
