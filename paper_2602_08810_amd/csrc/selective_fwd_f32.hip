// The forward kernels for float32 inputs, in an object of their own (they take as long to compile as those for bfloat16).
#define LRNNX_FWD_F32
#include "selective_fwd.hip"
