// IEEE half build of layer_slice.hip (storage and matrix-core operands; accumulation and statistics stay float32).
#define FF_LAYER_F16 1
#include "layer_slice.hip"
