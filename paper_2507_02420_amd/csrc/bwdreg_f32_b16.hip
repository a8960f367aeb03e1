// Register backward, radix 16, f32.
#include "gtt_bwd_reg.hpp"

GTT_BWD_REG_INSTANTIATE(f32, float, 16)
