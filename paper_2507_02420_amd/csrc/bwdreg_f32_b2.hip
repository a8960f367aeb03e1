// Register backward, radix 2, f32.
#include "gtt_bwd_reg.hpp"

GTT_BWD_REG_INSTANTIATE(f32, float, 2)
