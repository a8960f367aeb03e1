// Register backward, radix 16, f16.
#include "gtt_bwd_reg.hpp"

GTT_BWD_REG_INSTANTIATE(f16, f16, 16)
