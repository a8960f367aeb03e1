// Register backward, radix 2, c64.
#include "gtt_bwd_reg.hpp"

GTT_BWD_REG_INSTANTIATE(c64, cf, 2)
