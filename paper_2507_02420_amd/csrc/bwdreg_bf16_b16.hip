// Register backward, radix 16, bf16.
#include "gtt_bwd_reg.hpp"

GTT_BWD_REG_INSTANTIATE(bf16, bf16, 16)
