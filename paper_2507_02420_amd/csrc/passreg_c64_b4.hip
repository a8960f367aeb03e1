// Register pass and filter, radix 4, c64.
#include "gtt_launch.hpp"
#include "gtt_pass_reg.hpp"

GTT_PASS_REG_INSTANTIATE(c64, cf, 4)
