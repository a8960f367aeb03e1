// Register pass and filter, radix 2, i32.
#include "gtt_launch.hpp"
#include "gtt_pass_reg.hpp"

GTT_PASS_REG_INSTANTIATE(i32, uint32_t, 2)
