// Register pass and filter, radix 2, f32.
#include "gtt_launch.hpp"
#include "gtt_pass_reg.hpp"

GTT_PASS_REG_INSTANTIATE(f32, float, 2)
