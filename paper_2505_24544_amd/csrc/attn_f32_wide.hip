// The float attention of heads of 68 .. 128 channels, compiled apart: with six or eight accumulators of 32 x 32 and the operands of
// two products a wave holds 310 - 490 registers, and only while the matrix instructions write accumulation registers are the vector
// registers left to the operands (build.py).
#include "attn_f32.h"

namespace beagle {
void launch_attn_fwd_f32_wide(const AttnArgs& a, hipStream_t s) { launch_fwd<3>(a, s); }
void launch_attn_bwd_f32_wide(const AttnArgs& a, hipStream_t s) { launch_bwd<3>(a, s); }
}  // namespace beagle
