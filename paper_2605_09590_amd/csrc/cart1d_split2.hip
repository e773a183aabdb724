// Phase-encode normal operator, split factor 2.
#include "cart1d_split.h"

namespace pico {

hipError_t launch_cart1d_split2(int mode, const Cart1dArgs& a, hipStream_t s) {
  switch (a.ny) {
    case 64: return split_launch<2, ColPlan<8, 4>>(mode, a, s);
    case 96: return split_launch<2, ColPlan<8, 6>>(mode, a, s);
    case 128: return split_launch<2, ColPlan<8, 8>>(mode, a, s);
    case 160: return split_launch<2, ColPlan<10, 8>>(mode, a, s);
    case 192: return split_launch<2, ColPlan<12, 8>>(mode, a, s);
    case 256: return split_launch<2, ColPlan<16, 8>>(mode, a, s);
    case 288: return split_launch<2, ColPlan<12, 12>>(mode, a, s);
    case 320: return split_launch<2, ColPlan<16, 10>>(mode, a, s);
    case 384: return split_launch<2, ColPlan<16, 12>>(mode, a, s);
    case 512: return split_launch<2, ColPlan<16, 16>>(mode, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pico
