// Phase-encode normal operator, split factor 3.
#include "cart1d_split.h"

namespace pico {

hipError_t launch_cart1d_split3(int mode, const Cart1dArgs& a, hipStream_t s) {
  switch (a.ny) {
    case 96: return split_launch<3, ColPlan<8, 4>>(mode, a, s);
    case 192: return split_launch<3, ColPlan<8, 8>>(mode, a, s);
    case 288: return split_launch<3, ColPlan<12, 8>>(mode, a, s);
    case 384: return split_launch<3, ColPlan<16, 8>>(mode, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pico
