// Phase-encode normal operator, split factor 1.
#include "cart1d_split.h"

namespace pico {

hipError_t launch_cart1d_split1(int mode, const Cart1dArgs& a, hipStream_t s) {
  switch (a.ny) {
    case 96: return split_launch<1, ColPlan<12, 8>>(mode, a, s);
    case 256: return split_launch<1, ColPlan<16, 16>>(mode, a, s);
    case 384: return split_launch<1, ColPlan<24, 16>>(mode, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pico
