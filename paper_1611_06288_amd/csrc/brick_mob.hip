// Brick launches of the FP64 cycle with variable mobility (phi* as a fourth
// LDS field); brick.h has the kernels.
#include "brick.h"

namespace pfc {

void launch_brick64_mob(hipStream_t s, const BrickArgs<double> &a, int kind, int sweeps, int form) {
    brick_launch<double, BP_FAS, false, true>(s, a, kind, sweeps, form);
}

}  // namespace pfc
