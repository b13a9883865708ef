// Brick launches of the mixed form's FP32 correction cycle; brick.h has the
// kernels.
#include "brick.h"

namespace pfc {

void launch_brick32(hipStream_t s, const BrickArgs<float> &a, int kind, int sweeps, int form) {
    brick_launch<float, BP_FAS, true, false>(s, a, kind, sweeps, form);
}

}  // namespace pfc
