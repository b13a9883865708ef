// Brick launches of the FP64 cycle (M = 1); brick.h has the kernels.
#include "brick.h"

namespace pfc {

void launch_brick64(hipStream_t s, const BrickArgs<double> &a, int kind, int sweeps, int form) {
    if (a.op.mob.phs) return launch_brick64_mob(s, a, kind, sweeps, form);
    brick_launch<double, BP_FAS, false, false>(s, a, kind, sweeps, form);
}

}  // namespace pfc
