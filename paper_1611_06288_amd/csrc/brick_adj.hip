// Brick launches of the adjoint's linear cycle; brick.h has the kernels.
#include "brick.h"

namespace pfc {

void launch_brick_adj(hipStream_t s, const BrickArgs<double> &a, int kind, int sweeps, int form) {
    brick_launch<double, BP_ADJ, false, false>(s, a, kind, sweeps, form);
}

}  // namespace pfc
