// Launches of the two-level tail (tail.h).
#include "tail.h"

namespace pfc {

template <typename T, int PH, bool DELTA, bool MOB, int N>
__global__ __launch_bounds__((Tail<T, PH, DELTA, MOB, N>::kThreads)) void k_tail(TailArgs<T> a) {
    __shared__ typename Tail<T, PH, DELTA, MOB, N>::Shared sm;
    if (gate_closed(a.op.gate)) return;
    Tail<T, PH, DELTA, MOB, N> t(a, sm);
    t.run();
}

template <typename T, int PH, bool DELTA, bool MOB>
static void tail_launch(hipStream_t s, const TailArgs<T> &a) {
    if (a.op.lay.n == 8)
        hipLaunchKernelGGL((k_tail<T, PH, DELTA, MOB, 8>), dim3(1), dim3(Tail<T, PH, DELTA, MOB, 8>::kThreads), 0,
                           s, a);
    else
        hipLaunchKernelGGL((k_tail<T, PH, DELTA, MOB, 6>), dim3(1), dim3(Tail<T, PH, DELTA, MOB, 6>::kThreads), 0,
                           s, a);
}

void launch_tail64(hipStream_t s, const TailArgs<double> &a) {
    if (a.op.mob.phs)
        tail_launch<double, BP_FAS, false, true>(s, a);
    else
        tail_launch<double, BP_FAS, false, false>(s, a);
}

void launch_tail32(hipStream_t s, const TailArgs<float> &a) { tail_launch<float, BP_FAS, true, false>(s, a); }

void launch_tail_adj(hipStream_t s, const TailArgs<double> &a) {
    tail_launch<double, BP_ADJ, false, false>(s, a);
}

}  // namespace pfc
