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

// Both sizes in one launch (the smaller's spare threads only meet the barriers).
__global__ __launch_bounds__(256) void kb_tail(const TailArgs<double> *__restrict__ segs, int fcycle) {
    using T8 = Tail<double, BP_FAS, false, false, 8, 256>;
    using T6 = Tail<double, BP_FAS, false, false, 6, 256>;
    __shared__ union Both {
        typename T8::Shared a;
        typename T6::Shared b;
        __device__ Both() {}
    } sm;
    TailArgs<double> a = segs[blockIdx.x];
    if (gate_closed(a.op.gate)) return;
    a.fcycle = fcycle;
    if (a.op.lay.n == 8) {
        T8 t(a, sm.a);
        t.run();
    } else {
        T6 t(a, sm.b);
        t.run();
    }
}

void launch_batch_tail(hipStream_t s, const TailArgs<double> *segs, int nseg, int fcycle) {
    hipLaunchKernelGGL(kb_tail, dim3(nseg), dim3(256), 0, s, segs, fcycle);
}

}  // namespace pfc
