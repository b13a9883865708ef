// Brick launches of the FP64 cycle (M = 1); brick.h has the kernels.
#include "brick.h"

namespace pfc {

void launch_brick64(hipStream_t s, const BrickArgs<double> &a, int kind, int sweeps, int form) {
    if (a.op.mob.phs) return launch_brick64_mob(s, a, kind, sweeps, form);
    brick_launch<double, BP_FAS, false, false>(s, a, kind, sweeps, form);
}

// ---- batched form: 4^3 boxes of many levels in one launch ----

template <int S, bool TAU>
__global__ __launch_bounds__((BrickPre<double, BP_FAS, false, false, 4, 4, 4, S, TAU, false, false>::TH),
                             (BrickPre<double, BP_FAS, false, false, 4, 4, 4, S, TAU, false, false>::WAVES)) void
kb_brick_pre(const BrickArgs<double> *__restrict__ segs, const BlockRef *__restrict__ blocks) {
    using K = BrickPre<double, BP_FAS, false, false, 4, 4, 4, S, TAU, false, false>;
    __shared__ typename K::Shared sm;
    const BlockRef b = blocks[blockIdx.x];
    const BrickArgs<double> a = segs[b.seg];
    K::run(a, (int)b.blk, sm, nullptr);
}

template <int S>
__global__ __launch_bounds__((BrickSweep<double, BP_FAS, false, false, 4, 4, 4, S, true, false, false, false>::TH),
                             (BrickSweep<double, BP_FAS, false, false, 4, 4, 4, S, true, false, false, false>::WAVES)) void
kb_brick_post(const BrickArgs<double> *__restrict__ segs, const BlockRef *__restrict__ blocks) {
    using K = BrickSweep<double, BP_FAS, false, false, 4, 4, 4, S, true, false, false, false>;
    __shared__ typename K::Shared sm;
    const BlockRef b = blocks[blockIdx.x];
    const BrickArgs<double> a = segs[b.seg];
    K::run(a, (int)b.blk, sm, nullptr);
}

void launch_batch_brick(hipStream_t s, int kind, int sweeps, bool first, const BrickArgs<double> *segs,
                        const BlockRef *blocks, unsigned count) {
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(count), dim3(threads), 0, s, segs, blocks);
    };
    using P1 = BrickPre<double, BP_FAS, false, false, 4, 4, 4, 1, false, false, false>;
    using P2 = BrickPre<double, BP_FAS, false, false, 4, 4, 4, 2, false, false, false>;
    using Q1 = BrickSweep<double, BP_FAS, false, false, 4, 4, 4, 1, true, false, false, false>;
    using Q2 = BrickSweep<double, BP_FAS, false, false, 4, 4, 4, 2, true, false, false, false>;
    if (kind == BRICK_POST)
        sweeps == 1 ? go(kb_brick_post<1>, Q1::TH) : go(kb_brick_post<2>, Q2::TH);
    else if (first)
        sweeps == 1 ? go(kb_brick_pre<1, true>, P1::TH) : go(kb_brick_pre<2, true>, P2::TH);
    else
        sweeps == 1 ? go(kb_brick_pre<1, false>, P1::TH) : go(kb_brick_pre<2, false>, P2::TH);
}

}  // namespace pfc
