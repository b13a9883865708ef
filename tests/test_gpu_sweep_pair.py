"""Two red-black sweeps in one launch (levels of at least 128^3, M = 1).

A V-cycle is compared with the cycle put together from the kernel-level entry
points, whose full sweeps are one launch each: the kernels share every point's
arithmetic, so the tolerance is equality.  128 and 192: several short plane
ranges per column, ragged at 192; 256: a coarse 128^3 level, which takes its
pre-sweeps from I u after the tau correction; odd sweep counts leave a single
sweep beside the pair.  (The stop test's halves and the time loop on pairs:
test_gpu_split_norm.py, test_gpu_timeloop.py.)
"""
import math

import pytest
import torch

from paper_1611_06288_amd import Solver, inputs
from test_gpu_brick import cycle_by_parts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nu,kw", [(128, (2, 2), {}), (192, (2, 2), {}), (128, (2, 1), {}),
                                     (128, (3, 3), {}), (128, (2, 2), dict(lin="picard")),
                                     (192, (2, 2), dict(scheme=1)), (256, (2, 2), {}),
                                     (256, (3, 4), {})])
def test_cycle_equals_kernel_level_cycle(n, nu, kw):
    s = Solver(n, n * math.pi / 4, 0.25, 0.5, nu1=nu[0], nu2=nu[1], **kw)
    g = inputs.rng(300 + n)
    rnd = lambda *shape: torch.from_numpy(g.uniform(-1, 1, shape)).cuda()  # noqa: E731
    phk, prev = 0.285 + 0.1 * rnd(n, n, n), 0.285 + 0.1 * rnd(n, n, n)
    f = s.source(prev, phk) + 0.01 * rnd(3, n, n, n)  # no structure between f and phi^k
    u = (torch.stack([phk, *s.init_guess(phk)]) + 0.05 * rnd(3, n, n, n)).contiguous()
    ref = u.clone()
    cycle_by_parts(s, ref, f, phk, nu)
    s.reset_coarse_cache()  # as the kernel-level coarsest solve
    got = u.clone()
    s.vcycle(got, f, phk)
    torch.cuda.synchronize()
    assert torch.isfinite(ref).all()
    assert torch.equal(got, ref)
