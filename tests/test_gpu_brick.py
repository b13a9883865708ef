"""One V-cycle against the same cycle put together on the host from the
kernel-level entry points (half-sweep kernels, thread-per-point residual,
8-child means, interpolation, coarsest solve), bit for bit.

The cycle runs levels of 12^3 to 96^3 as one launch on either side of the
descent (boxes with halos in LDS) and the 8^3 (6^3) level with the coarsest
one in a single launch; the entry points run one kernel per operation.  The
kernels share every point's arithmetic, so the tolerance is equality.  Sizes:
both box sizes, the smallest level of each, odd multiples of the box (24, 48,
96) where the halo wraps round the grid, and levels below a larger finest
level.
"""
import math

import numpy as np
import pytest
import torch

from paper_1611_06288_amd import Solver, inputs

pytestmark = pytest.mark.gpu

MOB = (1.0, 0.0, -1.0, 0.05)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def cycle_by_parts(s, u, f, phk, nu):
    """One V(nu1, nu2) cycle in place on u, from kernel-level calls."""
    last = len(s.levels) - 1
    phks = [phk]
    for l in range(last):
        phks.append(s.restrict(l, phks[-1], 1))

    def cyc(l, u, f):
        if l == last:
            s.coarse_solve(u, f, phks[l])
            return
        for _ in range(nu[0]):
            s.smooth(l, 2, u, f, phks[l])
        r, _ = s.residual(l, u, f, phks[l])
        ub, rr = s.restrict(l, u, 3), s.restrict(l, r, 3)
        minus_n, _ = s.residual(l + 1, ub, torch.zeros_like(ub), phks[l + 1])
        fc = rr - minus_n
        v = ub.clone()
        cyc(l + 1, v, fc)
        s.prolong_add(l, v, ub, u, 3)
        for _ in range(nu[1]):
            s.smooth(l, 2, u, f, phks[l])

    cyc(0, u, f)


CASES = [(n, (2, 2), {}) for n in (12, 16, 24, 32, 48, 64, 96, 128, 192)]
CASES += [(n, nu, {}) for n in (16, 24, 64) for nu in ((1, 1), (1, 2), (2, 1))]
CASES += [(24, (2, 2), dict(lin="picard")), (64, (2, 2), dict(lin="picard")),
          (48, (2, 2), dict(scheme=1)), (128, (2, 2), dict(scheme=1))]
CASES += [(n, nu, dict(mobility=MOB)) for n, nu in ((16, (2, 2)), (24, (1, 2)), (48, (2, 2)),
                                                    (64, (2, 1)), (128, (2, 2)))]


@pytest.mark.parametrize("n,nu,kw", CASES)
def test_cycle_equals_kernel_level_cycle(n, nu, kw):
    L, eps, dt = n * math.pi / 4, 0.25, 0.5
    s = Solver(n, L, eps, dt, nu1=nu[0], nu2=nu[1], **kw)
    g = inputs.rng(900 + n)
    phk = dev(0.285 + 0.1 * g.uniform(-1, 1, (n, n, n)))
    prev = dev(0.285 + 0.1 * g.uniform(-1, 1, (n, n, n)))
    f = s.source(prev, phk)
    f = f + dev(0.01 * g.uniform(-1, 1, (3, n, n, n)))  # no structure between f and phi^k
    u = torch.stack([phk, *s.init_guess(phk)])
    u = (u + dev(0.05 * g.uniform(-1, 1, (3, n, n, n)))).contiguous()
    if "mobility" in kw:
        s.set_phistar(0, 1.5 * phk - 0.5 * prev)
    ref = u.clone()
    cycle_by_parts(s, ref, f, phk, nu)
    s.reset_coarse_cache()  # as the kernel-level coarsest solve
    got = u.clone()
    s.vcycle(got, f, phk)
    torch.cuda.synchronize()
    assert torch.isfinite(ref).all()
    assert torch.equal(got, ref)
