"""Two red-black sweeps in one launch (levels of at least 128^3).

A V-cycle is compared with the cycle put together from the kernel-level entry
points, whose full sweeps are one launch each: the kernels share every point's
arithmetic, so the tolerance is equality.  128 and 192: several short plane
ranges per column, ragged at 192; 256: a coarse 128^3 level, which takes its
pre-sweeps from I u after the tau correction; odd sweep counts leave a single
sweep beside the pair.  (The stop test's halves and the time loop on pairs:
test_gpu_split_norm.py, test_gpu_timeloop.py.)

The batched form's small depths (bricks of 12^3 and 16^3, tails of 8^3 and 6^3
of both sizes in one launch) run in the same test.

The batched pairs take 32 x 16 boxes: one step of a batch against single steps
(bricks up to 96^3), bit for bit with the norms; 48-point rows leave half a
box, a tolerance met by one instance long before the others masks it.
"""
import math

import pytest
import torch

from paper_1611_06288_amd import Solver, inputs
from paper_1611_06288_amd.solver import Batch
from test_gpu_brick import cycle_by_parts

pytestmark = pytest.mark.gpu

MOB = (1.0, 0.0, -1.0, 0.05)


@pytest.mark.parametrize("n,nu,kw", [(128, (2, 2), {}), (192, (2, 2), {}), (128, (2, 1), {}),
                                     (128, (3, 3), {}), (128, (2, 2), dict(lin="picard")),
                                     (192, (2, 2), dict(scheme=1)), (256, (2, 2), {}),
                                     (256, (3, 4), {}), (128, (2, 2), dict(mobility=MOB)),
                                     (192, (2, 2), dict(mobility=MOB)), (256, (2, 2), dict(mobility=MOB))])
def test_cycle_equals_kernel_level_cycle(n, nu, kw):
    s = Solver(n, n * math.pi / 4, 0.25, 0.5, nu1=nu[0], nu2=nu[1], **kw)
    g = inputs.rng(300 + n)
    rnd = lambda *shape: torch.from_numpy(g.uniform(-1, 1, shape)).cuda()  # noqa: E731
    phk, prev = 0.285 + 0.1 * rnd(n, n, n), 0.285 + 0.1 * rnd(n, n, n)
    f = s.source(prev, phk) + 0.01 * rnd(3, n, n, n)  # no structure between f and phi^k
    u = (torch.stack([phk, *s.init_guess(phk)]) + 0.05 * rnd(3, n, n, n)).contiguous()
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


@pytest.mark.parametrize("sizes,kw", [((32,), {}), ((48, 32, 64), {}), ((96, 48, 128, 64, 32), {}),
                                      ((64, 96, 48), dict(cycle="F")), ((48, 64), dict(lin="picard")), ((16, 24, 12), {}), ((24, 24), dict(cycle="F")),
                                      ((32, 12, 16, 48), dict(nu1=1, nu2=2)),
                                      ((32, 48, 96), dict(max_cycles=3))])
def test_batch_step_equals_single_steps(sizes, kw):
    tol = 1e-14 if "max_cycles" in kw else 1e-10
    params = [dict(n=n, L=n * math.pi / 4, eps=0.1 + 0.03 * i, dt=0.1 if i else 0.01)
              for i, n in enumerate(sizes)]
    g = inputs.rng(11)
    fields = [torch.from_numpy(0.2 + 0.05 * g.uniform(-1, 1, (n, n, n))).cuda() for n in sizes]
    b = Batch(params, tol=tol, **kw)
    for i, f in enumerate(fields):
        b.init_state(i, f)
    infos = b.run(1, raise_on_error=False)
    for i, (p, f) in enumerate(zip(params, fields)):
        s = Solver(p["n"], p["L"], p["eps"], p["dt"], tol=tol, **kw)
        mu, om = s.init_guess(f)
        nxt, info = s.step(f, f, mu, om, raise_on_error=False)
        _, phi, bmu, bom = b.get_state(i)
        torch.cuda.synchronize()
        x = infos[i][0]
        assert (x.cycles, x.status, x.res0, x.res_final) == (info.cycles, info.status, info.res0,
                                                             info.res_final)
        assert torch.equal(phi, nxt) and torch.equal(bmu, mu) and torch.equal(bom, om)
