"""The cycle loop whose decisions the device takes: what it enqueues behind and
ahead of a decision."""
import math
import time

import pytest
import torch

from paper_1611_06288_amd import inputs
from test_gpu_split_norm import MOB, host_loop, make, workload

pytestmark = pytest.mark.gpu


def least(f, reps=12):
    """Least time of f in seconds, the device idle before and after."""
    best = math.inf
    for _ in range(reps):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("n,nu,cycle,mobility", [(64, (4, 4), "F", None), (96, (2, 2), "V", None),
                                                 (96, (2, 2), "F", MOB), (128, (4, 4), "F", None)])
def test_a_step_without_cycles_costs_less_than_a_cycle(n, nu, cycle, mobility):
    """A constant density is a fixed point: the step tests it and returns.  Nothing
    of a cycle is launched, so the whole call takes less than one cycle does
    (pfc_fas_vcycle on the same handle)."""
    s = make(n, n * math.pi / 4, 0.25, 0.1, nu1=nu[0], nu2=nu[1], cycle=cycle, mobility=mobility)
    phi = torch.full((n, n, n), 0.2, dtype=torch.float64, device="cuda")
    mu, om = s.init_guess(phi)
    f, out = s.source(phi, phi), torch.empty_like(phi)
    u = torch.stack([phi, mu, om])
    infos = []
    step = least(lambda: infos.append(s.step(phi, phi, mu, om, out=out)[1]))
    assert all(i.cycles == 0 and i.status == 0 for i in infos)
    cyc = least(lambda: s.vcycle(u, f, phi))
    print(f"n={n} {nu} {cycle}: step {step * 1e6:.0f} us, cycle {cyc * 1e6:.0f} us", flush=True)
    assert step < 0.75 * cyc


@pytest.mark.parametrize("n,nu,cycle,kw", [(4, (2, 2), "V", {}), (16, (2, 2), "F", {}), (24, (1, 2), "V", {}), (48, (2, 2), "V", {}),
                                           (64, (3, 3), "V", {}), (64, (2, 2), "V", dict(mobility=MOB)),
                                           (128, (2, 2), "V", {}), (128, (3, 3), "V", {}),
                                           (128, (1, 1), "F", {}), (128, (1, 2), "V", {}),
                                           (128, (2, 2), "V", dict(mobility=MOB)),
                                           (128, (2, 2), "V", dict(scheme=1))])
@pytest.mark.parametrize("cap", [1, 2, 3, 400])
def test_steps_equal_the_host_loop(n, nu, cycle, kw, cap):
    """Two untimed steps (the second with phi_prev != phi_cur) against a host loop
    of single cycles and whole-level norms: fields, cycle counts, statuses and both
    norms bit for bit, converged and stopped by the cap; and once more on the same
    handles with a tolerance that the guess meets after no or one cycle."""
    p, phi = workload(n, 300 + n)
    mob = kw.get("mobility")
    for tol in (1e-10, None):
        if tol is None:  # between the norms before and after the first cycle
            tol = res0 * 0.9
        s = make(n, p.L, p.eps, p.dt, tol=tol, max_cycles=cap, nu1=nu[0], nu2=nu[1], cycle=cycle, **kw)
        ref = make(n, p.L, p.eps, p.dt, tol=tol, max_cycles=cap, nu1=nu[0], nu2=nu[1], cycle=cycle, **kw)
        mu, om = s.init_guess(phi)
        mu_h, om_h = mu.clone(), om.clone()
        prev, cur = phi, phi
        for _ in range(2):
            s.reset_coarse_cache()
            ref.reset_coarse_cache()
            u, c, status, res0, res = host_loop(ref, prev, cur, mu_h, om_h, tol, cap, mob)
            nxt, info = s.step(prev, cur, mu, om, raise_on_error=False)
            torch.cuda.synchronize()
            assert (info.cycles, info.status) == (c, status)
            assert info.res0 == res0 and info.res_final == res
            assert torch.equal(nxt, u[0]) and torch.equal(mu, u[1]) and torch.equal(om, u[2])
            prev, cur = cur, nxt
            mu_h, om_h = u[1].clone(), u[2].clone()
