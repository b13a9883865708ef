"""FP32 sweeps two per launch (levels of 256^3 and larger) with a single sweep left
over on one or both sides of the descent, and as a coarse level's first sweeps
(512^3, fields without a period): the mixed step against the FP64 step.

Bar: the mixed form's for cycles that smooth less than V(2,2), 1e-11 after the same
number of cycles, at most two cycles more than FP64 takes."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nu,cycle", [(256, (3, 2), "V"), (256, (2, 3), "V"), (256, (5, 4), "F"),
                                        (512, (2, 2), "V"), (512, (3, 2), "V")])
def test_mixed_step_equals_fp64_step(n, nu, cycle):
    from paper_1611_06288_amd import Solver
    g = torch.Generator(device="cuda").manual_seed(n + nu[0])
    phi = 0.2 + 0.1 * (torch.rand((n, n, n), generator=g, dtype=torch.float64, device="cuda") - 0.5)
    args = (n, n * math.pi / 4, 0.25, 0.1)
    kw = dict(nu1=nu[0], nu2=nu[1], cycle=cycle)
    m = Solver(*args, precision="mixed", **kw)
    mu0, om0 = m.init_guess(phi)
    mu, om = mu0.clone(), om0.clone()
    got, im = m.step(phi, phi, mu, om)
    m.close()
    f = Solver(*args, max_cycles=400, **kw)
    mu_f, om_f = mu0.clone(), om0.clone()
    want, i_f = f.step(phi, phi, mu_f, om_f)
    if im.cycles != i_f.cycles:
        f.close()
        f = Solver(*args, tol=1e-300, max_cycles=im.cycles, **kw)
        mu_f, om_f = mu0.clone(), om0.clone()
        want, _ = f.step(phi, phi, mu_f, om_f, raise_on_error=False)
    f.close()
    err = max(float((a - b).abs().max()) for a, b in ((got, want), (mu, mu_f), (om, om_f)))
    print(f"{n}^3 {nu} {cycle}: cycles {im.cycles}, FP64 {i_f.cycles}, difference {err:.2e}", flush=True)
    assert im.status == 0 and im.res_final <= 1e-10
    assert i_f.cycles <= im.cycles <= i_f.cycles + 2
    assert err <= 1e-11
