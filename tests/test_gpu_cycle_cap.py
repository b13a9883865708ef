"""max_cycles up to the largest int (a caller's "no cap"): a step, the time loop,
the adjoint and a batch give what they give under a cap of 400, bit for bit."""
import math

import pytest
import torch

from paper_1611_06288_amd import inputs

pytestmark = pytest.mark.gpu

N, L = 16, 4 * math.pi


def everything(max_cycles, precision="fp64"):
    from paper_1611_06288_amd.solver import Batch, Solver
    phi = torch.from_numpy(0.2 + 0.05 * inputs.rng(31).uniform(-1, 1, (N, N, N))).cuda()
    s = Solver(N, L, 0.25, 0.1, max_cycles=max_cycles, precision=precision)
    mu, om = s.init_guess(phi)
    nxt, info = s.step(phi, phi, mu, om, raise_on_error=False)
    out = [nxt, mu, om]
    counts = [(info.cycles, info.status)]
    if precision == "fp64":
        prev, cur = phi.clone(), nxt.clone()
        infos = s.run(prev, cur, mu, om, 2, raise_on_error=False)
        counts += [(i.cycles, i.status) for i in infos]
        gc, gp, ge = torch.zeros_like(phi), torch.zeros_like(phi), torch.zeros(1, dtype=phi.dtype, device="cuda")
        counts.append(s.adjoint_step(phi, phi, nxt, phi - 0.2, gc, gp, ge, adj_tol=1e-10))
        b = Batch([dict(n=N, L=L, eps=0.25, dt=0.1)], max_cycles=max_cycles)
        b.init_state(0, phi)
        counts += [(i.cycles, i.status) for i in b.run(1, raise_on_error=False)[0]]
        out += [prev, cur, gc, gp, ge, *b.get_state(0)]
    return out, counts


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("cap", [2 ** 31 - 3, 2 ** 31 - 2, 2 ** 31 - 1])
def test_largest_caps(cap, precision):
    want, wc = everything(400, precision)
    got, gc = everything(cap, precision)
    print(wc, gc, flush=True)
    assert wc == gc and all(c[0] > 2 for c in wc if isinstance(c, tuple))
    assert all(torch.equal(a, b) for a, b in zip(want, got))
