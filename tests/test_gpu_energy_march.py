"""Energies on sizes whose parts are walked in z (128^3 and larger) against the
same sums in numpy FP64.

Each of the six sums adds n^3 terms, all but the mass's non-negative, in a tree
over a few thousand parts of at most a few thousand terms: relative error below
(64 + 8 + 64 + 8) roundings plus a handful per term, under 200 * 1.1e-16.  The
energy combines four of them with cancellation (the gradient term enters with a
minus), so the bound is taken on the sum of their magnitudes: 5e-14.
96: the largest size below; 128 and 192: one and two passes, the second ragged; 256: four whole ones."""
import numpy as np
import pytest
import torch

from paper_1611_06288_amd import Solver, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [96, 128, 192, 256])
@pytest.mark.parametrize("with_prev", [False, True])
def test_energy_equals_plain_sums(n, with_prev):
    h, eps = 0.7, 0.2
    g = inputs.rng(17 + n)
    phi = 0.2 + 0.3 * g.uniform(-1, 1, (n, n, n))
    prev = phi + 0.05 * g.uniform(-1, 1, (n, n, n)) if with_prev else None
    grad2 = lambda v: sum(np.sum(((np.roll(v, -1, a) - v) / h) ** 2) for a in range(3))  # noqa: E731
    lap = sum(np.roll(phi, 1, a) + np.roll(phi, -1, a) for a in range(3)) - 6.0 * phi
    terms = [0.25 * np.sum(phi ** 4), 0.5 * (1 - eps) * np.sum(phi ** 2), -grad2(phi),
             0.5 * np.sum((lap / h ** 2) ** 2)]
    extra = 0.5 * grad2(phi - prev) if with_prev else 0.0
    F, Fm, mass = Solver(n, n * h, eps, 0.1).energy(
        torch.from_numpy(phi).cuda(), torch.from_numpy(prev).cuda() if with_prev else None)
    size = h ** 3 * sum(abs(t) for t in terms)
    assert abs(F - h ** 3 * sum(terms)) <= 5e-14 * size
    assert abs(Fm - h ** 3 * (sum(terms) + extra)) <= 5e-14 * (size + h ** 3 * extra)
    assert abs(mass - h ** 3 * np.sum(phi)) <= 5e-14 * h ** 3 * np.sum(np.abs(phi))
