"""pfc_energy_static takes every n in [4, 1024], the sizes that the solver does
not have (neither 2^k nor 3*2^k) among them: energies and mass against numpy.

Tolerance: a sum of P <= 4.1e6 terms passes through at most 16 additions in a
thread, 8 in a workgroup's tree, 64 + 8 over the workgroups, each term through
about 20 operations: 120 u < 1.4e-14 of the sum of the terms' magnitudes S, and
numpy's own below that.  1e-13 S."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1611_06288_amd import _lib, inputs

pytestmark = pytest.mark.gpu


def _sums(phi, prev, h, eps):
    """(F, modified F, mass) and the magnitudes of their terms."""
    def grad2(v):
        return sum(float(((np.roll(v, -1, ax) - v) ** 2).sum()) for ax in range(3)) / h ** 2
    lap = sum(np.roll(phi, 1, ax) + np.roll(phi, -1, ax) for ax in range(3)) - 6.0 * phi
    bulk = 0.25 * float((phi ** 4).sum()) + 0.5 * (1.0 - eps) * float((phi ** 2).sum())
    g, l2 = grad2(phi), 0.5 * float((lap ** 2).sum()) / h ** 4
    d = 0.5 * grad2(phi - prev) if prev is not None else 0.0
    F = bulk - g + l2
    h3 = h ** 3
    return (h3 * F, h3 * (F + d), h3 * float(phi.sum())), h3 * (abs(bulk) + g + l2 + d + float(np.abs(phi).sum()))


@pytest.mark.parametrize("n", [5, 7, 10, 33, 50, 100, 130, 160])
def test_sizes_without_a_solver(n):
    lib = _lib.lib()
    L, eps = 0.8 * n, 0.25
    g = inputs.rng(900 + n)
    phi = 0.285 + 0.1 * g.uniform(-1, 1, (n, n, n))
    prev = 0.285 + 0.1 * g.uniform(-1, 1, (n, n, n))
    dphi, dprev = torch.from_numpy(phi).cuda(), torch.from_numpy(prev).cuda()
    out3 = torch.full((3,), float("nan"), dtype=torch.float64, device="cuda")
    for pv, dpv in ((prev, dprev), (None, None)):
        print(f"n={n} prev={pv is not None}", flush=True)
        st = lib.pfc_energy_static(n, L, eps, C.c_void_p(dphi.data_ptr()),
                                   None if dpv is None else C.c_void_p(dpv.data_ptr()),
                                   C.c_void_p(out3.data_ptr()),
                                   C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == _lib.PFC_OK, lib.pfc_last_error(None)
        torch.cuda.synchronize()
        want, mag = _sums(phi, pv, L / n, eps)
        for a, b in zip(out3.cpu().tolist(), want):
            assert abs(a - b) <= 1e-13 * mag, (n, a, b)


@pytest.mark.parametrize("n", [128, 192, 256])
def test_plane_walk_equals_pfc_energy(n):
    """From 128^3 on the sums come from the walk over planes; the static form's are
    bitwise the handle's there too."""
    from paper_1611_06288_amd import Solver
    s = Solver(n, 0.8 * n, 0.25, 0.5)
    g = torch.Generator(device="cuda").manual_seed(n)
    phi, prev = (0.285 + 0.1 * torch.rand((n, n, n), generator=g, dtype=torch.float64, device="cuda")
                 for _ in range(2))
    out3 = torch.empty(3, dtype=torch.float64, device="cuda")
    for pv in (prev, None):
        want = s.energy(phi, pv)
        st = _lib.lib().pfc_energy_static(n, 0.8 * n, 0.25, C.c_void_p(phi.data_ptr()),
                                          None if pv is None else C.c_void_p(pv.data_ptr()),
                                          C.c_void_p(out3.data_ptr()),
                                          C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == _lib.PFC_OK
        assert out3.cpu().tolist() == list(want)
