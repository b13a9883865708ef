"""Device memory that a handle and a batch hold: what their fields need.

Per point of a level: the iterate, the right-hand side and I u (three fields each)
and phi^k, 10 values; 3 more on the finest level from 48^3 on and on every finest
level of a batch in paired sweeps (a second iterate), 6 more on a coarse level (a
second iterate, I r).  A batch keeps 5 fields of every instance beside them.  Tables:
the coarsest level's (0.2 MB) and the sums' partials (1.2 MB from 64^3 on).  The
allocator's pages are up to 2 MiB."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

PAGE = 2 << 20


def need(n, finest, coarse):
    b, first = 1.5e6 if n >= 64 else 0.4e6, True
    while n >= 3:
        b += 8 * (finest if first else coarse) * n ** 3
        first = False
        if n % 2:
            break
        n //= 2
    return b


def free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("n,count", [(16, 64), (32, 32), (48, 16), (64, 16), (96, 8), (128, 4)])
def test_handle(n, count):
    from paper_1611_06288_amd import Solver
    args = (n, n * math.pi / 4, 0.25, 0.1)
    Solver(*args).close()  # the device code is loaded
    before = free()
    hs = [Solver(*args) for _ in range(count)]
    held = (before - free()) / count
    limit = 1.05 * need(n, 10 if n < 48 else 13, 16)
    print(f"{n}^3: {held / 1e6:.2f} MB, limit {limit / 1e6:.2f} + a page", flush=True)
    assert held <= limit + PAGE
    for h in hs:
        h.close()
    assert free() >= before - 2 * PAGE


@pytest.mark.parametrize("sizes", [[16] * 64, [32] * 64, [48, 64, 96, 32] * 4])
def test_batch(sizes):
    from paper_1611_06288_amd.solver import Batch
    ps = [dict(n=n, L=n * math.pi / 4, eps=0.25, dt=0.1) for n in sizes]
    Batch(ps).close()
    before = free()
    b = Batch(ps)
    held = before - free()
    limit = sum(1.05 * need(n, 18, 16) for n in sizes)
    print(f"{len(sizes)} instances: {held / 1e6:.2f} MB, limit {limit / 1e6:.2f} MB + pages", flush=True)
    # a page for an instance's levels and its five fields of their own where those exceed one
    assert held <= limit + sum(PAGE * (1 + 5 * (8 * n ** 3 > PAGE // 4)) for n in sizes) + 4 * PAGE
    b.close()
