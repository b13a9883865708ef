"""The autotuner's cache file: an entry stands for the launches that were timed,
which depend on the instance sizes and on the sweep counts."""
import json
import math

import pytest

pytestmark = pytest.mark.gpu

SIZES = [16, 32, 48]


def make(nu):
    from paper_1611_06288_amd.solver import Batch
    return Batch([dict(n=n, L=n * math.pi / 4, eps=0.2, dt=0.1) for n in SIZES], nu1=nu[0], nu2=nu[1])


def test_entries_are_per_sweep_count(tmp_path):
    path = tmp_path / "tiles.json"
    keys = set()
    for nu in ((2, 2), (1, 1), (0, 3)):
        b = make(nu)
        chosen = b.autotune(cache_path=path)
        new = set(json.loads(path.read_text())) - keys
        print(nu, chosen, sorted(new), flush=True)
        # every phase of its own, the tau phase where the cycle launches it
        phases = {k.split("|")[-1] for k in new}
        assert {"smooth", "resid_restrict", "prolong", "coarse_err"} <= phases
        assert ("tau" in phases) == (nu[0] == 0)
        keys |= new
        b.close()
        b = make(nu)
        assert b.autotune(cache_path=path) == chosen and set(json.loads(path.read_text())) == keys
        b.close()


def test_entries_without_sweep_counts_are_not_taken(tmp_path):
    """A file whose entries name the device, the sizes and the phase only: its
    choices are not adopted, its entries stay."""
    path = tmp_path / "tiles.json"
    b = make((2, 2))
    b.autotune(cache_path=path)
    b.close()
    entries = json.loads(path.read_text())
    parts = next(iter(entries)).split("|")
    prefix = "|".join(parts[:2])
    phases = ("smooth", "resid_restrict", "tau", "prolong", "coarse_err")
    old = {f"{prefix}|{p}": 106400 for p in phases}  # persistent, 64 threads, W = 64, Z = 1
    path.write_text("{\n" + ",\n".join(f'  "{k}": {v}' for k, v in old.items()) + "\n}\n")
    b = make((2, 2))
    b.autotune(cache_path=path)
    b.close()
    now = json.loads(path.read_text())
    assert all(now[k] == v for k, v in old.items())
    assert set(entries) <= set(now) and not set(entries) & set(old)
