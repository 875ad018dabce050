"""Several steps in one launch against the same steps one by one where part of
the lattice is not a number: the same sites are, and the others have the same
bits (no value stands in for a NaN in the comparison)."""
import pytest
import torch

from tests.parity_util import make_sim, random_state
from tests.test_gpu_overlap import CASES

pytestmark = pytest.mark.gpu

NAMES = sorted(n for n, p in CASES.items() if p.get("collision") != "elbm")


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16s"])
@pytest.mark.parametrize("name", NAMES)
def test_nan_sites_match_single_steps(name, storage):
    for nx, ny in ((70, 37), (181, 163)):
        p = dict(lattice="D2Q9", nx=nx, ny=ny, nu=2e-3, **CASES[name])
        f0 = random_state(p, 29, amp=0.1, kind=p.get("equilibrium", "poly"))
        f0[3, ny // 2, nx // 2] = float("nan")
        f0[7, 0, nx - 1] = float("nan")
        a, b = (make_sim(p, storage) for _ in range(2))
        for s in (a, b):
            s.set_populations(f0.cuda())
            if p.get("omega_field"):
                s.set_omega(torch.linspace(1.0, 1.9, nx * ny, device="cuda",
                                           dtype=torch.float64).view(ny, nx))
        for n in (4, 7):
            a.step(n)
            b.profile_step(n)
            fa, fb = a.populations(), b.populations()
            bad = fa.isnan()
            assert torch.equal(bad, fb.isnan()), (nx, ny, n)
            assert 0 < int(bad.sum()) < bad.numel()
            assert torch.equal(fa[~bad], fb[~bad]), (nx, ny, n)
            assert a.counters() == b.counters(), (nx, ny, n)
