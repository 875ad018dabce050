"""Many steps of a short D1Q3 lattice in one launch (lbm_step) against the
same steps one by one through the step and selection kernels
(lbm_profile_step): the same site arithmetic and an exact selection, so the
same bits, selections and counters.  Sizes at the edges of the sites per
thread (1024, 2048, 4096) and beyond the largest; budgets of no site, a few,
more than are ranked by counting (512) and every site; flat states whose
Delta S all tie; a floor left behind by either path taken up by the other."""
import pytest
import torch

from tests.parity_util import make_sim, random_state

pytestmark = pytest.mark.gpu

CASES = {
    # name: (nx, storage, k, options)
    "n1_f64": (1, "f64", 1, dict(bc="periodic")),
    "n2_f32": (2, "f32", 1, dict(bc="bounceback")),
    "n800_f64_k4": (800, "f64", 4, dict(bc="bounceback", positivity=True)),
    "n1023_f32_k0": (1023, "f32", 0, dict(bc="periodic")),
    "n1024_f64_k50": (1024, "f64", 50, dict(bc="periodic")),
    "n1025_f16s_k30": (1025, "f16s", 30, dict(bc="periodic", positivity=True)),
    "n2048_f32_k200": (2048, "f32", 200, dict(bc="bounceback")),
    "n2049_bf16s_k600": (2049, "bf16s", 600, dict(bc="periodic")),
    "n4096_f64_k9": (4096, "f64", 9, dict(bc="bounceback", ehr_delta=1e-4)),
    "n4096_f32_all": (4096, "f32", 5000, dict(bc="periodic")),
    "n4097_f64_k9": (4097, "f64", 9, dict(bc="periodic")),
}


def _sims(name, state):
    nx, storage, k, opts = CASES[name]
    p = dict(lattice="D1Q3", nx=nx, ny=1, nu=1e-3, ehrenfest=True, ehr_k=k,
             **{"ehr_delta": 0.0, **opts})
    f0 = random_state(p, 17, amp=0.3).cuda()
    if state == "ties":
        f0 = f0[:, :, :1].expand(3, 1, nx).contiguous()
    sims = [make_sim(p, storage) for _ in range(2)]
    for s in sims:
        s.set_populations(f0)
    return sims


def _same(a, b):
    assert torch.equal(a.populations(), b.populations())
    assert a.selected() == b.selected()
    assert a.counters() == b.counters()


@pytest.mark.parametrize("state", ["random", "ties"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_one_launch_matches_single_steps(name, state):
    a, b = _sims(name, state)
    for n in (1, 2, 19):
        a.step(n)
        b.profile_step(n)
        _same(a, b)
    a.profile_step(3)
    b.step(3)
    _same(a, b)
    a.step(4)
    b.profile_step(4)
    _same(a, b)
