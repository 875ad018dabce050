"""Candidate lists of a short D1Q3 lattice in one launch (lbm_step) around the
length up to which they are ranked by counting (32), and longer ones: every site
listed (the budget is no less than a tenth of the lattice), the budget inside a
tie group or between two, against the step and selection kernels
(lbm_profile_step): the same bits and selections."""
import pytest
import torch

from tests.parity_util import make_sim, random_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("state", ["random", "ties", "two_levels"])
@pytest.mark.parametrize("n,k", [(31, 9), (32, 16), (33, 16), (33, 32), (257, 130), (700, 256), (1500, 700),
                                 (4096, 2100)])
def test_lists(n, k, state, storage):
    p = dict(lattice="D1Q3", nx=n, ny=1, bc="periodic", nu=1e-3, ehrenfest=True, ehr_k=k, ehr_delta=0.0)
    f0 = random_state(p, 29, amp=0.3).cuda()
    if state != "random":
        a = f0[:, :, :1].expand_as(f0).contiguous()
        if state == "two_levels":      # stronger sites in the middle third
            a[:, :, n // 3:2 * n // 3] = f0[:, :, 1:2]
        f0 = a
    a, b = make_sim(p, storage), make_sim(p, storage)
    for s in (a, b):
        s.set_populations(f0)
    for steps in (1, 2, 6):
        a.step(steps)
        b.profile_step(steps)
        assert torch.equal(a.populations(), b.populations())
        assert a.selected() == b.selected()
