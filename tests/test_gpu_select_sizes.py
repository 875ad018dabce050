"""The Ehrenfest selection on both sides of each bound of its launches: one
workgroup up to 64 regions of 64 sites, one sweep workgroup up to 1024,
several beyond.  Steps on a carried floor and steps that rescan (omega = 1
collapses Delta S below the floor), each against the oracle's step from the
same input."""
import pytest
import torch

import oracle as O
from tests.parity_util import lattice, make_sim, near_tie_ok, oracle_config, random_state, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,rtol,ftol", [("f64", 1e-9, 1e-12), ("f32", 1e-5, 1e-5)])
@pytest.mark.parametrize("nx,ny", [(64, 64), (64, 68), (128, 128), (128, 132), (255, 256), (256, 257), (300, 300)])
def test_selection_and_rescans(nx, ny, storage, rtol, ftol):
    k = max(9, nx * ny // 1000)
    p = dict(lattice="D2Q9", nx=nx, ny=ny, bc="periodic", collision="lbgk", nu=1.0 / 6.0,
             ehrenfest=True, ehr_k=k, ehr_delta=0.0)
    sim = make_sim(p, storage)
    sim.set_populations(random_state(p, 131, amp=0.05).cuda())
    fb0 = int(sim.stats().select_fallbacks)
    for t in range(5):
        f_in = sim.populations().cpu()
        sim.step(1)
        f_gpu = sim.populations().cpu()
        sel = sorted(sim.selected())
        with torch.no_grad():
            f_ora, info = O.step(lattice(p), oracle_config(p), f_in)
        sel_ora = sorted(info["selected"].tolist())
        assert len(sel) == k, (t, len(sel))
        assert near_tie_ok(sel, sel_ora, info["dS"], k, rtol), t
        if sel == sel_ora:
            assert rel_err(f_gpu, f_ora) <= ftol, t
    assert int(sim.stats().select_fallbacks) > fb0
