"""FP64 ELBM on both sides of 256 workgroups, where sites near equilibrium
change from the iteration to the series root: one step against the oracle, from
states with every site near (max |f*_i - f_i| / f_i < 2^-5), with none, and with
both kinds side by side."""
import pytest

import oracle as O
from tests.parity_util import gpu_run, oracle_run, random_state, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("amp", [0.005, 0.04, 0.2])
@pytest.mark.parametrize("size,bc", [((256, 256), "cavity"), ((256, 257), "cavity"), ((64, 1024), "periodic"),
                                     ((65, 513), "periodic"), ((200, 150), "diffusive"),
                                     ((300, 140), "couette")])
def test_one_step_beside_256_workgroups(size, bc, amp):
    p = dict(lattice="D2Q9", nx=size[0], ny=size[1], bc=bc, collision="elbm", equilibrium="entropic",
             nu=1e-3, u_lid=0.1 if bc != "periodic" else 0.0)
    f0 = random_state(p, 77, amp=amp, umax=0.02, kind="entropic")
    _, f_gpu, sim = gpu_run(p, f0, 1, "f64")
    f_ora, infos = oracle_run(p, f0, 1)
    assert rel_err(f_gpu, f_ora) <= 1e-12
    c = sim.counters()
    assert c[2] == int((infos[0]["branch"] == O.ELBM_NOROOT).sum())
    assert c[4] == int((infos[0]["branch"] == O.ELBM_NONPOS).sum())
