"""The adjoint on a lattice whose 16-bit population planes lie within 4 GiB
and whose FP32 adjoint planes do not: a uniform flow of 2^30 + 128 sites, a
loss at sites on both sides of the 2^30-th.  The state is the same at every
site, so the gradient around them is that of a short lattice, bit for bit, and
zero elsewhere."""
import pytest
import torch

from paper_1110_0270_amd import lbm as B

pytestmark = pytest.mark.gpu


def _gradient(n, at, g):
    """dL/df0 (window of 64 sites from `at`, sum of |.| outside) of one ELBM
    step, with dL/df given by g on that window and zero elsewhere."""
    cfg = B.make_config(lattice="D1Q3", nx=n, ny=1, bc="periodic", nu=1e-2, collision="elbm",
                        equilibrium="entropic", storage="f16s", checkpoint_every=1, max_steps=1)
    sim = B.Simulation(cfg)
    rho = torch.ones(1, n, device="cuda", dtype=torch.float32)
    sim.set_equilibrium(rho, rho * 0.05)
    del rho
    sim.step(1)
    dT = torch.zeros(3, 1, n, device="cuda", dtype=torch.float32)
    dT[:, 0, at + 16:at + 48] = g
    d0 = torch.empty_like(dT)
    sim.backward(dT, d0)
    win = d0[:, 0, at:at + 64].clone()
    d0[:, 0, at:at + 64] = 0
    return win.cpu(), max(float(d0[i].abs().max()) for i in range(3))


def test_planes_beyond_4_gib():
    n = (1 << 30) + 128
    if torch.cuda.mem_get_info()[0] < 150 << 30:
        pytest.skip("needs 150 GiB of free device memory")
    g = torch.linspace(-1, 1, 96, device="cuda").view(3, 32)
    want, _ = _gradient(4096, 1024, g)
    got, rest = _gradient(n, (1 << 30) - 32, g)
    torch.cuda.empty_cache()
    assert float(want.abs().max()) > 0
    assert torch.equal(got, want)
    assert rest == 0.0
