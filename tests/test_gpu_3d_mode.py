"""The D3Q27 median step's choice between its two kernels (it decides the time
of a step, not its result): the marching kernel alone from the step after one
that flags more than a quarter of the chunks, also where the flagged sites lie
just under delta, and so it stays over steady values of that kind; back once
fewer than an eighth of the chunks hold a site above 7/8 delta."""
import pytest
import torch

import oracle as O
from oracle.lbm_oracle import kullback_dS
from tests.parity_util import make_sim

pytestmark = pytest.mark.gpu

NX, NY, NZ = 128, 16, 64


def _chunk(storage):
    return (64, 8, 16 if storage == "f64" else 32)


def _dense(sim, storage):
    """`dense` of Med3State: the layout's last blocks are the state with one
    16-byte record per chunk, and two of 256 bytes."""
    cx, cy, cz = _chunk(storage)
    chunks = (NX // cx) * (NY // cy) * (NZ // cz)
    size = 128 + 16 * 128 + 16 * chunks
    at = sim._ws.numel() - 512 - (size + 255) // 256 * 256
    torch.cuda.synchronize()
    tally, dense = sim._ws[at:at + 16].view(torch.int64).tolist()
    assert tally == 0
    return dense & 0xffffffff


def _uniform(amp):
    """f* (1 + amp x) at every site, x of one random draw without mass and
    momentum; its Delta S."""
    feq = O.init_equilibrium3(torch.ones(1, 1, 1), *[torch.zeros(1, 1, 1)] * 3)
    gen = torch.Generator().manual_seed(5)
    lat = O.Lattice3()
    d = torch.rand(27, generator=gen, dtype=torch.float64) - 0.5
    basis = torch.linalg.qr(torch.stack([torch.ones(27, dtype=torch.float64), lat.vx, lat.vy, lat.vz], 1))[0]
    d -= basis @ (basis.T @ d)
    f = feq + (amp / (d.view(27, 1, 1, 1) / feq).abs().max()) * d.view(27, 1, 1, 1)
    return f, float(kullback_dS(f, feq))


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
def test_mode(storage):
    f, dS = _uniform(0.05)
    rest = O.init_equilibrium3(torch.ones(1, 1, 1), *[torch.zeros(1, 1, 1)] * 3)
    # the bound is within 1 + 2/3 0.05 of Delta S, delta above it by 0.5 %
    sim = make_sim(dict(lattice="D3Q27", nx=NX, ny=NY, nz=NZ, bc="periodic", nu=1e-2, median=True,
                        med_delta=1.005 * dS), storage)
    full = f.expand(27, NZ, NY, NX).contiguous()
    cx, cy, cz = _chunk(storage)

    def step(state):
        sim.set_populations(state.cuda())
        sim.step(1)
        return _dense(sim, storage)

    # one chunk in eight holds such sites (a margin of two sites keeps the
    # pull from reaching the next): no quarter
    part = rest.expand(27, NZ, NY, NX).contiguous()
    part[:, 2:cz - 2, 2:cy - 2, 2:cx - 2] = f
    assert step(part) == 0
    c0 = sim.counters()
    assert step(full) == 1            # flagged everywhere, no site above delta
    assert step(full) == 1            # 0.995 delta: as it was
    low = rest + (0.9 ** 0.5) * (f - rest)
    assert step(low.expand_as(full).contiguous()) == 1     # 0.895 delta
    low = rest + (0.8 ** 0.5) * (f - rest)
    assert step(low.expand_as(full).contiguous()) == 0     # 0.796 delta
    assert step(low.expand_as(full).contiguous()) == 0
    assert sim.counters() == c0       # nothing was filtered
