"""FP32 arithmetic, ELBM on a periodic lattice (the row kernel, with the first
terms of the series for sites near equilibrium): what a site becomes depends on
its own populations, not on the other sites of its wavefront.  Every site pulls
f* (1 + x) with alpha max |x_i| at or just under 2^-8, where those terms and
the whole series differ most; then one site of each wavefront is driven
further from equilibrium (past 2^-8, and past 0.1, where the series ends), and
the others have the same bits."""
import pytest
import torch

import oracle as O
from tests.parity_util import lattice, make_sim, random_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("far", [0.02, 0.3])
@pytest.mark.parametrize("top", [0.5, 0.98])
@pytest.mark.parametrize("lattice_,nx,ny", [("D2Q9", 512, 1024), ("D2Q9", 300, 61), ("D1Q3", 65536, 1)])
def test_sites_do_not_depend_on_their_wavefront(lattice_, nx, ny, top, far):
    p = dict(lattice=lattice_, nx=nx, ny=ny, bc="periodic", collision="elbm",
             equilibrium="entropic", nu=1e-3)
    lat = lattice(p)
    feq = random_state(p, 3, amp=0.0, kind="entropic")
    # noise without mass and momentum, its largest |D_i| / f_i scaled to
    # top * 2^-9 (alpha = 2 brings alpha |D_i| / f_i to top * 2^-8)
    gen = torch.Generator().manual_seed(7)
    d = torch.rand(feq.shape, generator=gen, dtype=torch.float64) - 0.5
    rows = [torch.ones(lat.Q, dtype=torch.float64), lat.vx] + ([lat.vy] if lat.Q == 9 else [])
    basis = torch.linalg.qr(torch.stack(rows, 1))[0]
    d -= torch.einsum("qk,pk,pyx->qyx", basis, basis, d)
    d /= (d.abs() / feq).amax(0)
    near = feq + d * (top * 2.0 ** -9)
    hit = torch.zeros(ny, nx, dtype=torch.bool)
    hit[:, 20::64] = True
    mixed = torch.where(hit, feq + d * far, near)
    out = []
    for pulled in (near, mixed):
        # f_i(x) = pulled_i(x + v_i): the step's pull restores it
        f = torch.stack([torch.roll(pulled[i], (-b, -a), (0, 1)) for i, (a, b) in enumerate(lat.vel)])
        assert torch.equal(O.stream(lat, f, "periodic"), pulled)
        sim = make_sim(p, "f32")
        sim.set_populations(f.cuda())
        sim.step(1)
        out.append(sim.populations().cpu())
    a, b = (o[:, ~hit] for o in out)
    assert torch.equal(a, b), f"{int((a != b).any(0).sum())} of {a.shape[1]} sites differ"
    assert bool((out[0] != out[1])[:, hit].any(0).all())
