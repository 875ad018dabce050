"""The D3Q27 median step's two kernels: a lattice stepped through the flagged
chunks only against one whose previous lattice left the step to the marching
kernel alone (every site above delta).  Same populations and counters bit for
bit, with no site above delta, with a few spots above it (in the lattice's
corners, at chunk edges, across ragged ones), and with all of them."""
import numpy as np
import pytest
import torch

import oracle as O
from tests.parity_util import make_sim

pytestmark = pytest.mark.gpu


def _states(nx, ny, nz):
    rng = np.random.default_rng(11)
    z, y, x = np.meshgrid(*(2 * np.pi * np.arange(n) / n for n in (nz, ny, nx)), indexing="ij")
    u = [0.02 * np.sin(x) * np.cos(y), -0.02 * np.cos(x) * np.sin(y), 0.01 * np.sin(z)]
    smooth = O.init_equilibrium3(np.ones_like(x), *u)
    spots = smooth.clone()
    for px, py, pz in ((0, 0, 0), (nx - 1, ny - 1, nz - 1), (min(63, nx - 1), min(7, ny - 1), nz // 2),
                       (nx // 2, ny // 2, min(31, nz - 1))):
        spots[:, pz, py, px] *= torch.tensor(1 + rng.uniform(-0.9, 0.9, 27))
    noisy = smooth * (1 + torch.tensor(rng.uniform(-0.5, 0.5, smooth.shape)))
    return {"smooth": smooth, "spots": spots, "noisy": noisy}


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("size", [(64, 8, 32), (70, 13, 35), (9, 5, 3), (130, 20, 40)])
def test_flagged_chunks_match_the_marching_kernel(size, storage):
    nx, ny, nz = size
    states = _states(nx, ny, nz)
    p = dict(lattice="D3Q27", nx=nx, ny=ny, nz=nz, bc="periodic", nu=1e-2, median=True,
             med_delta=1e-3, positivity=True)
    for name, f0 in states.items():
        a, b = make_sim(p, storage), make_sim(p, storage)
        b.set_populations(states["noisy"].cuda())
        b.step(1)                      # leaves the next step to the marching kernel
        c0 = b.counters()
        for s in (a, b):
            s.set_populations(f0.cuda())
        for step in range(4):
            a.step(1)
            b.step(1)
            fa, fb = a.populations(), b.populations()
            assert torch.equal(fa, fb), (name, step)
            assert a.counters() == [v - w for v, w in zip(b.counters(), c0)], (name, step)
