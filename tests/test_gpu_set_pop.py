"""lbm_set_populations on both sides of the input size from which it no longer
reads through the caches (256 MiB): FP64 and FP32 input come back unchanged
from FP64 storage, and from FP32 storage what rounding the shifted value gives."""
import pytest
import torch

from tests.parity_util import make_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("dtype,nx,ny", [(torch.float64, 1931, 1930), (torch.float64, 1931, 1931),
                                         (torch.float32, 2731, 2730), (torch.float32, 2731, 2731)])
def test_round_trip(dtype, nx, ny, storage):
    bytes_in = 9 * nx * ny * (8 if dtype == torch.float64 else 4)
    assert (bytes_in > 256 << 20) == (nx == ny)
    gen = torch.Generator(device="cuda").manual_seed(3)
    f = torch.rand(9, ny, nx, generator=gen, device="cuda", dtype=dtype)
    sim = make_sim(dict(lattice="D2Q9", nx=nx, ny=ny, bc="periodic", nu=1e-3), storage)
    sim.set_populations(f)
    got = sim.populations()
    if storage == "f64":
        assert torch.equal(got, f.double())
    else:
        w1 = torch.tensor((1 / 6, 2 / 3, 1 / 6), dtype=torch.float64, device="cuda")
        w = (w1.view(3, 1) * w1.view(1, 3)).reshape(9, 1, 1)
        # rounding of f - w to FP32: half a unit of a value below 1
        assert float((got - f.double()).abs().max()) <= 2.0 ** -25 * (1 + 1e-6)
        assert torch.equal((got - w).float(), (f.double() - w).float())
