"""Several steps in one launch by overlapped tiles (lbm_step without the
Ehrenfest selection) against the same steps one by one (lbm_profile_step):
the same site arithmetic, so the same bits and counters.  Lattices narrower
than a tile and its halo, one site wide, and of every tile shape;
every boundary, with and without the median filter."""
import pytest
import torch

from tests.parity_util import make_sim, random_state

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (3, 3), (9, 5), (10, 10), (26, 17), (70, 37), (181, 163), (301, 289)]
CASES = {
    "lbgk_periodic": dict(bc="periodic"),
    "lbgk_pos_cavity": dict(bc="cavity", u_lid=0.1, positivity=True),
    "lbgk_couette": dict(bc="couette", u_lid=0.05),
    "lbgk_median_periodic": dict(bc="periodic", median=True, med_delta=1e-4),
    "lbgk_median_cavity": dict(bc="cavity", u_lid=0.1, median=True, med_delta=1e-3),
    "lbgk_median_couette": dict(bc="couette", u_lid=0.1, median=True, med_delta=0.0),
    "lbgk_median_diffusive": dict(bc="diffusive", u_lid=0.1, median=True, med_delta=1e-4,
                                  equilibrium="entropic"),
    "mrt_bounceback": dict(bc="bounceback", collision="mrt"),
    "mrt_median_omega": dict(bc="cavity", u_lid=0.1, collision="mrt", mrt_basis="M2", median=True,
                             med_delta=1e-4, omega_field=True),
    "elbm_cavity": dict(bc="cavity", u_lid=0.1, collision="elbm", equilibrium="entropic",
                        positivity=True),
    "elbm_median_periodic": dict(bc="periodic", collision="elbm", equilibrium="entropic",
                                 median=True, med_delta=1e-4),
}


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16s"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_overlapped_tiles_match_single_steps(name, storage):
    for nx, ny in SIZES:
        if CASES[name]["bc"] == "diffusive" and min(nx, ny) < 3:
            continue
        p = dict(lattice="D2Q9", nx=nx, ny=ny, nu=2e-3, **CASES[name])
        f0 = random_state(p, 23, amp=0.2, kind=p.get("equilibrium", "poly")).cuda()
        a, b = (make_sim(p, storage) for _ in range(2))
        for s in (a, b):
            s.set_populations(f0)
            if p.get("omega_field"):
                s.set_omega(torch.linspace(1.0, 1.9, nx * ny, device="cuda",
                                           dtype=torch.float64).view(ny, nx))
        for n in (16, 37):
            a.step(n)
            b.profile_step(n)
            fa, fb = a.populations(), b.populations()
            assert torch.equal(torch.nan_to_num(fa), torch.nan_to_num(fb)), (nx, ny, n)
            assert a.counters() == b.counters(), (nx, ny, n)
