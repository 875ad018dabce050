"""How many steps one launch takes (D2Q9 without the Ehrenfest selection), by
storage, collision, filter and size: four without the median filter up to 256
tiles of 26 x 26; with it two up to 256 tiles of 26 x 26, in FP64 two up to 256
tiles of 10 x 10 and one up to 512 of 30 x 14; none for ELBM.  The comparisons
on the GPU rest on it: a size of 0 compares the single steps with themselves."""
import ctypes

import pytest

from paper_1110_0270_amd import lbm as B

F64, F32, F16, BF16 = range(4)
LBGK, MRT, ELBM = range(3)


def _steps(storage, coll, median, nx, ny):
    fn = getattr(B.library(), "_ZN3lbm11multi_stepsEiibii")
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_int, ctypes.c_int]
    return fn(storage, coll, median, nx, ny)


@pytest.mark.parametrize("coll", [LBGK, MRT])
@pytest.mark.parametrize("storage", [F64, F32, F16, BF16])
def test_steps_per_launch(storage, coll):
    for nx, ny in [(1, 1), (9, 5), (70, 37), (160, 160), (161, 160), (301, 289), (416, 416), (2210, 60)]:
        assert _steps(storage, coll, False, nx, ny) == 4, (nx, ny)
    for nx, ny in [(417, 416), (512, 512), (4096, 4096), (26 * 257, 1)]:
        assert _steps(storage, coll, False, nx, ny) == 0, (nx, ny)
    med = [((1, 1), 2, 2), ((70, 37), 2, 2), ((160, 160), 2, 2), ((161, 160), 1, 2), ((301, 289), 1, 2),
           ((416, 416), 1, 2), ((417, 416), 1, 0), ((480, 448), 1, 0), ((481, 448), 0, 0),
           ((4096, 4096), 0, 0)]
    for (nx, ny), f64, other in med:
        assert _steps(storage, coll, True, nx, ny) == (f64 if storage == F64 else other), (nx, ny)


@pytest.mark.parametrize("storage", [F64, F32, F16, BF16])
def test_elbm_takes_single_steps(storage):
    for size in [(1, 1), (70, 37), (301, 289), (4096, 4096)]:
        assert _steps(storage, ELBM, False, *size) == _steps(storage, ELBM, True, *size) == 0
