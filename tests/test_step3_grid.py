"""The D3Q27 median step's screening kernel takes 256 threads a row and segment;
where that is 2^32 or more the step goes to the marching kernel alone, which
takes such a lattice (64 x 2^12 x 2^12 and its neighbours)."""
import ctypes

from paper_1110_0270_amd import lbm as B


def test_grid_limit():
    fn = getattr(B.library(), "_ZN3lbm13step3_screensEiii")
    fn.restype, fn.argtypes = ctypes.c_bool, [ctypes.c_int] * 3
    for nx, ny, nz in ((1, 1, 1), (256, 256, 256), (64, 4096, 4095), (256, 4096, 4095), (512, 2048, 4095),
                       (257, 2048, 4095), (64, 1, 2 ** 24 - 1)):
        assert -(-nx // 256) * 256 * ny * nz < 2 ** 32 and fn(nx, ny, nz), (nx, ny, nz)
    for nx, ny, nz in ((64, 4096, 4096), (1, 4096, 4097), (257, 2048, 4096), (16, 8192, 8192),
                       (1, 2 ** 15, 2 ** 15), (64, 1, 2 ** 24)):
        assert -(-nx // 256) * 256 * ny * nz >= 2 ** 32 and not fn(nx, ny, nz), (nx, ny, nz)
    # what a plane below 4 GiB leaves of these: 16-bit, nx <= 64, fewer than
    # 2^25 rows; the marching kernel's 512 threads for 64 x 8 columns of 32
    # layers hold them
    for ny, nz in ((4096, 4096), (8191, 4096), (8, 2 ** 22 - 1), (2 ** 20, 31)):
        assert -(-ny // 8) * -(-nz // 32) * 512 < 2 ** 32
