"""The 7^3 Gaussian-kernel pass on short lines with steps of a third of a cell and
more, whose cells lie in LDS together: boxes of cells that just fit (at most 1348)
and just do not, one pixel, very long steps, windows that wrap around a small box,
origins near the ends of 64-bit positions; against the oracle's 343-voxel sums."""
import numpy as np
import pytest

from tests.test_gpu_gauss_edges import L, T32, _check, _table  # noqa: F401

pytestmark = pytest.mark.gpu


# cells per axis along z: 7 x 7 x (7 + span), so span 20 fits and 21 does not; the
# oblique ones 8 x 8 x 21 (fits), 8 x 8 x 22 and 7 x 8 x 25 (do not)
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("u,npix", [((0, 0, 1.0), 21), ((0, 0, 1.0), 22), ((0, 0, -0.5), 41), ((0, 0, -0.5), 43),
                                    ((0.05, 0.05, 0.7), 21), ((0.05, -0.05, 0.75), 21), ((0.0, 0.0625, 0.95), 20),
                                    ((0.34, 0.0, 0.0), 60), ((0.0, -0.34, 0.1), 30), ((2.5, -2.5, 2.5), 2),
                                    ((300.0, 0.0, 0.0), 2), ((1e6, 1e5, -1e6), 5), ((0.7, 0.3, -0.5), 130)])
def test_boxes_of_cells(L, u, npix, bf16):  # noqa: F811
    print("short lines", u, npix, bf16, flush=True)
    rng = np.random.default_rng([npix, int(1000 * u[2]) & 0xFFFF])
    n = 32
    grid = rng.normal(0.0, 1.0, (n, n, n, 2)).astype(np.float32)
    S = 24
    lens = [npix, npix - 1, 1, max(npix // 2, 1)] * (S // 4)
    _check(L, grid, _table(n, np.tile(np.asarray(u, float), (S, 1)), lens, npix), bf16=bf16)


def test_boxes_near_the_ends_of_positions(L):  # noqa: F811
    rng = np.random.default_rng(3)
    n = 32
    grid = rng.normal(0.0, 1.0, (n, n, n, 2)).astype(np.float32)
    sk = _table(n, np.tile([0.0, -0.4, 0.5], (16, 1)), [20] * 16, 5)
    sk["origin_fx"][:8, 2] = 2 ** 63 - 1 - 3 * T32 * np.arange(8)
    sk["origin_fx"][8:, 1] = -2 ** 63 + 2 * T32 * np.arange(8)
    with np.errstate(over="ignore"):
        _check(L, grid, sk)
