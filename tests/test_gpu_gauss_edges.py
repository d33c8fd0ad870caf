"""The 7^3 Gaussian-kernel pass at the edges of its shared-window path: steps
around a third of a cell (where pixels stop sharing a window), long and short z
runs, planes staged in several parts, lines ending around 64 pixels, wrapping
windows, and a voxel that is not finite; against the oracle's 343-voxel sums."""
import numpy as np
import pytest

from oracle import skewers
from tests.lyahelp import gpu_skewers, padded_box, rel_rms

pytestmark = pytest.mark.gpu
T32 = 2 ** 32


@pytest.fixture(scope="module")
def L():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_18996_amd import lyamock
    lyamock.load()
    return lyamock


def _table(n, step, npix, seed):
    rng = np.random.default_rng(seed)
    S = len(npix)
    off = np.zeros(S, np.int64)
    off[1:] = np.cumsum(npix[:-1])
    o = rng.uniform(-3.0 * n, 3.0 * n, (S, 3))
    o[::5] = np.round(o[::5] * 2) / 2   # grid points and half-cell ties
    return dict(origin_fx=np.round(o * T32).astype(np.int64), step_fx=np.round(step * T32).astype(np.int64),
                npix=np.asarray(npix, np.int32), offset=off, chi0=np.full(S, 4000.0), dchi=0.2, id_base=0,
                total=int(np.sum(npix)))


def _check(L, grid, sk, bf16=False):
    import torch
    n = grid.shape[0]
    fld = padded_box(L, grid)
    if bf16:
        fld = fld.to(torch.bfloat16)
        grid = L.box_view(fld, n).float().cpu().numpy()
        fld = fld.contiguous().view(torch.int32).view(-1)
    out = gpu_skewers(L, fld, n, 1.0, sk, 5, 0.0, 1.0, 0.2, storage=int(bf16), want=("dens", "eta"), gauss=True)
    rd, re_ = skewers.draw_skewers(grid[..., 0].astype(np.float64), grid[..., 1].astype(np.float64), sk, 5, 0.0, 1.0,
                                   0.2, interp=skewers.gauss7)
    # sums of 343 products in FP32: 2^-24 sqrt(343) = 1.1e-6, and the weights' 3e-7
    e = (rel_rms(out["dens"], rd), rel_rms(out["eta"], re_))
    print("rel rms %.2e %.2e" % e, flush=True)
    assert max(e) < 2e-6, e


LENGTHS = [1, 2, 3, 4, 5, 63, 64, 65, 66, 127, 128, 129, 200]


@pytest.mark.parametrize("n", [32, 64])
@pytest.mark.parametrize("size", [0.0, 0.0913, 0.1249, 0.13, 0.2, 0.3330, 0.3334, 1.5])
def test_step_sizes(L, n, size):
    rng = np.random.default_rng(int(size * 1e4) + n)
    grid = rng.normal(size=(n, n, n, 2)).astype(np.float32)
    u = rng.normal(size=(len(LENGTHS) * 6, 3))
    u[0::6], u[1::6], u[2::6] = [0, 0, 1], [0, -1, 0], [1, 0, 0]   # axes, then every direction
    u[3::6] = np.array([0.05, -0.06, 1.0])
    u /= np.abs(u).max(axis=1)[:, None]                             # largest component = the step size
    print("n %d step %.4f" % (n, size), flush=True)
    _check(L, grid, _table(n, u * size, np.repeat(LENGTHS, 6), n), bf16=n == 32)


def test_voxels_not_finite_stay_in_their_reach(L):
    n = 32
    rng = np.random.default_rng(3)
    grid = rng.normal(size=(n, n, n, 2)).astype(np.float32)
    grid[7, 11, 20, 0] = np.nan
    grid[20, 5, 9, 1] = np.inf
    step = np.tile([[0.02, 0.03, 0.0913]], (60, 1))
    sk = _table(n, step, np.full(60, 150), 9)
    out = gpu_skewers(L, padded_box(L, grid), n, 1.0, sk, 5, 0.0, 1.0, 0.2, want=("dens", "eta"), gauss=True)
    # one component at a time: the oracle's complex product would carry a voxel
    # that is not finite into the other component
    zero = np.zeros((n, n, n))
    with np.errstate(all="ignore"):
        rd, re_ = (skewers.draw_skewers(grid[..., c].astype(np.float64), zero, sk, 5, 0.0, 1.0, 0.2,
                                        interp=skewers.gauss7)[0] for c in (0, 1))
    for got, want in ((out["dens"], rd), (out["eta"], re_)):
        assert 0 < np.sum(~np.isfinite(want)) < want.size
        np.testing.assert_array_equal(np.isfinite(got), np.isfinite(want))
        ok = np.isfinite(want)
        assert rel_rms(got[ok], want[ok]) < 2e-6
