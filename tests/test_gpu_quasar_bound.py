"""The quasar draw's early rejection keeps every voxel that the full evaluation
selects: an observer inside the box (distances that are not monotone along a
line, all redshifts from 0), wide voxels (large redshift steps between a thread's
voxels), probabilities from 1e-6 to above 1 (every voxel selected, the waves'
lists flushed in mid-tile), several tiles per wave, and values that are not
finite."""
import numpy as np
import pytest

from oracle import cosmology, quasars
from tests.test_gpu_quasars import ZB3, L, _compare, _draw, _voxel_ids  # noqa: F401

pytestmark = pytest.mark.gpu
NZ = np.array([0.0, 0.5, 1.5, 2.5, 4.0])
# exponents up to |x| ~ 20 in FP32: 20 2^-24 and the factors' own few ulp
BAND = 1e-5


def case(n, dx, n_box, where, seed):
    rng = np.random.default_rng([n, n_box, seed])
    f = [rng.normal(scale=s, size=(n, n, n)).astype(np.float32) for s in (0.8, 0.6, 0.5)[:n_box]]
    var = [float(np.var(x.astype(np.float64))) for x in f]
    mid = n * dx / 2
    obs = np.array([mid, mid, mid + 0.3 * dx if where == "inside" else -cosmology.chi_of_z(1.7)])
    return f, var, obs, (list(ZB3) if n_box == 3 else [2.2])


@pytest.mark.parametrize("n,dx,n_box,where,density", [
    (32, 15.0, 1, "inside", 1e-5), (32, 100.0, 3, "inside", 1e-7), (32, 60.0, 3, "outside", 1e-9),
    (64, 10.0, 3, "outside", 1e-4), (64, 20.0, 1, "outside", 1.0), (64, 20.0, 3, "inside", 1.0)])
def test_draw_against_the_full_evaluation(L, n, dx, n_box, where, density):  # noqa: F811
    print("%d^3 of %g, %d boxes, observer %s, density %g" % (n, dx, n_box, where, density), flush=True)
    f, var, obs, zb = case(n, dx, n_box, where, 1)
    nb = density * np.array([1.0, 3.0, 2.0, 0.5, 0.1])
    xi5 = 0.82 if n_box == 3 else 0.0
    c, pos = _draw(L, f, dx, obs, zb, var, NZ, nb, 91, xi5=xi5)
    idx, fx, p, u = quasars.draw([x.astype(np.float64) for x in f], dx, obs, zb, var, NZ, nb, 91,
                                 xi5=xi5 if n_box == 3 else None)
    _compare(n, c, pos, idx, fx, p, u, band=BAND)


@pytest.mark.parametrize("n_box,density", [(1, 3e-6), (3, 2e-2)])
def test_draw_of_several_tiles_per_wave(L, n_box, density):  # noqa: F811
    n, dx = 256, 6.0
    print("%d^3, %d boxes, density %g" % (n, n_box, density), flush=True)
    f, var, obs, zb = case(n, dx, n_box, "outside", 2)
    nb = density * np.array([1.0, 3.0, 2.0, 0.5, 0.1])
    c, pos = _draw(L, f, dx, obs, zb, var, NZ, nb, 92, xi5=0.82 if n_box == 3 else 0.0)
    gid = np.sort(_voxel_ids(pos, n))
    assert c == len(gid) and np.all(np.diff(gid) > 0)
    lin = np.unique(np.random.default_rng(5).integers(0, n ** 3, 300_000))
    p, _ = quasars.probability_at(lin, [x.reshape(-1)[lin].astype(np.float64) for x in f], n, dx, obs, zb, var, NZ, nb,
                                  xi5=0.82 if n_box == 3 else None)
    u = quasars.decision_uniforms_at(92, lin)
    inside = np.isin(lin, gid)
    assert np.all(inside[u < p * (1 - BAND) - 1e-9]) and not np.any(inside[u > p * (1 + BAND) + 1e-9])
    assert abs(c / (np.minimum(p, 1).mean() * float(n) ** 3) - 1) < 0.1
    order = np.argsort(_voxel_ids(pos, n))
    np.testing.assert_array_equal(pos[order][:5000], quasars.positions(92, gid[:5000], n))


def test_values_that_are_not_finite(L):  # noqa: F811
    n, dx = 32, 12.0
    f, var, obs, zb = case(n, dx, 1, "outside", 3)
    flat = f[0].reshape(-1)
    nan, inf, low = np.arange(7, 4000, 131), np.arange(9, 4000, 127), np.arange(11, 4000, 113)
    flat[low], flat[inf], flat[nan] = -np.inf, np.inf, np.nan
    c, pos = _draw(L, f, dx, obs, zb, var, NZ, np.full(5, 1e-9), 93)
    gid = _voxel_ids(pos, n)
    assert c == len(gid)
    # p is not a number, or infinite: taken; zero: not
    assert np.all(np.isin(nan, gid)) and np.all(np.isin(inf, gid))
    assert not np.any(np.isin(np.setdiff1d(low, np.concatenate([nan, inf])), gid))
