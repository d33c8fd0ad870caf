"""Trilinear pixels through the wave's cell records (calls with more lines than
waves, steps that cross few cells in 64 pixels) against the per-pixel gathers of
a call with few lines, bit for bit, and those against the oracle: steps up to and
past what 16 records hold, in all directions and along single axes, both storage
types, the wide-angle boxes (whose calls with few lines walk cells too, and are held
against the oracle in test_gpu_wide), lines ending around 64 pixels, and outputs
left out."""
import numpy as np
import pytest
import torch

from oracle import fgpa, skewers
from tests.lyahelp import gpu_skewers, padded_box, rel_rms
from tests.test_gpu_skewers import L  # noqa: F401

pytestmark = pytest.mark.gpu
T32 = 2 ** 32
LENGTHS = [1, 2, 63, 64, 65, 127, 128, 129, 200, 1025, 2048]
COEF = [[-0.9, 0.4, 0.05], [1.6, 0.0, 0.0], [0.3, 0.2, 0.0]]


def _table(n, step, seed, extra):
    """A line per length and step direction, then `extra` lines without pixels."""
    rng = np.random.default_rng(seed)
    dirs = [(1, 1, 1), (-1, 1, -1), (-1, -1, -1), (1, -1, 0), (1, 0, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1)]
    u = np.repeat(np.array(dirs, float), len(LENGTHS), axis=0)
    npix = np.array(LENGTHS * len(dirs) + [0] * extra, np.int32)
    S = len(npix)
    o = rng.uniform(-2.0 * n, 2.0 * n, (S, 3))
    o[::4] = np.round(o[::4])            # on grid points
    st = np.zeros((S, 3))
    st[:len(u)] = u * np.asarray(step)
    off = np.concatenate([[0], np.cumsum(npix[:-1].astype(np.int64))])
    return dict(origin_fx=np.round(o * T32).astype(np.int64), step_fx=np.round(st * T32).astype(np.int64), npix=npix,
                offset=off, chi0=rng.uniform(3900.0, 4300.0, S), dchi=0.2, id_base=3, total=int(npix.sum()))


@pytest.mark.parametrize("kind", ["f32", "bf16", "wide"])
@pytest.mark.parametrize("n,step", [(32, (0.0, 0.0, 0.0)), (32, (0.01, 0.02, 0.0913)), (64, (0.0527, 0.0527, 0.0527)),
                                    (32, (0.0793, 0.0793, 0.0793)), (32, (0.0794, 0.0794, 0.0794)),
                                    (64, (0.2063, 0.0, 0.0)), (64, (0.0, 0.0, 0.2064)), (32, (0.7, 0.3, 0.2))])
def test_same_as_single_gathers(L, kind, n, step):  # noqa: F811
    print("cell walk", kind, n, step, flush=True)
    rng = np.random.default_rng([n, 7])
    grids = [rng.normal(0.0, 1.0, (n, n, n, 2)).astype(np.float32) for _ in range(4 if kind == "wide" else 1)]
    f = [padded_box(L, g) for g in grids]
    if kind == "bf16":
        f = [f[0].to(torch.bfloat16).contiguous().view(torch.int32).view(-1)]
    field = f if kind == "wide" else f[0]
    edges = fgpa.chi_edges_for_z(np.linspace(1.8, 3.5, 9))
    few, many = _table(n, step, 11, 0), _table(n, step, 11, 5000)
    many["chi0"][:len(few["npix"])] = few["chi0"]
    many["origin_fx"][:len(few["npix"])] = few["origin_fx"]
    args = (n, 1.0), (5, 1.0, 1.5, 0.2)
    kw = dict(storage=int(kind == "bf16"))
    a = gpu_skewers(L, field, *args[0], few, *args[1], COEF, edges, **kw)
    b = gpu_skewers(L, field, *args[0], many, *args[1], COEF, edges, **kw)
    for k in ("dens", "eta", "flux", "fsum", "count"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
    c = gpu_skewers(L, field, *args[0], many, *args[1], None, None, want=("eta",), **kw)
    np.testing.assert_array_equal(a["eta"], c["eta"])
    if kind == "f32":
        rd, re_ = skewers.draw_skewers(grids[0][..., 0].astype(np.float64), grids[0][..., 1].astype(np.float64), few,
                                       5, 1.0, 1.5, 0.2)
        assert rel_rms(b["dens"], rd) < 1e-5 and rel_rms(b["eta"], re_) < 1e-5
