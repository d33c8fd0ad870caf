"""Origins as far as 64-bit positions reach: a line whose pixels cross +-2^31 cells
(where positions wrap, consistently with the periodic box, since n is a power of
two) gives what the same line gives from the same place inside the box; all
interpolation modes and storage types, few and many lines."""
import numpy as np
import pytest
import torch

from tests.lyahelp import gpu_skewers, padded_box, rel_rms
from tests.test_gpu_skewers import L  # noqa: F401

pytestmark = pytest.mark.gpu
T32 = 2 ** 32
N = 32


def _tables(step, extra):
    """Lines that cross the wrap after 1, 20 .. cells along one axis or all, and
    their origins modulo the box."""
    dirs = [(1, 0, 0), (0, -1, 0), (0, 0, 1), (1, 1, 1), (-1, -1, -1), (1, -1, 0), (-1, 0, 1)]
    rng = np.random.default_rng(4)
    far, near, st = [], [], []
    for u in dirs:
        for cells in (0.4, 3.3, 7.0):
            o = [int(rng.integers(0, N * T32)) if d == 0 else d * (2 ** 63 - int(cells * T32)) - (d > 0) for d in u]
            o = [max(min(v, 2 ** 63 - 1), -2 ** 63) for v in o]
            far.append(o)
            near.append([v % (N * T32) for v in o])
            st.append([int(round(d * step * T32)) for d in u])
    S = len(far)
    npix = np.concatenate([np.full(S, 200), np.zeros(extra)]).astype(np.int32)
    pad = np.zeros((extra, 3), np.int64)
    off = np.concatenate([[0], np.cumsum(npix[:-1].astype(np.int64))])
    out = []
    for o in (far, near):
        out.append(dict(origin_fx=np.concatenate([np.array(o, np.int64), pad]),
                        step_fx=np.concatenate([np.array(st, np.int64), pad]), npix=npix, offset=off,
                        chi0=np.full(S + extra, 4100.0), dchi=0.2, id_base=0, total=int(npix.sum())))
    return out


@pytest.mark.parametrize("extra", [0, 5000])
@pytest.mark.parametrize("step", [0.0913, 0.3, 0.7])
@pytest.mark.parametrize("kind", ["tri", "bf16", "wide", "gauss"])
def test_same_as_inside_the_box(L, kind, step, extra):  # noqa: F811
    print("far origins", kind, step, extra, flush=True)
    rng = np.random.default_rng(6)
    f = [padded_box(L, rng.normal(0.0, 1.0, (N, N, N, 2)).astype(np.float32)) for _ in range(4 if kind == "wide" else 1)]
    if kind == "bf16":
        f = [f[0].to(torch.bfloat16).contiguous().view(torch.int32).view(-1)]
    far, near = _tables(step, extra)
    args = (N, 1.0), (5, 1.0, 1.5, 0.2)
    kw = dict(storage=int(kind == "bf16"), gauss=kind == "gauss", want=("dens", "eta"))
    a, b = (gpu_skewers(L, f if kind == "wide" else f[0], *args[0], t, *args[1], **kw) for t in (far, near))
    for k in ("dens", "eta"):
        if kind == "gauss":     # other order of summation over the 343 voxels
            assert rel_rms(a[k], b[k]) < 1e-6
        else:
            np.testing.assert_array_equal(a[k], b[k], err_msg=k)
