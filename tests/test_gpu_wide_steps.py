"""Wide-angle pixels against the oracle at all step lengths: through the cell
records up to what 16 of them hold (0.0793 cells along each axis, 0.2063 along
one), by the per-pixel gathers past that (0.0794, 0.2064, 0.7), both storage
types, few and many lines; and the same bits at every tuned unroll."""
import numpy as np
import pytest
import torch

from oracle import skewers
from tests.lyahelp import bf16_to_f32, gpu_skewers, padded_box, rel_rms
from tests.test_gpu_cell_walk import _table
from tests.test_gpu_skewers import L  # noqa: F401

pytestmark = pytest.mark.gpu
N = 32


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("step", [(0.01, 0.02, 0.0913), (0.0793, 0.0793, 0.0793), (0.0794, 0.0794, 0.0794),
                                  (0.2063, 0.0, 0.0), (0.0, 0.0, 0.2064), (0.7, 0.3, 0.2), (2.5, 1.0, 40.3)])
def test_wide_against_the_oracle(L, step, bf16):  # noqa: F811
    print("wide steps", step, bf16, flush=True)
    rng = np.random.default_rng([int(1e4 * step[0]), int(1e4 * step[2])])
    grids = [rng.normal(0.0, 1.0, (N, N, N, 2)).astype(np.float32) for _ in range(4)]
    f = [padded_box(L, g) for g in grids]
    if bf16:
        f = [x.to(torch.bfloat16).contiguous().view(torch.int32).view(-1) for x in f]
        grids = [bf16_to_f32(L.box_view(x, N)) for x in f]
    g = [x.astype(np.float64) for x in grids]
    eta6 = [g[1][..., 0], g[1][..., 1], g[0][..., 1], g[2][..., 0], g[2][..., 1], g[3][..., 0]]
    few, many = _table(N, step, 21, 0), _table(N, step, 21, 5000)
    many["origin_fx"][:len(few["npix"])] = few["origin_fx"]
    args = (N, 1.0), (7, 1.0, 1.5, 0.2)
    kw = dict(storage=int(bf16), want=("dens", "eta"))
    a = gpu_skewers(L, f, *args[0], few, *args[1], **kw)
    b = gpu_skewers(L, f, *args[0], many, *args[1], **kw)
    rd, re_ = skewers.draw_skewers_wide(g[0][..., 0], eta6, few, 7, 1.0, 1.5, 0.2)
    still = np.repeat(np.all(few["step_fx"] == 0, axis=1), few["npix"])
    assert np.array_equal(np.isnan(re_), still)
    re_[still] = 0.0     # a line without steps has no direction: eta_par 0
    print("rel rms %.2e %.2e" % (rel_rms(a["dens"], rd), rel_rms(a["eta"], re_)))
    assert rel_rms(a["dens"], rd) < 1e-5 and rel_rms(a["eta"], re_) < 1e-5
    was = L.get_tuning(N)
    try:
        for u in (2, 4):
            t = L.get_tuning(N)
            t.sk_unroll = u
            L.set_tuning(N, t)
            c = gpu_skewers(L, f, *args[0], many, *args[1], **kw)
            for k in ("dens", "eta"):
                np.testing.assert_array_equal(a[k], c[k], err_msg="unroll %d %s" % (u, k))
    finally:
        L.set_tuning(N, was)
    for k in ("dens", "eta"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
