"""Every component in both places of a box, with an even and an odd partner,
against the oracle: the multiplier's Nyquist planes (a quarter of the modes of the
smallest box lie on one), one spectrum without test hooks."""
import numpy as np
import pytest

from oracle import field
from tests.lyahelp import gpu_box, oracle_table, rel_rms
from tests.test_gpu_box import PK, L  # noqa: F401

pytestmark = pytest.mark.gpu
TOL = 1e-5   # of every box against the oracle: FP32 amplitudes, noise and transform


@pytest.mark.parametrize("n,two_buffer", [(32, False), (64, True)])
@pytest.mark.parametrize("comp", ["delta", "xx", "yy", "zz", "xy", "xz", "yz", "vx", "vy", "vz"])
def test_component_in_either_place(L, comp, n, two_buffer):  # noqa: F811
    dx, seed, f = 2.19, 19, 0.8
    tab = oracle_table(PK, n, dx)
    for comps in ((comp, "yz"), (comp, "vy"), ("xx", comp), ("vz", comp), (comp, "none")):
        print("components %s of a %d^3 box" % (comps, n), flush=True)
        g = gpu_box(L, n, dx, seed, f, comps=comps, two_buffer=two_buffer, **PK).cpu().numpy().astype(np.float64)
        ref = field.make_box(n, seed, tab, comps[:1] if comps[1] == "none" else comps, f=f, box_len=n * dx)
        if comps[1] == "none":
            assert np.all(g[..., 1] == 0.0)
        # the pair is one complex transform: its rounding goes with the pair's size
        assert rel_rms(np.stack([g[..., 0], g[..., 1]]), np.stack([ref.real, ref.imag])) < TOL
