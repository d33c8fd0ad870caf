"""The amplitude table's first launch in its forms: an analytic spectrum (sigma8
sums, then twiddles), a tabulated one (twiddles only), and both in one pair box,
where the second table must not disturb the first, at the smallest box (fewer
twiddles than a block has threads) and at one with several blocks of them."""
import numpy as np
import pytest

from oracle import field, power
from tests.lyahelp import rel_rms
from tests.test_gpu_box import PK, L  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-5   # of every box against the oracle: FP32 amplitudes, noise and transform


@pytest.mark.parametrize("n", [32, 64])
@pytest.mark.parametrize("kinds", ["aa", "at", "ta", "tt"])
def test_pair_of_tables(L, n, kinds):  # noqa: F811
    dx, seed = 2.19, 71
    print("pair box %d^3, tables %s" % (n, kinds), flush=True)
    k = np.exp(np.linspace(np.log(1e-4), np.log(30.0), 400))
    p = 3e4 * k / (1.0 + (k / 0.02) ** 2) ** 1.3
    kt, pt = torch.from_numpy(k).cuda(), torch.from_numpy(p).cuda()
    sig = dict(PK, sigma8=0.7)
    specs = [(L.pk_struct(**(PK if i == 0 else sig)), power.PowerSpectrum(**(PK if i == 0 else sig)))
             if c == "a" else (L.pk_struct(k_tab=kt, p_tab=pt), power.TabulatedPower(k, p))
             for i, c in enumerate(kinds)]
    box = L.box_struct(n, dx)
    work = torch.empty(L.workspace_size(L.LYA_OP_BOX, box), dtype=torch.uint8, device="cuda")
    fld = torch.empty((L.field_elems(box), 2), dtype=torch.float32, device="cuda")
    L.make_box_pair(box, specs[0][0], specs[1][0], seed, fld, work)
    torch.cuda.synchronize()
    got = L.box_view(fld, n).cpu().numpy()
    for c in range(2):
        ref = field.make_box(n, seed, power.amplitude_table(specs[c][1], n, dx), ("delta",))
        assert rel_rms(got[..., c], np.real(ref)) < TOL
