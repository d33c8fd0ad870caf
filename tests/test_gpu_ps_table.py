"""Amplitudes of delta_S from the per-call table: every line length class (2 to
2048 pixels), with and without a tabulated ratio (bin edges on modes, below the
first and past the last), fixed amplitudes; against the oracle."""
import numpy as np
import pytest
import torch

from oracle import skewers
from tests.lyahelp import gpu_skewers, padded_box, skewer_tensors
from tests.test_gpu_skewers import L  # noqa: F401

pytestmark = pytest.mark.gpu
NPIX = np.array([2, 3, 4, 5, 8, 9, 16, 31, 33, 64, 100, 200, 256, 500, 513, 1024, 1025, 2047, 2048], np.int32)


def _table():
    off = np.concatenate([[0], np.cumsum(NPIX[:-1].astype(np.int64))])
    z = np.zeros((len(NPIX), 3), np.int64)
    return dict(origin_fx=z, step_fx=z, npix=NPIX, offset=off, chi0=np.full(len(NPIX), 4000.0), dchi=0.2, id_base=9,
                total=int(NPIX.sum()))


@pytest.mark.parametrize("fixed", [False, True])
def test_plain(L, fixed):  # noqa: F811
    sk, n = _table(), 32
    out = gpu_skewers(L, padded_box(L, np.zeros((n, n, n, 2), np.float32)), n, 1.0, sk, 21, 1.3, 1.5, 0.2,
                      want=("dens",), ps_fixed=fixed)
    for q, m in enumerate(NPIX):
        o = sk["offset"][q]
        ref = skewers.delta_s(21, 9 + q, int(m), 0.2, 1.3, 1.5, fixed)
        # P_s below FP32's range (2^-126; lines of 2 pixels hold k = 10 kcut alone) is an amplitude below 1.1e-19
        err = np.linalg.norm(out["dens"][o:o + m].astype(np.float64) - ref)
        assert err <= 1e-5 * np.linalg.norm(ref) + 1e-18, (q, m, err)


def test_ratio_scales_every_mode(L):  # noqa: F811
    # a ratio that is the same in every bin scales delta_S by its root, whatever the bin a mode falls into;
    # edges on modes of the longest line, the first above k_1 and the last below the highest modes
    sk = _table()
    edges = torch.from_numpy(2 * np.pi / (2048 * 0.2) * np.array([3.0, 10.0, 64.0, 200.0, 700.0])).cuda()
    s, keep = skewer_tensors(L, sk)
    zero = torch.zeros(sk["total"], dtype=torch.float32, device="cuda")
    work = torch.empty(L.workspace_size(L.LYA_OP_SKEWERS), dtype=torch.uint8, device="cuda")
    flux = torch.empty_like(zero)
    coef = [[1.0, 0.0, 0.0], [1.0, 0.0, 0.0], [0.0, 0.0, 0.0]]   # F = exp(-exp(delta_S))

    def draw(ratio):
        r = torch.tensor(ratio, dtype=torch.float32, device="cuda")
        t = L.PsTable(4, edges.data_ptr(), r.data_ptr())
        L.apply_fgpa_ds(s, L.Cosmo(0.3147), zero, zero, L.Ps1d(0.01, 1.5, 0.2, 0), t, 21, L.fgpa_struct(coef), flux,
                        None, work)
        return torch.log(-torch.log(flux.double())).cpu().numpy()
    one, four = draw([1.0] * 4), draw([4.0] * 4)
    for q, m in enumerate(NPIX):
        o = sk["offset"][q]
        ref = skewers.delta_s(21, 9 + q, int(m), 0.2, 0.01, 1.5)[:m]
        # FP32 fluxes around exp(-1): 6e-8 of F, two exponentials of 2 units in the last place, over |ln F| > 0.4
        assert np.max(np.abs(one[o:o + m] - ref)) < 2e-6 and np.max(np.abs(four[o:o + m] - 2 * ref)) < 2e-6, (q, m)
    # only the lowest bin raised: the lines too short for its modes stay as they were
    low = draw([4.0, 1.0, 1.0, 1.0])
    o = sk["offset"][0]
    np.testing.assert_array_equal(low[o:o + 13], one[o:o + 13])
    o = sk["offset"][-1]
    assert np.max(np.abs(low[o:] - one[o:])) > 1e-4
