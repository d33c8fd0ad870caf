"""Every line of a call is taken exactly once, whatever the split of the lines over
the work queue: fewer lines than waves, one more than the waves of a full grid,
pulls of several lines, a last pull that is not full, and lengths under which all
the work falls to one of the queue's 16 counters, so that the waves of the others
go on with it."""
import numpy as np
import pytest

import mockinputs
from oracle import cosmology, fgpa
from tests.lyahelp import FBAR_RTOL, fbar_bin_err, gpu_apply_fgpa, rel_rms
from tests.test_gpu_skewers import L  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sk,every,length", [(1, 1, 1), (3, 1, 5), (4095, 1, 2), (4096, 1, 1), (4097, 1, 3),
                                               (8 * 4096, 1, 1), (65537, 1, 1), (262144 + 7, 1, 1),
                                               (8192, 16, 200), (9001, 32, 700)])
def test_every_line_once(L, n_sk, every, length):  # noqa: F811
    print("%d lines, every %d-th of %d pixels" % (n_sk, every, length), flush=True)
    cfg = mockinputs.config("tiny")
    npix = np.zeros(n_sk, np.int32)
    npix[::every] = length
    offset = np.concatenate([[0], np.cumsum(npix[:-1].astype(np.int64))])
    z = np.linspace(2.0, 3.4, 257)
    chi0 = cosmology.chi_of_z(z)[np.arange(n_sk) % 257]
    sk = dict(npix=npix, offset=offset, chi0=chi0, dchi=mockinputs.DPIX, id_base=0,
              origin_fx=np.zeros((n_sk, 3), np.int64), step_fx=np.zeros((n_sk, 3), np.int64), total=int(npix.sum()))
    rng = np.random.default_rng([n_sk, 5])
    dens = rng.normal(0.0, 1.0, sk["total"]).astype(np.float32)
    eta = rng.normal(0.0, 0.2, sk["total"]).astype(np.float32)
    edges = fgpa.chi_edges_for_z(np.linspace(1.8, 3.5, 9))
    out = gpu_apply_fgpa(L, sk, dens, eta, cfg["fgpa"], edges)
    ref, _ = fgpa.apply_fgpa(dens, eta, sk, cfg["fgpa"])
    assert rel_rms(out["flux"], ref) < 1e-5        # a pixel never written is NaN
    fs, cnt = fgpa.mean_flux_bins(ref, fgpa.pixel_chi(sk, sk["total"]), edges)
    np.testing.assert_array_equal(out["count"], cnt)   # a line taken twice counts twice
    assert fbar_bin_err(out["fsum"], fs, cnt) <= FBAR_RTOL
