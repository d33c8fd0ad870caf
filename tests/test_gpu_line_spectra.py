"""GPU parity of the 1D power and of the tuning evaluation at the edges of their
work split: bin counts that give a bin 8, 4, 2 or 1 lanes, one line and many (one
to 128 partial sums, pulls of one and of several lines), lines without a
transform, of one mode, of every power of two up to the 2048-pixel cap and
beyond it, k bins that start at the first mode or end at the last, and 64
distance bins."""
import numpy as np
import pytest

from oracle import cosmology, fgpa, p1d, tune
from tests.lyahelp import rel_rms
from tests.test_gpu_p1d import L, bin_sums, run_gpu, smooth_flux  # noqa: F401
from tests.test_gpu_tune import Spec

pytestmark = pytest.mark.gpu
DPIX = 0.2
# FP32 transforms of at most 2^10 points: 11 eps log2-stages of 2^-24 each on
# amplitudes, twice that on powers, below 2e-6 of the rms power
TOL = 1e-5


def line_table(npix, seed, gap=1):
    rng = np.random.default_rng([seed, 17])
    n = len(npix)
    npix = np.asarray(npix, np.int32)
    offset = np.zeros(n, np.int64)
    offset[1:] = np.cumsum(npix[:-1].astype(np.int64) + gap)
    chi0 = np.array([cosmology.chi_of_z(z) for z in np.linspace(2.0, 3.5, 64)])[rng.integers(0, 64, n)]
    return dict(npix=npix, offset=offset, chi0=chi0, dchi=DPIX, id_base=0, origin_fx=np.zeros((n, 3), np.int64),
                step_fx=np.zeros((n, 3), np.int64), total=int(offset[-1] + npix[-1]))


def lengths(n, top, seed):
    edge = [0, 1, 2, 3, 4, 7, 8, 31, 32, 127, 128, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 2600]
    out = [v for v in edge if v <= top][:n]
    rng = np.random.default_rng([seed, 18])
    out = np.concatenate([out, rng.integers(0, min(top, 40) + 1, n - len(out))]).astype(np.int32)
    return rng.permutation(out)


def k_bins(nk):
    """From below the first mode of the longest line to the last mode of any."""
    dv = p1d.dv_pixel(2.4, DPIX)
    return p1d.log_k_edges(nk, 0.97 * 2.0 * np.pi / (2048 * dv), 1.01 * np.pi / dv)


@pytest.mark.parametrize("n_sk,top,nk,nz", [(1, 0, 1, 1), (3, 1, 8, 2), (24, 2600, 8, 64), (255, 2600, 9, 3),
                                            (256, 600, 16, 64), (300, 2600, 17, 8), (520, 130, 32, 1),
                                            (24, 2600, 33, 63), (6300, 64, 64, 64), (20000, 32, 64, 2)])
def test_p1d_at_the_edges(L, n_sk, top, nk, nz):  # noqa: F811
    print("p1d lines %d up to %d pixels, %d k bins, %d distance bins" % (n_sk, top, nk, nz), flush=True)
    sk = line_table(lengths(n_sk, top, n_sk + nk), nk)
    flux = smooth_flux(sk["total"] + 1, nk)
    edges = np.sort(fgpa.chi_edges_for_z(np.linspace(1.9, 3.4, nz + 1)))
    fsum, cnt = bin_sums(flux, sk, edges)
    ps, pc = run_gpu(L, sk, flux, edges, fsum, cnt, k_bins(nk), 2.4, DPIX)
    fmean = np.where(cnt > 0, fsum / np.maximum(cnt, 1), 1.0)
    ps_r, pc_r = p1d.p1d(flux, sk, edges, fmean, k_bins(nk), 2.4, DPIX)
    np.testing.assert_array_equal(pc, pc_r)
    assert np.all(ps[pc_r == 0] == 0.0)
    assert rel_rms(ps, ps_r) < TOL or not np.any(ps_r)


@pytest.mark.parametrize("n_sk,top,nk", [(1, 2, 1), (24, 2600, 8), (255, 2600, 16), (300, 600, 32), (24, 2600, 64),
                                         (4000, 64, 33)])
def test_tuning_statistics_at_the_edges(L, n_sk, top, nk):  # noqa: F811
    import torch
    print("tuning statistics of %d lines up to %d pixels, %d k bins" % (n_sk, top, nk), flush=True)
    sk = line_table(lengths(n_sk, top, n_sk) if n_sk > 1 else [2], nk, gap=0)
    rng = np.random.default_rng([nk, 19])
    dens = rng.normal(0.0, 1.0, sk["total"]).astype(np.float32)
    eta = rng.normal(0.0, 0.2, sk["total"]).astype(np.float32)
    sp = Spec(L, sk, dens, eta, k_bins(nk), [2.4], [1.1], [0.8], np.ones((1, nk)))
    draws = np.array([[0.3, 1.4, 1.1, 2.0 + 0.15 * i] for i in range(9)])
    y = torch.full((len(draws), nk + 1), -1.0, dtype=torch.float32, device="cuda")
    L.emulator_labels(sp.spec, draws, y, sp.work)
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    for i, (a, b, c, z) in enumerate(draws):
        if i not in (0, 7, 8):   # the first and last of a full launch, and the draw of the next
            continue
        fb, pk = tune.evaluate(dens, eta, sk, a, b, c, z, k_bins(nk), DPIX)
        assert abs(y[i, 0] / fb - 1) < TOL
        have = np.isfinite(pk)
        np.testing.assert_array_equal(np.isfinite(y[i, 1:]), have)
        assert rel_rms(y[i, 1:][have], pk[have]) < TOL or not have.any()
