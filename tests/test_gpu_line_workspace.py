"""Workspaces of the calls that sum over lines: no bytes past the size that the
size calls give are touched, with one partial sum and with several, and the
tuning workspace holds what its kernels write, not per-line bin counts as well."""
import numpy as np
import pytest

from tests.test_gpu_line_spectra import DPIX, k_bins, line_table
from tests.test_gpu_p1d import L, bin_sums, smooth_flux  # noqa: F401
from tests.test_gpu_tune import Spec

pytestmark = pytest.mark.gpu
PAD = 4096


def _guarded(size):
    import torch
    buf = torch.full((size + PAD,), 0x5A, dtype=torch.uint8, device="cuda")
    return buf, buf[:size]


@pytest.mark.parametrize("n_sk", [1, 255, 256, 700, 17000])
@pytest.mark.parametrize("nk", [1, 64])
def test_nothing_beyond_the_workspace(L, n_sk, nk):  # noqa: F811
    import torch
    print("workspace of %d lines, %d bins" % (n_sk, nk), flush=True)
    rng = np.random.default_rng([n_sk, nk])
    sk = line_table(rng.integers(0, 40, n_sk), nk)
    flux = smooth_flux(sk["total"] + 1, nk)
    sp = Spec(L, sk, flux - 1.0, flux - 1.0, k_bins(nk), [2.4], [1.1], [0.8], np.ones((1, nk)))
    size = L.tune_workspace_size(n_sk, nk)
    buf, work = _guarded(size)
    draws = np.array([[0.3, 1.4, 1.1, 2.0 + 0.1 * i] for i in range(9)])   # a full launch and one more
    y = torch.zeros((9, nk + 1), dtype=torch.float32, device="cuda")
    L.emulator_labels(sp.spec, draws, y, work)
    torch.cuda.synchronize()
    assert bool((buf[size:] == 0x5A).all())
    edges = np.array([0.0, 9000.0])
    fsum, cnt = bin_sums(flux, sk, edges)
    f, e, s, c, ke = (torch.from_numpy(np.asarray(v)).cuda() for v in
                      (flux.astype(np.float32), edges, fsum.astype(np.float64), cnt.astype(np.int64), k_bins(nk)))
    psum = torch.zeros(nk, dtype=torch.float64, device="cuda")
    pcount = torch.zeros(nk, dtype=torch.int64, device="cuda")
    size = L.p1d_workspace_size(n_sk, nk)
    buf, work = _guarded(size)
    L.p1d(sp.s, L.Cosmo(0.3147), f, L.zbins_struct(e, s, c), L.P1dSpec(nk, ke.data_ptr(), 2.4, DPIX), psum, pcount, work)
    torch.cuda.synchronize()
    assert bool((buf[size:] == 0x5A).all())


def test_tuning_workspace_is_what_the_kernels_write(L):  # noqa: F811
    # 8 draws' sums of 64 bins and of F per line, FP64, and about 1 MB besides
    n = 1_000_000
    assert L.tune_workspace_size(n, 64) < 8 * n * 65 * 8 + (4 << 20)
