"""The transforms of lya_lognormal_pk against the same quadratures summed node
by node in FP64, at the edges of the kernel's node groups (32), lanes (256) and
segments (one segment writes the caller's arrays directly)."""
import numpy as np
import pytest

from oracle import cosmology, power, quasars

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_18996_amd import lyamock
    lyamock.load()
    return lyamock


def _sines(f, nodes, x, chunk=1 << 22):
    """sum_j f_j sin(nodes_j x) / x (x = 0: sum_j f_j nodes_j)."""
    out = np.empty(len(x))
    step = max(1, chunk // len(nodes))
    for s in range(0, len(x), step):
        xs = x[s:s + step]
        with np.errstate(all="ignore"):
            out[s:s + step] = np.where(xs > 0, (np.sin(np.outer(xs, nodes)) @ f) / xs, f @ nodes)
    return out


@pytest.mark.parametrize("n_r,n_k,rmax", [(3, 1, 40.0), (31, 2, 40.0), (33, 257, 300.0), (255, 64, 300.0),
                                          (4097, 65, 700.0), (33, 300001, 20.0), (262145, 5, 5.0)])
def test_sums(L, n_r, n_k, rmax):
    import torch
    s = 2.19
    k = np.linspace(0.0, 1.5, n_k)   # k = 0 is the limit
    kt = torch.from_numpy(k).cuda()
    pq, xi = torch.empty_like(kt), torch.empty(n_r, dtype=torch.float64, device="cuda")
    work = torch.empty(L.lognormal_workspace_size(s, rmax, n_r), dtype=torch.uint8, device="cuda")
    print("n_r %d n_k %d rmax %g" % (n_r, n_k, rmax), flush=True)
    L.lognormal_pk(L.pk_struct(smooth=s), 2.75, 2.75, L.Cosmo(cosmology.OMEGA_M), rmax, n_r, kt, pq, xi, work)
    pq, xi = pq.cpu().numpy(), xi.cpu().numpy()
    # xi: Simpson on k_j = j h
    kmax = 12.0 / s
    m = int(2 * np.ceil(kmax / (2 * min(0.1 / rmax, kmax / 64.0))))
    h = kmax / m
    kj = h * np.arange(1, m + 1)
    w = np.where(np.arange(1, m + 1) % 2 == 1, 4.0, 2.0)
    w[-1] = 1.0
    f = w * h / 3 * power.PowerSpectrum()(kj) * np.exp(-(kj * s) ** 2) * kj
    r = rmax / (n_r - 1) * np.arange(n_r)
    want = _sines(f, kj, r) / (2 * np.pi ** 2)
    # phases up to kmax rmax are rounded a few times (4 units in the last place)
    # and turned up to 48 times from an exact one; the spectrum itself to 1e-12
    eps = 2.0 ** -53

    def bound(f, nodes, x, span):
        return np.sum(np.abs(f) * np.minimum(nodes, 1.0 / max(x, 1e-300))) * (1e-12 + eps * (4 * span + 64))
    tol = np.array([bound(f, kj, v, kmax * rmax) for v in r[:: max(1, n_r // 64)]]) / (2 * np.pi ** 2)
    got, ref = xi[:: max(1, n_r // 64)], want[:: max(1, n_r // 64)]
    assert np.all(np.abs(got - ref) <= tol), float(np.max(np.abs(got - ref) / tol))
    # P_q from the library's own xi, so that only this sum is compared
    wr = np.where(np.arange(n_r) % 2 == 1, 4.0, 2.0)
    wr[0] = wr[-1] = 1.0
    g = wr * (r[1] / 3) * np.log1p(quasars.box_bias2(2.75, 2.75) * xi) * r
    want = 4 * np.pi * _sines(g, r, k)
    want = np.maximum(want, 1e-12 * want.max())
    at = np.arange(0, n_k, max(1, n_k // 64))
    tol = np.array([bound(g, r, v, 1.5 * rmax) for v in k[at]]) * 4 * np.pi
    assert np.all(np.abs(pq[at] - want[at]) <= tol), float(np.max(np.abs(pq[at] - want[at]) / tol))
