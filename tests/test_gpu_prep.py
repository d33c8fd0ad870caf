"""The z(chi) table every skewer and FGPA call builds (a group of 16 lanes per
node, started on a Gauss-Legendre rule) against the rule it stands for: Newton
on the 128-interval Simpson chi(z), node by node in FP64."""
import numpy as np
import pytest

from oracle import cosmology

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_18996_amd import lyamock
    lyamock.load()
    return lyamock


def _simpson_z(chi, om):
    """z with (c/H0) Simpson_128[1/E on [0, z]] = chi."""
    w = np.where(np.arange(129) % 2 == 1, 4.0, 2.0)
    w[0] = w[-1] = 1.0
    z = chi / cosmology.C_OVER_H0
    for _ in range(30):
        s = np.sum(w / cosmology.hubble_e(z[:, None] / 128 * np.arange(129), om), axis=1)
        z = z - (s * z / 384 - chi / cosmology.C_OVER_H0) * cosmology.hubble_e(z, om)
    return z


@pytest.mark.parametrize("om", [0.05, 0.3147, 1.0])
def test_pixel_redshifts(L, om):
    """-ln F = a(z) = (1 + z)/10 with b = 0: pixels on the table's nodes and
    half-way between them, from the observer to z = 10 (or 6000 Mpc/h)."""
    import torch
    npix, dchi = 2048, 0.25
    chi_max = min(6000.0, float(cosmology.chi_of_z(np.array([10.0]), om)[0]))
    n_sk = int(chi_max / (npix * dchi))
    chi0 = (np.arange(n_sk) + 1) * npix * dchi - dchi   # down to 0 in all
    print("om %.4f: %d skewers to %.1f Mpc/h" % (om, n_sk, chi0[-1]), flush=True)
    dev = dict(npix=torch.full((n_sk,), npix, dtype=torch.int32, device="cuda"),
               offset=torch.arange(n_sk, device="cuda") * npix, chi0=torch.from_numpy(chi0).cuda())
    s = L.skewers_struct(n_sk, None, None, dev["npix"], dev["offset"], dev["chi0"], dchi)
    z0 = torch.zeros(n_sk * npix, dtype=torch.float32, device="cuda")
    flux = torch.empty_like(z0)
    work = torch.empty(L.workspace_size(L.LYA_OP_SKEWERS), dtype=torch.uint8, device="cuda")
    L.apply_fgpa(s, L.Cosmo(om), z0, z0, L.fgpa_struct([[0.0, 0.1, 0.0], [0.0, 0, 0], [0.0, 0, 0]]), flux, None, work)
    got = -np.log(flux.cpu().numpy().astype(np.float64)) / 0.1
    chi = (chi0[:, None] - np.arange(npix) * dchi).ravel()
    lo = np.floor(chi / 0.5) * 0.5
    z_lo, z_hi = _simpson_z(lo, om), _simpson_z(lo + 0.5, om)
    want = 1.0 + z_lo + (chi - lo) / 0.5 * (z_hi - z_lo)
    # rounding: 2.4e-7 in ln F (F and the exponential, two units in the last
    # place) over 0.1, and 4e-7 relative in a (table, interpolation, polynomial)
    tol = 3e-6 + 4e-7 * want
    assert np.all(np.abs(got - want) <= tol), float(np.max(np.abs(got - want) / tol))
