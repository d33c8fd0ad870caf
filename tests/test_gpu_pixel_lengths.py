"""Pixel lengths that put a line's next pixel far outside the z(chi) table: the
redshift of every pixel of such a line is still the table's, continued linearly
beyond its ends.  Lengths of which (pixels + 127) steps make a whole number of
turns of the kernel's 64-bit table positions are among them."""
import numpy as np
import pytest

from oracle import cosmology, fgpa
from tests.lyahelp import gpu_skewers, padded_box
from tests.test_gpu_skewers import L  # noqa: F401

pytestmark = pytest.mark.gpu
# constant a, b = 0: F = exp(-(a0 + a1 (1+z))), a function of z alone
COEF = [[0.5, 0.5, 0.0], [0.0, 0.0, 0.0], [0.0, 0.0, 0.0]]
TAB_END = 10000.0


# (npix + 127) dchi 2^33 is a multiple of 2^64 for the powers of two here
@pytest.mark.parametrize("npix,dchi", [(1, 2.0 ** 24), (129, 2.0 ** 23), (385, 2.0 ** 22), (1, 1.0e9), (1, 3.0e4),
                                       (65, 70.0), (2048, 5.0), (1, 0.0)])
def test_pixel_lengths_beyond_the_table(L, npix, dchi):  # noqa: F811
    print("pixel length", npix, dchi, flush=True)
    S, empty = 40, 5000                        # more lines than waves: the cell walk
    chi0 = cosmology.chi_of_z(np.linspace(2.0, 3.4, S))
    sk = dict(origin_fx=np.zeros((S + empty, 3), np.int64), step_fx=np.zeros((S + empty, 3), np.int64),
              npix=np.concatenate([np.full(S, npix), np.zeros(empty)]).astype(np.int32),
              offset=np.minimum(np.arange(S + empty, dtype=np.int64), S) * npix,
              chi0=np.concatenate([chi0, np.full(empty, chi0[0])]), dchi=dchi, id_base=0, total=S * npix)
    field = padded_box(L, np.zeros((32, 32, 32, 2), np.float32))
    out = gpu_skewers(L, field, 32, 1.0, sk, 1, 0.0, 1.5, 0.2, COEF)
    flux = out["flux"].reshape(S, npix)
    # the pixels within the table (the first one always is)
    inside = (chi0[:, None] - np.arange(npix) * dchi) >= 0.0
    assert inside[:, 0].all() and chi0.max() < TAB_END
    chi = np.where(inside, chi0[:, None] - np.arange(npix) * dchi, chi0[:, None])
    ref = np.exp(-(0.5 + 0.5 * (1.0 + cosmology.z_of_chi(chi.ravel()).reshape(chi.shape))))
    # F32: x = 1 + z to 2^-23, exponent about 2: 1e-6; the table's interpolation adds 1e-7
    assert np.max(np.abs(flux / ref - 1.0)[inside]) < 3e-6
    # beyond the table z continues the first interval linearly: F grows without
    # limit there (as far as 64-bit positions reach, 2^30 Mpc/h)
    beyond = ~inside & (np.arange(npix) * dchi < 2.0 ** 30)
    assert np.all(flux[beyond] > np.exp(-1.0)) and not np.isnan(flux[inside]).any()
