"""The quasar draw in boxes that reach past the horizon (omega_m = 0.7: no redshift
has a distance above 7010 Mpc/h, and the z(chi) table holds no numbers from 6800
on): voxels without a redshift have no p and are taken, as by the full evaluation,
also where a voxel near them has one; voxels up to z = 50 follow the oracle."""
import numpy as np
import pytest
import torch

from oracle import quasars
from tests.test_gpu_quasar_bound import NZ, case
from tests.test_gpu_quasars import L, _dev, _voxel_ids  # noqa: F401

pytestmark = pytest.mark.gpu
OM = 0.7


@pytest.mark.parametrize("n_box", [1, 3])
@pytest.mark.parametrize("dx", [38.9, 90.0])
def test_voxels_without_a_redshift(L, n_box, dx):  # noqa: F811
    n = 32
    print("horizon, %d boxes, dx %g" % (n_box, dx), flush=True)
    f, var, _, zb = case(n, dx, n_box, "outside", 6)
    span = (n - 1) * dx
    obs = np.array([0.5 * span, 0.3 * span, span - 7100.0])
    box = L.box_struct(n, dx)
    boxes = []
    for c in ([f[:2], f[2:]] if n_box == 3 else [f]):
        b = torch.zeros((L.field_elems(box), 2), dtype=torch.float32, device="cuda")
        for i, x in enumerate(c):
            L.box_view(b, n)[..., i].copy_(torch.from_numpy(x))
        boxes.append(b)
    vt, nb = _dev(var), 1e-9 * np.array([1.0, 3.0, 2.0, 0.5, 0.1])
    spec = L.qso_spec(boxes, zb, [vt.data_ptr() + 8 * i for i in range(len(var))], obs, _dev(NZ), _dev(nb), 95,
                      0.82 if n_box == 3 else 0.0)
    work = torch.empty(L.workspace_size(L.LYA_OP_QUASARS, box), dtype=torch.uint8, device="cuda")
    pos = torch.zeros((n ** 3, 3), dtype=torch.int64, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    L.draw_quasars(box, spec, L.Cosmo(OM), pos, cnt, work)
    gid = np.sort(_voxel_ids(pos[:int(cnt.item())].cpu().numpy(), n))
    assert np.all(np.diff(gid) > 0)
    lin = np.arange(n ** 3)
    x = np.stack([lin // (n * n), (lin // n) % n, lin % n], axis=1) * dx - obs
    chi = np.sqrt(np.sum(x * x, axis=1))
    far, near = lin[chi > 6900.0], lin[chi < 5970.0]
    assert len(far) > 100 and (dx < 80 or len(near) > 1000)
    assert np.all(np.isin(far, gid))
    if len(near):
        p, _ = quasars.probability_at(near, [v.reshape(-1)[near].astype(np.float64) for v in f], n, dx, obs, zb, var,
                                      NZ, nb, xi5=0.82 if n_box == 3 else None, omega_m=OM)
        u, got = quasars.decision_uniforms_at(95, near), np.isin(near, gid)
        assert np.all(got[u < p * (1 - 1e-5) - 1e-9]) and not np.any(got[u > p * (1 + 1e-5) + 1e-9])
