"""The quasar draw from boxes that start on any cell: 8-byte aligned ones give the
catalogue that 16-byte aligned ones give."""
import numpy as np
import pytest
import torch

from oracle import cosmology
from tests.test_gpu_quasar_bound import NZ, case
from tests.test_gpu_quasars import L, _dev, _voxel_ids  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_box", [1, 3])
@pytest.mark.parametrize("off_a,off_b", [(1, 0), (0, 1), (1, 1)])
def test_boxes_on_any_cell(L, n_box, off_a, off_b):  # noqa: F811
    print("quasar boxes off by %d, %d cells, %d boxes" % (off_a, off_b, n_box), flush=True)
    n, dx = 64, 10.0
    f, var, obs, zb = case(n, dx, n_box, "outside", 4)
    box = L.box_struct(n, dx)
    work = torch.empty(L.workspace_size(L.LYA_OP_QUASARS, box), dtype=torch.uint8, device="cuda")
    comps = [f[:2] if n_box == 3 else f[:1], f[2:]]
    vt, nz, nb = _dev(var), _dev(NZ), _dev(1e-5 * np.array([1.0, 3.0, 2.0, 0.5, 0.1]))
    out = []
    for offs in ((0, 0), (off_a, off_b)):
        boxes = []
        for c, o in zip(comps[:1 if n_box == 1 else 2], offs):
            b = torch.zeros((L.field_elems(box) + o, 2), dtype=torch.float32, device="cuda")[o:]
            v = L.box_view(b, n)
            for i, x in enumerate(c):
                v[..., i].copy_(torch.from_numpy(x))
            assert b.data_ptr() % 16 == 8 * o
            boxes.append(b)
        spec = L.qso_spec(boxes, zb, [vt.data_ptr() + 8 * i for i in range(len(var))], obs, nz, nb, 94,
                          0.82 if n_box == 3 else 0.0)
        pos = torch.zeros((n ** 3, 3), dtype=torch.int64, device="cuda")
        cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
        L.draw_quasars(box, spec, L.Cosmo(cosmology.OMEGA_M), pos, cnt, work)
        p = pos[:int(cnt.item())].cpu().numpy()
        out.append(p[np.argsort(_voxel_ids(p, n))])
    assert len(out[0]) > 100
    np.testing.assert_array_equal(out[0], out[1])
