"""Tuning the skewer launch shape on few skewers, which every shape launches
alike, leaves the table as it was: times that differ by noise alone choose
nothing for later, larger calls."""
import pytest
import torch

import mockinputs
from tests.lyahelp import skewer_tensors
from tests.test_gpu_skewers import L  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sk", [1, 500])
def test_same_launches_choose_nothing(L, n_sk):  # noqa: F811
    print("autotune on few skewers", n_sk, flush=True)
    n = 64
    cfg = mockinputs.config("mid", n=n, n_sk=n_sk)
    sk = mockinputs.skewer_table(cfg)
    s, keep = skewer_tensors(L, sk)
    box = L.box_struct(n, 2.19)
    field = torch.zeros((L.field_elems(box), 2), dtype=torch.float32, device="cuda")
    out = [torch.empty(sk["total"], dtype=torch.float32, device="cuda") for _ in range(3)]
    work = torch.empty(L.workspace_size(L.LYA_OP_SKEWERS, box), dtype=torch.uint8, device="cuda")
    saved = L.get_tuning(n)
    shape = lambda t: (t.sk_chunk, t.sk_blocks_per_cu, t.sk_unroll)  # noqa: E731
    try:
        for was in (shape(saved), (8, 3, 2), (1000, 4, 1)):
            L.set_tuning(n, L.Tuning(saved.fft_y, saved.fft_x, *was))
            t, ms = L.autotune_skewers(box, field, s, L.Ps1d(1.0, 1.5, 0.2, 0), 5, L.Cosmo(cfg["omega_m"]),
                                       L.fgpa_struct(cfg["fgpa"]), *out, None, work, reps=1)
            assert all(x > 0 for a in ms for b in a for x in b)
            assert shape(t) == was and shape(L.get_tuning(n)) == was
    finally:
        L.set_tuning(n, saved)
