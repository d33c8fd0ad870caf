"""One bfloat16 training batch of the emulator at the edges of its row blocks
(4, 8 or 16 rows a block by the batch), MFMA steps (16 rows) and output tiles
(16 columns), against the same products of bfloat16-rounded operands in FP64;
and Adam's step with the packed weights it keeps."""
import numpy as np
import pytest

from oracle import mlp
from tests.lyahelp import rel_rms
from tests.test_gpu_tune import _new_emulator, _oracle_params, _upload_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_18996_amd import lyamock
    lyamock.load()
    return lyamock


def _bf(x):
    """Rounded to bfloat16 (nearest even), FP64."""
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


def _batch(params, x0, t):
    """Loss and gradients with the hidden and output products on bfloat16
    operands (the first layer and the bias sums take FP32 ones)."""
    W, b = params[0::2], params[1::2]
    z = [x0 @ W[0] + b[0]]
    h = [mlp.gelu(z[0])]
    for l in (1, 2):
        z.append(_bf(h[-1]) @ _bf(W[l]) + b[l])
        h.append(mlp.gelu(z[-1]))
    y = _bf(h[2]) @ _bf(W[3]) + b[3]
    loss = np.mean((y - t) ** 2)
    d = 2.0 * (y - t) / t.size
    grads = [None] * 8
    for l in (3, 2, 1):
        grads[2 * l], grads[2 * l + 1] = _bf(h[l - 1]).T @ _bf(d), d.sum(0)
        d = (_bf(d) @ _bf(W[l]).T) * mlp.gelu_grad(z[l - 1])
    grads[0], grads[1] = x0.T @ d, d.sum(0)
    return loss, grads


@pytest.mark.parametrize("batch,n_out", [(1, 1), (3, 64), (4, 16), (5, 17), (17, 33), (63, 15), (64, 48), (65, 1),
                                         (1024, 33), (1025, 16), (2049, 17)])
def test_gradients_at_the_edges(L, batch, n_out):
    import torch
    print("batch %d n_out %d" % (batch, n_out), flush=True)
    params = _oracle_params(3, n_out)
    emu = _new_emulator(L, n_out, n_out)
    _upload_params(L, emu, params)
    rng = np.random.default_rng(batch * 100 + n_out)
    x0 = rng.uniform(-1, 1, (batch, 4)).astype(np.float32)
    t = rng.normal(size=(batch, n_out)).astype(np.float32)
    loss_r, grads_r = _batch(params, x0.astype(np.float64), t.astype(np.float64))
    g = torch.full((L.emulator_param_count(n_out),), float("nan"), dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    work = torch.empty(L.emulator_train_workspace_size(batch, n_out), dtype=torch.uint8, device="cuda")
    L.emulator_loss_grad(emu, torch.from_numpy(x0).cuda(), torch.from_numpy(t).cuda(), batch, True, g, loss, work)
    g = g.cpu().numpy().astype(np.float64)
    # FP32 sums differ by some 2^-24 sqrt(256) ~ 1e-6 relative, which moves about
    # one operand in 500 across a bfloat16 rounding (2^-9 of it): 2^-9 / sqrt(500)
    # ~ 1e-4 of a gradient at worst; ten times that is allowed for small batches
    o = 0
    for k, gr in enumerate(grads_r):
        e = rel_rms(g[o:o + gr.size], gr.reshape(-1))
        assert e < 1e-3, (k, e)
        o += gr.size
    assert abs(loss.item() / loss_r - 1) < 1e-3


@pytest.mark.parametrize("batch,n_out", [(16, 33), (130, 17), (1030, 5)])
def test_training_steps_use_the_updated_weights(L, batch, n_out):
    import torch
    params = _oracle_params(5, n_out)
    emu = _new_emulator(L, n_out, n_out)
    p0 = _upload_params(L, emu, params)
    rng = np.random.default_rng(batch)
    n = 2 * batch
    x = torch.from_numpy(rng.uniform(-1, 1, (n, 4)).astype(np.float32)).cuda()
    y = torch.from_numpy(rng.normal(size=(n, n_out)).astype(np.float32)).cuda()
    work = torch.empty(L.emulator_train_workspace_size(batch, n_out), dtype=torch.uint8, device="cuda")
    g = torch.zeros(p0.size, dtype=torch.float32, device="cuda")
    losses = []
    one = torch.zeros(1, dtype=torch.float32, device="cuda")
    both = emu.clone()
    hist = torch.zeros(2, dtype=torch.float32, device="cuda")
    L.emulator_train(both, x, y, n, 2, batch, 1e-3, True, hist, work)
    off = L.emulator_param_offset()
    for s in range(2):   # the same steps one call at a time, each gradient seen first
        L.emulator_loss_grad(emu, x[s * batch:], y[s * batch:], batch, True, g, one, work)
        losses.append(one.item())
        before = emu[off:off + 4 * p0.size].view(torch.float32).cpu().numpy().astype(np.float64)
        L.emulator_train(emu, x, y, n, 1, batch, 1e-3, True, None, work)
        if s == 0:   # Adam's first step: lr g / (|g| + eps)
            gg = g.cpu().numpy().astype(np.float64)
            after = emu[off:off + 4 * p0.size].view(torch.float32).cpu().numpy().astype(np.float64)
            # the FP32 moments (1 - beta and the corrections) round by some 1e-5
            np.testing.assert_allclose(after - before, -1e-3 * gg / (np.abs(gg) + 1e-8), rtol=1e-3, atol=1e-7)
    assert losses == hist.cpu().tolist()
    assert torch.equal(emu, both)
