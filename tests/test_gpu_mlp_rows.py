"""The training step where its row and K splits change: the smallest batch, a
batch whose K steps do not divide by the waves that share them, and FP32
inputs that are aligned to their values only."""
import numpy as np
import pytest

from test_gpu_mlp import U32, bf16_values

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [64, 192, 1088])
def test_gradients_from_stored_rows(hf, batch):
    """Every weight and bias gradient against FP64 sums over the step's own
    stored activations and adjoints (exact BF16 products, FP32 sums: the
    recursive-summation bound of (B + 8) 2^-24 sum |dz||a|), the loss against
    FP64 to the rounding of its FP32 result, and a step on unaligned copies
    of the inputs equal bit for bit."""
    import torch
    from oracle import mlp as om
    rng = np.random.default_rng(31 + batch)
    n = hf.mlp_nparams()
    p0 = torch.as_tensor(om.init_params(9), dtype=torch.float32).cuda()
    x0 = torch.as_tensor(rng.standard_normal((batch, om.IN)), dtype=torch.float32).cuda()
    t0 = torch.as_tensor(rng.standard_normal((batch, om.OUT)), dtype=torch.float32).cuda()

    def shifted(t, by):
        buf = torch.zeros(t.numel() + 4, dtype=t.dtype, device=t.device)
        v = buf[by:by + t.numel()].view(t.shape)
        v.copy_(t)
        return v

    runs = []
    for by in (0, 1):
        p, x, t = shifted(p0, by), shifted(x0, by), shifted(t0, by)
        m, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
        g, loss = torch.zeros(n, device="cuda"), torch.zeros(1, device="cuda")
        ws = hf.mlp_workspace(batch, "cuda")
        hf.mlp_train_step(p, m, v, 1, 1e-3, 1e-4, x, t, g, loss, ws)
        torch.cuda.synchronize()
        runs.append((p, m, v, g, loss, ws))
    for a, b in zip(runs[0][:5], runs[1][:5]):
        assert torch.equal(a, b)
    _, _, _, g, loss, ws = runs[0]
    views = hf.mlp_workspace_views(ws, batch)
    g = g.cpu().numpy().astype(np.float64)
    at = 0
    for l, (out, inn) in enumerate([(512, 256), (512, 512), (512, 512), (32, 512)]):
        a, dz = bf16_values(views["a%d" % l]), bf16_values(views["dz%d" % (l + 1)])
        bound = (batch + 8) * U32
        dw = g[at:at + out * inn].reshape(out, inn)
        assert np.all(np.abs(dw - dz.T @ a) <= bound * (np.abs(dz).T @ np.abs(a)) + 1e-30), l
        db = g[at + out * inn:at + out * inn + out]
        assert np.all(np.abs(db - dz.sum(0)) <= bound * np.abs(dz).sum(0) + 1e-30), l
        at += out * inn + out
    y = views["y"].cpu().numpy().astype(np.float64)[:, :5]
    # y - t is taken in FP32: one rounding of each difference
    d = y - t0.cpu().numpy().astype(np.float64)
    ref = np.mean(d * d)
    assert abs(loss.item() - ref) <= 4 * U32 * ref
