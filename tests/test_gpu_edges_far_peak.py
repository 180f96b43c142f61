"""Bin averages over explicit edges, of a peak so far away that nothing of it
is left in the histogram."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mean", [-1e60, -1e30, -1e9, -300.0, 300.0, 1e9, 1e30, 1e60])
@pytest.mark.parametrize("bins_per_width", [20.0, 400.0, 1e4])
def test_average_of_a_peak_far_away(hf, bins_per_width, mean):
    """Narrow bins (the Hermite series with 6, 3 and 2 terms), the peak at
    `mean` widths' distance and beyond: the value and the background's
    gradient of the model without it, bit for bit, and no gradient of its own
    parameters."""
    import torch
    n = 700
    rng = np.random.default_rng(6)
    e = np.concatenate([[0.0], np.cumsum(rng.uniform(0.9, 1.0, n))])
    s = bins_per_width
    h = hf.make_hist(rng.poisson(50.0, n).astype(np.uint32), None, edges=e)
    f64 = dict(dtype=torch.float64)
    alone = hf.nll_grad(h, hf.Model(hf.GAUSS_POLY, 0, 1, bin_average=1), torch.tensor([45.0, 0.01], **f64))
    m = hf.Model(hf.GAUSS_POLY, 1, 1, bin_average=1)
    th = torch.tensor([300.0, mean * s, s, 45.0, 0.01], **f64)
    status = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    nll, grad, _ = hf.nll_grad(h, m, th, status=status)
    assert status.item() == 0
    assert nll.item() == alone[0].item()
    assert torch.equal(grad[3:], alone[1])
    assert torch.equal(grad[:3], torch.zeros_like(grad[:3]))
