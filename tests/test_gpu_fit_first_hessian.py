"""The precision of the fit's starting Hessian."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_weights_of_the_expected_hessian(hf):
    """A constant c fitted to counts of 2c: n/mu is 2 exactly and the gradient
    -1 per bin exactly, so the first step from the Fisher start, of size c, is
    off by the roundings of the inverse Hessian c / bins and of the step
    itself.  In units of 2^-53 of the step: the weight 1/mu 1; the sum of a
    thread's four bins 2 and of the four waves 2 (by doubling, over the lanes,
    none); sigma^2 F 2; the factor's square root and its inverse 1 each, twice
    as the inverse is squared, and the square 1; sigma g 1; H g 1; sigma u + c,
    of twice the step's size, 2: 16 in all, 1.78e-15.  A weight good to 2.3e-15
    fails for the worst c."""
    import torch
    B, nb = 1000, 1024  # a workgroup of 256 threads each
    worst = 0.0
    for seed in range(5):
        rng = np.random.default_rng(seed)
        c = rng.uniform(1.0, 2.0, B) * 2.0 ** rng.integers(0, 10, B)
        n = torch.from_numpy(np.repeat(2.0 * c, nb)).cuda()
        off = torch.arange(0, B * nb + 1, nb).cuda()
        rg = torch.tensor([[0.0, 1.0]], dtype=torch.float64).repeat(B, 1).cuda()
        r = hf.fit_batch(n, off, rg, hf.Model(hf.GAUSS_POLY, 0, 0), torch.from_numpy(c[:, None]).cuda(),
                         max_iter=1, fixed_iters=True)
        assert torch.all(r.nevals == 2)
        worst = max(worst, np.max(np.abs((r.theta.cpu().numpy()[:, 0] - 2.0 * c) / c)))
    assert worst <= 16 * 2.0 ** -53, worst
