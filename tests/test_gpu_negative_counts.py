"""Floating-point counts below zero (background-subtracted histograms): the
Poisson objective then has no minimum of its own meaning, but it differs from
sum(mu - n ln mu) by a constant at every theta, as it does for other counts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["FP64", "FP32_BIN"])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_objective_differences_with_negative_counts(hf, dtype, prec):
    """mu a line, so that no exponential enters; n/mu passes -0.75 and the
    powers of two between the points.  A bin's constant is at most 2048 ln 2
    |n|, and the sum is exact to a few roundings of its size (1e-14), which
    1e-13 bounds; a constant that changed with theta would be off by 4096 ln 2
    |n| in a bin."""
    import torch
    n_bins = 1003
    rng = np.random.default_rng(4)
    n = np.round(rng.uniform(-150.0, 20.0, n_bins))
    x = (np.arange(n_bins) + 0.5) / n_bins
    h = hf.make_hist(n.astype(dtype), (0.0, 1.0))
    m = hf.Model(hf.GAUSS_POLY, 0, 1)
    points = [(30.0, 5.0), (70.0, 5.0), (100.0, 40.0), (220.0, -90.0), (2000.0, 100.0)]
    got = [hf.nll_eval(h, m, torch.tensor(p, dtype=torch.float64), precision=getattr(hf, prec)).item()
           for p in points]
    mu = [p[0] + p[1] * x for p in points]
    scale = np.sum(2048.0 * np.log(2.0) * np.abs(n) + np.abs(n) * 10.0 + 2100.0)
    for k in range(1, len(points)):
        want = np.sum(mu[k] - mu[0]) - np.sum(n * np.log(mu[k] / mu[0]))
        assert abs((got[k] - got[0]) - want) <= 1e-13 * scale, (points[k], got[k] - got[0], want)
