"""The factors applied to the unbinned gradient's sums once per call, which no
sum over events averages out."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_gradient_factors_are_unbiased(hf):
    """A Gaussian far below a background of 1, so that lambda is 1 to 2^-40 and
    its reciprocal adds no error: the relative errors of dL/dm and dL/ds over
    many widths, against 64-bit mantissas.  One call's error is that of
    kGaussU/s (half a unit in the last place, entering u^2 and the exponential)
    and of the factor (another half): below 1.5e-16 rms, so that the mean over
    900 calls is within 4 x 1.5e-16 / 30 = 2e-17 of 0.  A constant rounded to 53
    bits (3.3e-17 off in the width's factor) is seen."""
    import torch
    L = np.longdouble
    pi = L("3.14159265358979323846264338327950288")
    rng = np.random.default_rng(8)
    n, calls = 2000, 900
    model = hf.Model(hf.GAUSS_POLY, 1, 0)
    got, ref, scale = [], [], []
    for _ in range(calls):
        s, m, A = rng.uniform(0.1, 0.3), rng.uniform(0.3, 0.7), 2.0 ** -40 * rng.uniform(1.0, 2.0)
        x = rng.uniform(0.02, 0.98, n)
        th = torch.tensor([A, m, s, 1.0], dtype=torch.float64, device="cuda")
        # every event inside, no boundary terms in the integral's gradient
        got.append(hf.nll_unbinned(torch.from_numpy(x).cuda(), m - 60 * s, m + 60 * s, model, th)[1])
        z = (x.astype(L) - L(m)) / L(s)
        G = L(A) * np.exp(-z * z / 2)
        w = G / (1 + G)
        ref.append([-np.sum(w * z) / L(s), np.sqrt(2 * pi) * L(A) - np.sum(w * z * z) / L(s)])
        scale.append([np.sum(w * np.abs(z)) / L(s), np.sum(w * z * z) / L(s)])
    g = torch.stack(got).cpu().numpy()[:, 1:3].astype(L)
    err = np.asarray((g - np.array(ref)) / np.array(scale), dtype=np.float64)
    assert np.all(np.sqrt(np.mean(err ** 2, axis=0)) <= 1.5e-16), np.sqrt(np.mean(err ** 2, axis=0))
    assert np.all(np.abs(err.mean(axis=0)) <= 2e-17), err.mean(axis=0)
