"""Rebinning at the sizes where the number of lanes per coarse bin changes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["u32", "f32", "f64"])
def test_rebin_lane_counts(hf, dtype):
    """1..64 lanes per coarse bin: one bin either side of every power of two,
    runs of unequal length, a run longer than one step of a wave.  Sums of
    integer counts are exact, so the only error is log1p's and the rounding
    to FP32: 2^-23 relative to the value before the shift and scale."""
    import torch

    import oracle.mlp as om
    sizes = [1, 2, 255, 256, 257, 300]
    for k in range(9, 17):
        sizes += [2 ** k - 1, 2 ** k, 2 ** k + 1]
    sizes += [50_001, 70_000, 131_071]
    rng = np.random.default_rng(11)
    counts = np.concatenate([rng.integers(0, 1000, n) for n in sizes])
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    ref = om.rebin_lognorm(counts.astype(np.uint32), offsets, 1.5, 2.0)
    cast = {"u32": np.int32, "f32": np.float32, "f64": np.float64}[dtype]
    x = hf.rebin_lognorm(torch.from_numpy(counts.astype(cast)).cuda(), torch.from_numpy(offsets).cuda(),
                         1.5, 2.0).cpu().numpy()
    np.testing.assert_allclose(x, ref, rtol=2.0 ** -23, atol=1.5 * 2.0 ** -23)


@pytest.mark.parametrize("n", [2 ** 21 - 1, 2 ** 21, 2 ** 21 + 1, 5_000_011])
def test_rebin_long_histograms(hf, n):
    """Either side of the length from which positions take 64 bits; the same
    bound."""
    import torch

    import oracle.mlp as om
    counts = np.random.default_rng(n).integers(0, 1000, n + 3).astype(np.int32)
    offsets = np.array([0, 3, n + 3], dtype=np.int64)
    ref = om.rebin_lognorm(counts.astype(np.uint32), offsets, 1.5, 2.0)
    x = hf.rebin_lognorm(torch.from_numpy(counts).cuda(), torch.from_numpy(offsets).cuda(),
                         1.5, 2.0).cpu().numpy()
    np.testing.assert_allclose(x, ref, rtol=2.0 ** -23, atol=1.5 * 2.0 ** -23)
