"""Rebinning of histograms whose coarse bins hold up to six counts, where a
thread takes a coarse bin's run alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["u32", "f32", "f64"])
def test_rebin_short_runs(hf, dtype):
    """One bin either side of every change of path, every run length; counts
    that are not whole (floating-point types), zero, and at the end of the
    buffer.  A coarse bin's mean is off by a rounding or two of its sum, so the
    FP32 result by its own rounding."""
    import torch

    import oracle.mlp as om
    sizes = [1, 2, 255, 256, 257, 511, 512, 513, 767, 768, 769, 1023, 1024, 1025, 1279, 1281, 1535, 1536,
             1537, 2047, 2048]
    rng = np.random.default_rng(12)
    counts = np.concatenate([rng.integers(0, 1000, n) * (rng.random(n) < 0.7) for n in sizes])
    if dtype != "u32":
        counts = (counts + rng.random(counts.size)).astype({"f32": np.float32, "f64": np.float64}[dtype])
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    ref = om.rebin_lognorm(counts, offsets, 1.5, 2.0)
    on = torch.from_numpy(counts.astype(np.int32) if dtype == "u32" else counts).cuda()
    x = hf.rebin_lognorm(on, torch.from_numpy(offsets).cuda(), 1.5, 2.0).cpu().numpy()
    np.testing.assert_allclose(x, ref, rtol=2.0 ** -23, atol=1.5 * 2.0 ** -23)
