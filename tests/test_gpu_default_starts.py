"""The plain method's starts where the search for the peak and its width
changes shape: peaks of every width at every place (the width's bounds within
one round of the search from the peak, several rounds, or the end of the range),
equal excesses (the first wins), all counts equal, counts up to 2^32 - 1, and
long windows.  The decisions are integers, so the starts equal the oracle's to
the rounding of their closed forms (1e-12)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def hists():
    rng = np.random.default_rng(21)
    out = []
    for nb in (4, 65, 513, 1024, 1027, 4096, 20_000, 70_001):
        i = (np.arange(nb) + 0.5) / nb
        for place in (0.02, 0.5, 0.97):
            for width in (0.003, 0.03, 0.3):
                mu = 40.0 * np.exp(-2.0 * i) + 30.0 * np.exp(-0.5 * ((i - place) / width) ** 2)
                out.append(rng.poisson(mu))
        out.append(np.full(nb, 7))
        c = np.full(nb, 3)
        c[nb // 4] = c[(3 * nb) // 4] = 50  # two equal excesses over a flat background
        out.append(c)
        out.append(rng.integers(0, 2 ** 32, nb))
    return out


@pytest.mark.parametrize("dtype", ["u32", "f64"])
def test_default_starts_searches(hf, dtype):
    import torch

    import oracle.mlp as om
    h = hists()
    off = np.concatenate([[0], np.cumsum([x.size for x in h])]).astype(np.int64)
    c = np.concatenate(h)
    rg = np.tile([0.0, 1.0], (len(h), 1))
    ref = om.default_starts(c, off, [(0.0, 1.0)] * len(h))
    ct = c.astype(np.uint32).view(np.int32) if dtype == "u32" else c.astype(np.float64)
    got = hf.default_starts(torch.from_numpy(ct).cuda(), torch.from_numpy(off).cuda(),
                            torch.from_numpy(rg).cuda(), hf.Model(hf.GAUSS_EXP, 1, -1)).cpu().numpy()
    np.testing.assert_allclose(got, np.asarray(ref), rtol=1e-12, atol=1e-12)
