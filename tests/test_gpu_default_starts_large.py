"""The plain method's starts on histograms far above the sizes of a batch: the
search for the peak's width on whole counts against the one on floating-point
counts, which walks every window position."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def hists(nb):
    rng = np.random.default_rng(nb)
    i = (np.arange(nb) + 0.5) / nb
    out = []
    for place in (0.003, 0.02, 0.5, 0.97):
        for width in (0.0003, 0.003, 0.03, 0.3):
            out.append(rng.poisson(40.0 * np.exp(-2.0 * i) + 30.0 * np.exp(-0.5 * ((i - place) / width) ** 2)))
    out.append(np.full(nb, 7))
    c = np.full(nb, 3)
    c[nb // 4] = c[(3 * nb) // 4] = 50 * (nb // 256)
    out.append(c)
    out.append(rng.integers(0, 2 ** 32, nb))
    return out


@pytest.mark.parametrize("nb", [3, 255, 511, 512, 1025, 8192, 65_536, 300_007, 1_200_000])
def test_whole_and_floating_counts_agree(hf, nb):
    """Sums of whole counts are exact in any order, so the decisions and the
    starts are the same bits."""
    import torch
    h = hists(nb)
    off = torch.arange(0, len(h) * nb + 1, nb).cuda()
    rg = torch.tensor([[0.0, 1.0]], dtype=torch.float64).repeat(len(h), 1).cuda()
    c = np.concatenate(h)
    m = hf.Model(hf.GAUSS_EXP, 1, -1)
    u = hf.default_starts(torch.from_numpy(c.astype(np.uint32).view(np.int32)).cuda(), off, rg, m)
    f = hf.default_starts(torch.from_numpy(c.astype(np.float64)).cuda(), off, rg, m)
    np.testing.assert_array_equal(u.cpu().numpy(), f.cpu().numpy())


def test_time_grows_with_the_size(hf):
    """A histogram without a peak is searched from end to end.  Eight times the
    bins take eight times as long, and less where the fixed part of the small
    one shows; 13 leaves room for clocks and caches.  Window sums rebuilt for
    every 64 positions take 35 times as long."""
    import torch
    m = hf.Model(hf.GAUSS_EXP, 1, -1)
    rg = torch.tensor([[0.0, 1.0]], dtype=torch.float64).cuda()

    def best(nb):
        c = torch.full((nb,), 7, dtype=torch.int32, device="cuda")
        off = torch.tensor([0, nb]).cuda()
        times = []
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            hf.default_starts(c, off, rg, m)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times)

    small, large = best(1 << 17), best(1 << 20)
    assert large <= 13.0 * small, (small, large)
