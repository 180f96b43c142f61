"""More workgroups asked for than a CU holds: results as at the default shape,
and the longest histogram does not wait for the others."""
import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu

TH = [500.0, 0.4, 0.1, 4.0, -0.7]
SPEC = datagen.model_spec(2, 1, -1, 0.0, 1.0)


def batch(hf, sizes, seed):
    import torch
    rng = np.random.default_rng(seed)
    lam = {n: datagen.intensity_1d(SPEC, np.array(TH), int(n), 0.0, 1.0) for n in set(sizes)}
    c = torch.from_numpy(np.concatenate([datagen.poisson_counts(lam[n], rng) for n in sizes]).view(np.int32)).cuda()
    off = torch.as_tensor(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)).cuda()
    th0 = torch.as_tensor(np.array([datagen.perturb(TH, 0.02, rng) for _ in sizes])).cuda()
    rg = torch.tensor([[0.0, 1.0]], dtype=torch.float64).repeat(len(sizes), 1).cuda()
    return c, off, rg, hf.Model.from_spec(SPEC), th0


@pytest.mark.parametrize("shape", [(16, 0, 256), (16, 0, 512), (4, 16000, 256), (16, 16000, 512), (1, 0, 512)])
@pytest.mark.parametrize("B", [255, 512, 2049])
def test_results_do_not_depend_on_the_shape(hf, shape, B):
    """Within one workgroup size the same bits, twice in a row (the queue is
    re-armed, or was never used)."""
    import torch
    sizes = np.random.default_rng(B).choice([30, 300, 2000, 9000], B)
    args = batch(hf, sizes, B)
    was = hf.fit_get_tuning(), hf.fit_get_wave_bins()

    def run():
        r = hf.fit_batch(*args)
        torch.cuda.synchronize()
        return np.concatenate([r.theta.cpu().numpy(), r.nll.cpu().numpy()[:, None],
                               r.nevals.cpu().numpy()[:, None]], axis=1)

    try:
        hf.fit_set_wave_bins(0)
        hf.fit_set_tuning(2, 0, shape[2])
        want = run()
        hf.fit_set_tuning(*shape)
        got = [run(), run()]
    finally:
        hf.fit_set_tuning(*was[0])
        hf.fit_set_wave_bins(was[1])
    for g in got:
        np.testing.assert_array_equal(g, want)


def test_longest_histogram_starts_first(hf):
    """As many histograms as workgroups asked for, eight times what fits: one
    of them takes as long as all the others together.  Last in the batch it
    costs no more than first (10% for noise): the batch is sorted.  In index order
    it would start when the others are done, and take half as long again."""
    import torch
    was = hf.fit_get_tuning(), hf.fit_get_wave_bins()
    B = 16 * torch.cuda.get_device_properties(torch.cuda.current_device()).multi_processor_count
    times = []
    try:
        hf.fit_set_wave_bins(0)
        hf.fit_set_tuning(16, 0, 512)
        for place in (0, B - 1):
            sizes = np.full(B, 1500)
            sizes[place] = 250_000
            args = batch(hf, sizes, 3)
            hf.fit_batch(*args)
            best = float("inf")
            for _ in range(8):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                hf.fit_batch(*args)
                e1.record()
                torch.cuda.synchronize()
                best = min(best, e0.elapsed_time(e1))
            times.append(best)
    finally:
        hf.fit_set_tuning(*was[0])
        hf.fit_set_wave_bins(was[1])
    assert times[1] <= 1.1 * times[0], times
