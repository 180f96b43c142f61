"""FP64 fits of Gaussians a few bins wide, which the recurrences over runs of
bins do not cover: groups of four bins with an exponential each, at the sizes
where their split over a group of threads changes."""
import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu

SIZES = [3, 4, 7, 253, 256, 1023, 1024, 1027, 2047, 2049, 4099, 8195]


@pytest.mark.parametrize("obj", [2, 0, 1])
@pytest.mark.parametrize("gauss", [1, 3])
def test_one_step_of_narrow_peaks(hf, orc, gauss, obj):
    """One steepest-descent step, which gives away the gradient, against the
    oracle's to 1e-10 of the gradient's condition scale times alpha sigma^2
    and the rounding of theta, from every source of counts (equal bit for bit)
    and by workgroups of 256, 512 and single waves.  One peak of 1.3 bins is
    enough to keep the recurrences off."""
    import torch
    rng = np.random.default_rng(9)
    spec = datagen.model_spec(1, gauss, 1, 0.0, 1.0)
    m, om = hf.Model.from_spec(spec), orc.Model(1, gauss, 1, 0.0, 1.0)
    th0, counts = [], []
    for n in SIZES:
        th = [900.0, 0.47, 1.3 / n]
        for g in range(1, gauss):
            th += [300.0, 0.15 + 0.35 * g, 0.04]
        th += [60.0, 20.0]
        counts.append(datagen.poisson_counts(datagen.intensity_1d(spec, np.array(th), n, 0.0, 1.0), rng))
        th0.append(datagen.perturb(th, 0.01, rng))
    th0 = np.array(th0)
    cat = np.concatenate(counts)
    off = torch.as_tensor(np.concatenate([[0], np.cumsum(SIZES)]).astype(np.int64))
    rg = torch.as_tensor(np.tile([0.0, 1.0], (len(SIZES), 1)))

    def run(c):
        r = hf.fit_batch(c, off, rg, m, torch.as_tensor(th0), objective=obj, max_iter=1, fixed_iters=True,
                         hessian_init=hf.IDENTITY)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (r.theta, r.nll, r.status, r.iters, r.nevals)]

    u32 = torch.from_numpy(cat.view(np.int32)).cuda()
    got = []
    try:
        hf.fit_set_wave_bins(0)
        for blk in (256, 512):
            hf.fit_set_tuning(2, 0, blk)
            base = run(u32)
            for c in (torch.from_numpy(cat.astype(np.float32)).cuda(),
                      torch.from_numpy(cat.astype(np.float64)).cuda()):
                for x, y in zip(base, run(c)):
                    np.testing.assert_array_equal(x, y)
            hf.fit_set_tuning(2, 9000, blk)
            for x, y in zip(base, run(u32)):
                np.testing.assert_array_equal(x, y)
            got.append(base)
        hf.fit_set_tuning(2, 0, 256)
        hf.fit_set_wave_bins(2048)
        got.append(run(u32))
    finally:
        hf.fit_set_wave_bins(0)
        hf.fit_set_tuning(2, 0, 256)
    for b, n in enumerate(SIZES):
        ref = orc.fit(om, obj, counts[b], th0[b], (0.0, 1.0), max_iter=1, fixed_iters=True, hessian_init=0)
        at0 = orc.nll_grad(om, obj, counts[b], th0[b], (0.0, 1.0))
        sig = np.array([max(abs(v), 1.0) for v in th0[b]])
        for g in range(gauss):
            sig[3 * g + 1], sig[3 * g + 2] = 0.01, abs(th0[b][3 * g + 2])
        for theta, nll, st, it, ne in got:
            assert (st[b], it[b], ne[b]) == (ref.status, ref.iters, ref.nevals), n
            alpha = 0.5 ** (ne[b] - 2)
            tol = alpha * sig ** 2 * 1e-10 * at0.scales[1:] + 4e-16 * (np.abs(th0[b]) + np.abs(theta[b]))
            assert np.all(np.abs(theta[b] - ref.theta) <= tol), (n, theta[b], ref.theta, tol)
            end = orc.nll_grad(om, obj, counts[b], theta[b], (0.0, 1.0))
            assert abs(nll[b] - end.nll) <= 1e-10 * end.scales[0], n
