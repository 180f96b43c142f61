"""The fit's FP64 sweep by runs of bins, at the sizes where its split changes:
fewer groups of four bins than threads, a full and a short last run, one to
eight groups per run, 0..3 bins after the last group."""
import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu

SIZES = [1, 3, 4, 5, 7, 64, 255, 256, 259, 1023, 1024, 1029, 2050, 4095, 5119, 5120, 5123, 7000, 10000,
         15361, 20483, 32767]
MODELS = {
    "gauss": (1, 1, -1, [300.0, 0.5, 0.2]),
    "quadratic": (1, 0, 2, [200.0, -30.0, 12.0]),
    "gauss-exp": (2, 1, -1, [500.0, 0.4, 0.1, 4.0, -0.7]),
    "2gauss-cubic": (1, 2, 3, [400.0, 0.3, 0.08, 250.0, 0.7, 0.11, 90.0, 14.0, -9.0, 5.0]),
    "narrow": (1, 1, 1, [400.0, 0.5, 0.001, 50.0, 20.0]),  # too narrow for the recurrences when bins are few
}


@pytest.mark.parametrize("obj", [2, 0, 1])
@pytest.mark.parametrize("name", list(MODELS))
def test_one_step_from_every_source_and_size(hf, orc, name, obj):
    """One steepest-descent step (identity start, one iteration) gives away
    the whole gradient: theta1 - theta0 = -alpha sigma^2 g.  Against the
    oracle's step, to 1e-10 of the gradient's condition scale times alpha
    sigma^2 (the library's FP64 tolerance) and the rounding of theta; the NLL
    at the end to 1e-10 of its scale.  Counts from memory as u32, f32 and f64
    and from the LDS cache take the same arithmetic: equal bit for bit."""
    import torch
    kind, ng, deg, th = MODELS[name]
    spec = datagen.model_spec(kind, ng, deg, 0.0, 1.0)
    rng = np.random.default_rng(5)
    counts = [datagen.poisson_counts(datagen.intensity_1d(spec, np.array(th), n, 0.0, 1.0), rng)
              for n in SIZES]
    cat = np.concatenate(counts)
    off = torch.as_tensor(np.concatenate([[0], np.cumsum(SIZES)]).astype(np.int64))
    th0 = np.array([datagen.perturb(th, 0.03, rng) for _ in SIZES])
    ranges = np.tile([0.0, 1.0], (len(SIZES), 1))
    m, om = hf.Model.from_spec(spec), orc.Model(kind, ng, deg, 0.0, 1.0)

    def run(c, **kw):
        r = hf.fit_batch(c, off, torch.as_tensor(ranges), m, torch.as_tensor(th0), objective=obj,
                         max_iter=1, fixed_iters=True, hessian_init=hf.IDENTITY, **kw)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (r.theta, r.nll, r.status, r.iters, r.nevals)]

    u32 = torch.from_numpy(cat.view(np.int32)).cuda()
    try:
        for blk in (256, 512):
            hf.fit_set_tuning(2, 0, blk)
            base = run(u32)
            for c in (torch.from_numpy(cat.astype(np.float32)).cuda(),
                      torch.from_numpy(cat.astype(np.float64)).cuda()):
                for x, y in zip(base, run(c)):
                    np.testing.assert_array_equal(x, y)
            hf.fit_set_tuning(2, hf.fit_max_cache_bins(m, obj, blk), blk)
            for x, y in zip(base, run(u32)):
                np.testing.assert_array_equal(x, y)
            hf.fit_set_tuning(2, 0, blk)
            hf.fit_set_wave_bins(2100)
            waves = run(u32)
            hf.fit_set_wave_bins(0)
            for theta, nll, st, it, ne in (base, waves):
                for b, n in enumerate(SIZES):
                    ref = orc.fit(om, obj, counts[b], th0[b], (0.0, 1.0), max_iter=1, fixed_iters=True,
                                  hessian_init=0)
                    assert (st[b], it[b], ne[b]) == (ref.status, ref.iters, ref.nevals), n
                    at0 = orc.nll_grad(om, obj, counts[b], th0[b], (0.0, 1.0))
                    sig = np.array([max(abs(v), 1.0) for v in th0[b]])
                    for g in range(ng):
                        sig[3 * g + 1], sig[3 * g + 2] = 0.01, abs(th0[b][3 * g + 2])
                    alpha = 0.5 ** (ne[b] - 2)
                    tol = alpha * sig ** 2 * 1e-10 * at0.scales[1:] + 4e-16 * (np.abs(th0[b]) + np.abs(theta[b]))
                    assert np.all(np.abs(theta[b] - ref.theta) <= tol), (n, theta[b], ref.theta, tol)
                    end = orc.nll_grad(om, obj, counts[b], theta[b], (0.0, 1.0))
                    assert abs(nll[b] - end.nll) <= 1e-10 * end.scales[0], n
    finally:
        hf.fit_set_wave_bins(0)
        hf.fit_set_tuning(2, 0, 256)


@pytest.mark.parametrize("B", [512, 513, 1024, 1500])
def test_batch_that_chooses_its_schedule(hf, B):
    """With no wave_bins set, the number of histograms decides whether the
    batch is sorted and whether small ones go one to a wave (512 workgroups:
    one each, one left over, two each, more): every fit as with wave_bins off
    (the order of a sum apart), empty histograms refused, twice in a row (the
    queue is re-armed, or was never used)."""
    import torch
    kind, ng, deg, th = MODELS["gauss-exp"]
    spec = datagen.model_spec(kind, ng, deg, 0.0, 1.0)
    rng = np.random.default_rng(B)
    sizes = rng.choice([0, 300, 300, 300, 700, 2047, 2048, 2049, 5000], B)
    sizes[-1] = 300
    lam = {n: datagen.intensity_1d(spec, np.array(th), int(n), 0.0, 1.0) for n in set(sizes) if n}
    counts = np.concatenate([datagen.poisson_counts(lam[n], rng) for n in sizes if n])
    off = torch.as_tensor(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)).cuda()
    th0 = torch.as_tensor(np.array([datagen.perturb(th, 0.02, rng) for _ in sizes])).cuda()
    rg = torch.tensor([[0.0, 1.0]], dtype=torch.float64).repeat(B, 1).cuda()
    c = torch.from_numpy(counts.view(np.int32)).cuda()
    m = hf.Model.from_spec(spec)

    def run():
        r = hf.fit_batch(c, off, rg, m, th0)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (r.theta, r.nll, r.status, r.iters, r.nevals)]

    contexts = (dict(hf._ctx), dict(hf._pool), dict(hf._wave_bins))
    try:
        for d in (hf._ctx, hf._pool, hf._wave_bins):
            d.clear()
        first, second = run(), run()
        hf.fit_set_wave_bins(0)
        off_ = run()
    finally:
        for d, was in zip((hf._ctx, hf._pool, hf._wave_bins), contexts):
            d.clear()
            d.update(was)
    for x, y in zip(first, second):
        np.testing.assert_array_equal(x, y)
    assert np.all((first[2] == hf.FIT_BADHIST) == (sizes == 0))
    ok = sizes > 0
    assert np.all(first[2][ok] == 0)
    for k in (2, 3, 4):
        np.testing.assert_array_equal(first[k], off_[k])
    # both converged to EDM < 1e-10: the parameters agree to 2 sqrt(2e-10) sigma,
    # sigma below 10% here
    np.testing.assert_allclose(first[0][ok], off_[0][ok], rtol=3e-6, atol=3e-6)
