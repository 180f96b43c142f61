"""Bin averages over bins of any widths, at the sizes where the steps of 64
bins and their split over the waves change, and the shared edge values of
neighbouring lanes far out in a peak's tail."""
import numpy as np
import pytest

import datagen
from test_gpu_edges import CASES, check, counts_for, edges_for, gpu, orc_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [2, 63, 64, 65, 127, 128, 129, 255, 257, 16384, 16385, 65537, 131_200])
def test_average_at_step_boundaries(hf, orc, nb):
    """Against the oracle at the library's tolerance (1e-10 of the condition
    scales), grad_w to FP32 rounding of the oracle's terms."""
    spec, th, r = CASES[1]
    e = edges_for(r[0], r[1], nb, seed=nb)
    at = np.array(th) * (1 + 0.02 * np.random.default_rng(nb).standard_normal(len(th)))
    counts = counts_for(orc, spec, e, th, 1, seed=nb + 7)
    w = np.random.default_rng(nb).uniform(0.5, 1.5, nb).astype(np.float32)
    ref = orc.nll_grad_edges(orc_model(orc, spec, 1), 2, counts, e, at, weights=w, want_ell=True)
    nll, grad, gw, st, ev = gpu(hf, spec, counts, e, at, 2, avg=1, weights=w, want_grad_w=True)
    check(ref, nll, grad, nb)
    assert st == 0 and ev == nll
    scale = np.abs(ref.ell) + np.abs(counts) + 1.0
    assert np.all(np.abs(gw - ref.ell) <= 2.0 ** -23 * np.abs(ref.ell) + 1e-9 * scale)


def test_average_in_the_tails(hf, orc):
    """Edges from 0 to 40 widths on both sides of a peak: every range of the
    erf (below 1, up to 6, beyond), with edges on its limits.  (Bins 1e-12 wide
    there are no test: the oracle's own erf differences are rounding noise in
    them, 3e-8 of the scale away from this kernel and, by the same amount,
    from one that calls the library's erf.)"""
    spec = datagen.model_spec(1, 1, 0, 0.0, 1.0)
    th = [1e6, 0.0, 1.0, 3.0]
    z = np.concatenate([-np.geomspace(40.0, 1e-3, 700), np.geomspace(1e-3, 40.0, 700)])
    lim = np.sqrt(2.0) * np.array([1.0, 6.0])
    e = np.unique(np.concatenate([z, lim, -lim]))
    counts = counts_for(orc, spec, e, th, 1, seed=3)
    at = np.array([1.02e6, 0.01, 1.01, 2.9])
    ref = orc.nll_grad_edges(orc_model(orc, spec, 1), 2, counts, e, at)
    nll, grad, _, st, _ = gpu(hf, spec, counts, e, at, 2, avg=1)
    check(ref, nll, grad, "tails")
    assert st == 0


@pytest.mark.parametrize("half", [1e-6, 2.0e-4, 2.2e-4, 1.5e-3, 1.7e-3, 0.031, 0.032, 0.2])
def test_average_series(hf, orc, half):
    """Bins of half-widths around the limits of each series (in units of the
    narrowest width), and steps that mix them with wide ones."""
    spec, _, _ = CASES[1]
    th = [700.0, 4.8, 0.4, 400.0, 5.2, 0.6, 100.0, -20.0, 10.0, 5.0]
    rng = np.random.default_rng(int(half * 1e7))
    n = 1000
    h = 2.0 * half * 0.4 * rng.uniform(0.9, 1.0, n)
    if half == 1.5e-3:
        h[[70, 200, 201, 640]] = [0.05, 0.5, 1e-5, 0.2]
    e = 4.0 + np.concatenate([[0.0], np.cumsum(h)])
    e = e[e < 9.9]
    counts = counts_for(orc, spec, e, th, 1, seed=5)
    ref = orc.nll_grad_edges(orc_model(orc, spec, 1), 2, counts, e, th, want_ell=True)
    nll, grad, gw, st, ev = gpu(hf, spec, counts, e, th, 2, avg=1, want_grad_w=True)
    # the oracle's erf differences lose about 2.3e-16 / half per bin
    tol = 1e-10 + 4.0 * 2.3e-16 / half
    assert st == ref.status == 0 and ev == nll
    assert abs(nll - ref.nll) <= tol * ref.scales[0]
    assert np.all(np.abs(grad - ref.grad) <= tol * ref.scales[1:])


def test_average_degenerate_bins(hf):
    """An empty bin is no number, with or without narrow bins beside it."""
    spec, th, _ = CASES[1]
    for n in (3, 64, 200):
        e = np.linspace(2.0, 2.001, n + 1)
        e[n // 2 + 1] = e[n // 2]
        nll, grad, _, st, _ = gpu(hf, spec, np.ones(n, dtype=np.uint32), e, th, 2, avg=1)
        assert st == 0 and np.isnan(nll) and np.isnan(grad).any()
