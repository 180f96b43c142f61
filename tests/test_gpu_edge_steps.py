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
