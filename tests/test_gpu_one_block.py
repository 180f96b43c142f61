"""The calls that one block covers and writes itself, around the sizes where a
second block (and the finishing kernel) begins: objective, expected Hessian
and unbinned likelihood against the FP64 oracle (|d| <= 1e-10 of its
condition scale), with seed, free mask, weights and every status."""
import math

import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu

TOL = 1e-10
SPEC = datagen.model_spec(1, 2, 3, 5.0, 5.0)
THETA = [700.0, 3.0, 0.4, 400.0, 6.2, 0.6, 100.0, -20.0, 10.0, 5.0]
RANGE = (0.0, 10.0)


def orc_model(orc):
    return orc.Model(SPEC["kind"], SPEC["n_gauss"], SPEC["poly_degree"], SPEC["t_shift"],
                     SPEC["t_scale"])


@pytest.mark.parametrize("nb", [1, 63, 4096, 4097, 8192, 8193])
@pytest.mark.parametrize("obj", [0, 1, 2])
def test_objective(hf, orc, nb, obj):
    import torch
    c = datagen.random_1d_case(SPEC, nb, *RANGE, THETA, seed=nb)
    w = np.random.default_rng(nb).uniform(0.5, 1.5, nb).astype(np.float32)
    h = hf.make_hist(c["counts"], RANGE, weights=w)
    m = hf.Model.from_spec(SPEC)
    st = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    mask = 0b1010010110
    nll, g, _ = hf.nll_grad(h, m, c["theta_eval"], objective=obj, seed=0.75, free_mask=mask,
                            status=st)
    ev = hf.nll_eval(h, m, c["theta_eval"], objective=obj)
    ref = orc.nll_grad(orc_model(orc), obj, c["counts"], c["theta_eval"], RANGE,
                       weights=w.astype(np.float64))
    free = np.array([(mask >> k) & 1 for k in range(10)])
    assert int(st.item()) == ref.status
    assert abs(nll.item() - ref.nll) <= TOL * ref.scales[0] and ev.item() == nll.item()
    err = np.abs(g.cpu().numpy() - 0.75 * free * ref.grad)
    assert np.all(err <= TOL * ref.scales[1:] * free)
    bad = np.array(c["theta_eval"])
    bad[1] = math.nan
    nll, g, _ = hf.nll_grad(h, m, bad, objective=obj, status=st)
    assert math.isnan(nll.item()) and torch.isnan(g).all() and int(st.item()) != 0
    if obj == 2:  # a Poisson mean below zero where counts are
        bad = np.array(c["theta_eval"])
        bad[[0, 3]] = -5e4
        h1 = hf.make_hist(np.full(nb, 3, dtype=np.uint32), RANGE)
        bad[6:] = [-1.0, 0.0, 0.0, 0.0]
        nll, g, _ = hf.nll_grad(h1, m, bad, objective=obj, status=st)
        assert nll.item() == math.inf and torch.isnan(g).all() and int(st.item()) != 0


@pytest.mark.parametrize("nb", [1, 64, 2048, 2049, 4096, 4097])
@pytest.mark.parametrize("obj", [0, 1, 2])
def test_expected_hessian(hf, orc, nb, obj):
    import torch
    c = datagen.random_1d_case(SPEC, nb, *RANGE, THETA, seed=nb + 1)
    h = hf.make_hist(c["counts"], RANGE)
    st = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    F = hf.nll_fisher(h, hf.Model.from_spec(SPEC), c["theta_eval"], objective=obj, status=st)
    F = F.cpu().numpy()
    ref = orc.fisher(orc_model(orc), obj, c["counts"], c["theta_eval"], RANGE)
    ref = ref[0] if isinstance(ref, tuple) else ref
    d = np.sqrt(np.outer(np.diag(ref), np.diag(ref)))
    assert np.all(np.abs(F - ref) <= TOL * d) and np.array_equal(F, F.T)
    assert int(st.item()) == 0


@pytest.mark.parametrize("n", [0, 1, 2047, 2048, 2049, 2050])
@pytest.mark.parametrize("weighted", [False, True])
def test_unbinned(hf, orc, n, weighted):
    import torch
    x = datagen.unbinned_events(SPEC, THETA, *RANGE, n, seed=n) if n else np.zeros(0)
    w = np.random.default_rng(n).uniform(0.5, 1.5, n).astype(np.float32) if weighted else None
    st = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    xt = torch.tensor(x, dtype=torch.float64, device="cuda")
    wt = torch.tensor(w, device="cuda") if weighted else None
    nll, g = hf.nll_unbinned(xt, *RANGE, hf.Model.from_spec(SPEC), THETA, weights=wt, status=st)
    ref = orc.unbinned(orc_model(orc), x, *RANGE, THETA,
                       weights=None if w is None else w.astype(np.float64))
    assert int(st.item()) == 0
    assert abs(nll.item() - ref.nll) <= TOL * ref.scales[0]
    assert np.all(np.abs(g.cpu().numpy() - ref.grad) <= TOL * ref.scales[1:])
