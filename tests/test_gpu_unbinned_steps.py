"""The unbinned likelihood where its event loop branches: whole steps of
events in the range, ragged last steps, steps with a few events outside, and
one pair per lane; intensities far from 1 (the product of the intensities
must neither overflow nor underflow), Gaussians of a width far below their
distance, and domain errors among events that are all in the range.  Against
the FP64 oracle, |d| <= 1e-10 of its condition scales; the domain errors'
outputs are exact."""
import math

import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu

TOL = 1e-10
LO, HI = 0.0, 10.0

MODELS = [
    (datagen.model_spec(1, 0, 2, 0.0, 5.0), [40.0, 5.0, 3.0]),
    (datagen.model_spec(1, 1, 0, 0.0, 5.0), [300.0, 4.0, 0.01, 20.0]),
    (datagen.model_spec(1, 2, 3, 5.0, 5.0),
     [200.0, 2.5, 0.5, 150.0, 6.5, 0.02, 30.0, -4.0, 2.0, 0.5]),
    (datagen.model_spec(1, 3, 0, 0.0, 1.0), [80.0, 2.0, 0.5, 120.0, 5.0, 0.8, 60.0, 7.5, 0.4, 15.0]),
    (datagen.model_spec(1, 4, 1, 5.0, 5.0),
     [80.0, 2.0, 0.5, 120.0, 5.0, 0.8, 60.0, 7.5, 0.4, 50.0, 8.8, 0.3, 15.0, 1.0]),
    (datagen.model_spec(2, 1, -1, 5.0, 5.0), [300.0, 4.0, 0.8, math.log(20.0), 1.2]),
]


def run(hf, spec, x, th, w=None):
    import torch
    st = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    xt = torch.tensor(x, dtype=torch.float64, device="cuda")
    wt = None if w is None else torch.tensor(w, device="cuda")
    nll, g = hf.nll_unbinned(xt, LO, HI, hf.Model.from_spec(spec), th, weights=wt, status=st)
    only, _ = hf.nll_unbinned(xt, LO, HI, hf.Model.from_spec(spec), th, weights=wt,
                              want_grad=False)
    return nll.item(), g.cpu().numpy(), int(st.item()), only.item()


def check(hf, orc, spec, x, th, w=None):
    m = orc.Model(spec["kind"], spec["n_gauss"], spec["poly_degree"], spec["t_shift"],
                  spec["t_scale"])
    ref = orc.unbinned(m, x, LO, HI, th, weights=None if w is None else w.astype(np.float64))
    nll, g, st, only = run(hf, spec, x, th, w)
    assert st == ref.status == 0
    assert abs(nll - ref.nll) <= TOL * ref.scales[0], (nll, ref.nll)
    assert abs(only - ref.nll) <= TOL * ref.scales[0], (only, ref.nll)
    assert np.all(np.abs(g - ref.grad) <= TOL * ref.scales[1:])


@pytest.mark.parametrize("case", range(len(MODELS)))
@pytest.mark.parametrize("weighted", [False, True])
def test_steps(hf, orc, case, weighted):
    spec, th = MODELS[case]
    for n in (256, 1023, 1024, 1025, 2048, 100_000, 786_432, 786_437):
        rng = np.random.default_rng(n + case)
        x = rng.uniform(LO, HI, n)
        w = rng.uniform(0.5, 1.5, n).astype(np.float32) if weighted else None
        check(hf, orc, spec, x, th, w)  # every step in the range
        x[[0, n // 2, n - 1]] = [LO, HI, math.nextafter(HI, 0.0)]
        x[n // 3] = math.nextafter(HI, 20.0)  # a single event outside
        check(hf, orc, spec, x, th, w)


@pytest.mark.parametrize("scale", [1e-280, 1e-30, 1e30, 1e280])
def test_intensities_far_from_one(hf, orc, scale):
    spec, th = MODELS[0]
    x = np.random.default_rng(3).uniform(LO, HI, 200_001)
    check(hf, orc, spec, x, list(np.array(th) * scale))


def test_domain_errors_inside_the_range(hf):
    spec = datagen.model_spec(1, 1, -1, 0.0, 1.0)
    x = np.random.default_rng(4).normal(5.0, 0.1, 4096)
    assert run(hf, spec, x, [500.0, 5.0, 0.1])[2] == 0
    x[1000] = 0.1  # 2^(-u^2) is 0 there, 49 widths from the mean
    for w in (None, np.ones(4096, dtype=np.float32)):
        nll, g, st, only = run(hf, spec, x, [500.0, 5.0, 0.1], w)
        assert nll == only == math.inf and np.all(np.isnan(g)) and st != 0
        nll, g, st, only = run(hf, spec, x[1024:], [-500.0, 5.0, 0.1], w if w is None else w[1024:])
        assert nll == only == math.inf and np.all(np.isnan(g)) and st != 0
