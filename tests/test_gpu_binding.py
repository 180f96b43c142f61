"""The native marshalling of the per-call entry points against the Python code
after it (a module that takes no call): same results, same outputs returned, the same
calls refused, converted arguments, several streams, capture and dispatch
modes."""
import dataclasses

import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu

SPEC = datagen.model_spec(1, 1, 1, 0.0, 1.0)
THETA = [300.0, 4.8, 0.7, 20.0, -1.2]
RANGE = (0.0, 10.0)


def setup(hf, n=5000):
    import torch
    c = datagen.random_1d_case(SPEC, n, *RANGE, THETA, seed=1)
    w = np.random.default_rng(2).uniform(0.5, 1.5, n).astype(np.float32)
    h = hf.make_hist(c["counts"], RANGE, weights=w)
    th = torch.tensor(THETA, dtype=torch.float64, device="cuda")
    ev = torch.rand(3000, dtype=torch.float64, device="cuda") * 10.0
    return h, hf.Model.from_spec(SPEC), th, ev


def calls(hf, h, m, th, ev):
    import torch
    f64 = dict(dtype=torch.float64, device="cuda")
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    B = 3
    off = torch.tensor([0, 1000, 2500, 5000], device="cuda")
    rg = torch.tensor([[0.0, 10.0]] * B, **f64)
    th0 = th.repeat(B, 1)
    seed = torch.tensor([0.5], **f64)
    F = hf.nll_fisher(h, m, th)
    return {
        "eval": lambda **k: hf.nll_eval(h, m, k.get("th", th), status=st),
        "eval_out": lambda **k: hf.nll_eval(h, m, k.get("th", th), out=torch.zeros(2, **f64)),
        "grad": lambda **k: hf.nll_grad(h, m, k.get("th", th), status=st),
        "grad_all": lambda **k: hf.nll_grad(h, m, k.get("th", th), hf.PEARSON, seed=seed,
                                            want_grad_w=True, free_mask=0b10110),
        "fisher": lambda **k: hf.nll_fisher(h, m, k.get("th", th)),
        "cov": lambda **k: hf.fisher_covariance(F, free_mask=0b1111),
        "cov_batch": lambda **k: hf.fisher_covariance(torch.stack([F, 2 * F])),
        "unbinned": lambda **k: hf.nll_unbinned(ev, 0.0, 10, m, k.get("th", th)),
        "unbinned_w": lambda **k: hf.nll_unbinned(ev, 0.0, 10.0, m, k.get("th", th),
                                                  weights=h.weights[:3000]),
        "fit": lambda **k: hf.fit_batch(h.counts, off, rg, m, th0, max_iter=50),
    }


def flat(r):
    import torch
    if isinstance(r, torch.Tensor):
        return [r]
    if dataclasses.is_dataclass(r):
        r = [getattr(r, f.name) for f in dataclasses.fields(r)]
    return [v for v in r if v is not None]


def same(a, b):
    import torch
    a, b = flat(a), flat(b)
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert x.shape == y.shape and x.dtype == y.dtype and x.device == y.device
        assert not x.requires_grad and torch.equal(x, y)


class TakesNothing:
    def __getattr__(self, name):
        return lambda *args: None


def test_same_results_as_the_python_code(hf, monkeypatch):
    import torch
    parts = setup(hf)
    fns = calls(hf, *parts)
    th = parts[2]
    other = [th.tolist(), th.cpu(), torch.stack([th, th], 1)[:, 0], th.clone().requires_grad_()]
    fast = {k: [f()] + [f(th=o) for o in other] for k, f in fns.items()}
    native = hf._fast
    assert native is not None
    args = (parts[0], parts[1], th, hf.POISSON, hf.FP64, None, None)
    assert native.nll_eval(*args) is not None  # the native code takes this call
    assert native.nll_eval(*args[:2], th.cpu(), *args[3:]) is None  # and leaves this one
    assert native.nll_eval(*args[:6], torch.zeros(1, device="cuda")) is None
    monkeypatch.setattr(hf, "_fast", TakesNothing())
    for k, f in fns.items():
        for r in fast[k]:
            same(r, f())


def test_given_outputs_and_refused_calls(hf):
    import torch
    h, m, th, ev = setup(hf)
    f64 = dict(dtype=torch.float64, device="cuda")
    nll, grad = torch.zeros(1, **f64), torch.zeros(5, **f64)
    r = hf.nll_grad(h, m, th, nll_out=nll, grad_out=grad)
    assert r[0] is nll and r[1] is grad and r[2] is None and nll.item() != 0.0
    for bad in (dict(out=torch.zeros(1, device="cuda")), dict(out=torch.zeros(1, dtype=torch.float64)),
                dict(status=torch.zeros(1, device="cuda"))):
        with pytest.raises(ValueError):
            hf.nll_eval(h, m, th, **bad)
    with pytest.raises(ValueError):
        hf.nll_eval(h, m, th[:4])
    with pytest.raises(ValueError):
        hf.nll_grad(h, m, th, grad_out=torch.zeros(4, **f64))
    with pytest.raises(ValueError):
        hf.nll_grad(h, m, th, seed=torch.zeros(2, **f64))
    with pytest.raises(ValueError):
        hf.nll_eval(dataclasses.replace(h, counts=h.counts[::2]), m, th)
    with pytest.raises(ValueError):
        hf.nll_eval(dataclasses.replace(h, weights=h.weights[:-1]), m, th)
    with pytest.raises(ValueError):
        hf.nll_eval(dataclasses.replace(h, counts=h.counts.cpu()), m, th)
    with pytest.raises(hf.HistfitError):
        hf.nll_eval(h, m, th, objective=7)
    with pytest.raises(hf.HistfitError):
        hf.fisher_covariance(hf.nll_fisher(h, m, th), free_mask=1 << 20)
    with pytest.raises(ValueError):
        hf.nll_unbinned(ev.float(), 0.0, 10.0, m, th)
    with pytest.raises(hf.HistfitError):
        hf.nll_unbinned(ev, 10.0, 0.0, m, th)


def test_streams_and_capture(hf):
    import torch
    h, m, th, ev = setup(hf)
    want = [v.clone() for v in flat(hf.nll_grad(h, m, th))]
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    for s in streams:
        with torch.cuda.stream(s):
            for _ in range(2):
                got = hf.nll_grad(h, m, th)
        s.synchronize()
        same(got, want)
    # captures on streams never seen before each take a spare context, and
    # native calls in between leave the spares to be made up
    for _ in range(6):
        s = torch.cuda.Stream()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            got = hf.nll_grad(h, m, th)
        for _ in range(3):
            for v in flat(got):
                v.zero_()
            g.replay()
            same(hf.nll_grad(h, m, th), want)
            torch.cuda.synchronize()
            same(got, want)


def test_dispatch_modes_see_the_allocations(hf):
    from torch.utils._python_dispatch import TorchDispatchMode

    class Seen(TorchDispatchMode):
        names = []

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.names.append(str(func))
            return func(*args, **(kwargs or {}))

    h, m, th, ev = setup(hf)
    want = hf.nll_grad(h, m, th)
    with Seen() as mode:
        got = hf.nll_grad(h, m, th)
    assert any("empty" in n for n in mode.names)
    same(got, want)
