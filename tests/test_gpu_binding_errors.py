"""A call that the library refuses raises from the native code, once."""
import pytest

from test_gpu_binding import calls, setup

pytestmark = pytest.mark.gpu


def test_refused_calls_are_made_once(hf, monkeypatch):
    """The library counts a refused call as any other: the Python code after
    the native one, which would make it again, is not reached."""
    import torch
    h, m, th, ev = setup(hf)
    fns = calls(hf, h, m, th, ev)
    for f in fns.values():
        f()  # every call is taken natively

    def reached(*args, **kw):
        raise AssertionError("the call went on to the Python code")

    F = hf.nll_fisher(h, m, th)
    off = torch.tensor([0, 1000, 2500], device="cuda")
    rg = torch.tensor([[0.0, 10.0]] * 2, dtype=torch.float64, device="cuda")
    th0 = th.repeat(2, 1)
    monkeypatch.setattr(hf, "context", reached)
    monkeypatch.setattr(hf, "_check_hist_sizes", reached)
    bad = {
        "objective 7 unknown": [lambda: hf.nll_eval(h, m, th, objective=7), lambda: hf.nll_grad(h, m, th, 7),
                                lambda: hf.nll_fisher(h, m, th, 7), lambda: hf.fisher_covariance(F, 7)],
        "precision 9 unknown": [lambda: hf.nll_eval(h, m, th, precision=9)],
        "range must be finite": [lambda: hf.nll_unbinned(ev, 10.0, 0.0, m, th)],
        "fit options out of range": [lambda: hf.fit_batch(h.counts, off, rg, m, th0, max_iter=0)],
    }
    for message, fs in bad.items():
        for f in fs:
            with pytest.raises(hf.HistfitError, match="histfit error -1: .*" + message):
                f()
    for f in fns.values():
        f()
