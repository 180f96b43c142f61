"""Host-only check that the autotuner treats the automatic schedule of small
histograms as a setting: restored when no shape agrees, and a candidate, on a
sample of the size from which it does anything (the stand-ins of
test_autotune_host)."""
import pytest

import paper_2203_06139_amd as hf
from paper_2203_06139_amd import autotune
from test_autotune_host import _batch, _install


def _tune(B, sample):
    counts, off, rg, th0 = _batch(B=B)
    return autotune.tune_fit(counts, off, rg, hf.Model(hf.GAUSS_EXP, 1), th0, sample=sample, use_cache=False)


def test_automatic_setting_is_restored(monkeypatch):
    state = _install(monkeypatch, agreeing=set())
    state["waves"] = hf.WAVE_AUTO
    with pytest.raises(RuntimeError, match="no launch shape"):
        _tune(8, 8)
    assert state["waves"] == hf.WAVE_AUTO


@pytest.mark.parametrize("B, tried", [(7, False), (8, True), (64, True)])
def test_automatic_setting_is_a_candidate(monkeypatch, B, tried):
    """Four workgroups here, so the automatic setting is on from eight
    histograms: a batch of fewer leaves it out, a larger one is timed with it on
    eight, whatever the first stage's sample."""
    state = _install(monkeypatch, agreeing={(256, 1)})
    monkeypatch.setattr(autotune, "_workgroups", lambda counts, wg: 4)
    real, seen = autotune.fit_batch, []

    def fit_batch(counts, off, *a, **kw):
        seen.append((state["waves"], off.numel() - 1))
        return real(counts, off, *a, **kw)

    def timed(fn, reps=2):
        fn()
        return state["shape"][0] * (0.5 if state["waves"] == hf.WAVE_AUTO else 1.0)

    monkeypatch.setattr(autotune, "fit_batch", fit_batch)
    monkeypatch.setattr(autotune, "_time", timed)
    best, _ = _tune(B, 4)
    sizes = {n for waves, n in seen if waves == hf.WAVE_AUTO}
    assert sizes == ({8} if tried else set())
    assert best["wave_bins"] == state["waves"] == (hf.WAVE_AUTO if tried else 0)
