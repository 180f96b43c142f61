"""One record of the library's contexts: the native calls use what the Python
code's dictionaries hold at the time of the call."""
import ctypes

import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu


def batch(hf):
    import torch
    spec = datagen.model_spec(2, 1, -1, 0.0, 1.0)
    lam = datagen.intensity_1d(spec, np.array([500.0, 0.4, 0.1, 4.0, -0.7]), 300, 0.0, 1.0)
    c = torch.from_numpy(datagen.poisson_counts(lam, np.random.default_rng(1)).view(np.int32)).cuda()
    args = (c, torch.tensor([0, 300]).cuda(), torch.tensor([[0.0, 1.0]], dtype=torch.float64).cuda(),
            hf.Model.from_spec(spec), torch.tensor([[480.0, 0.41, 0.1, 4.0, -0.6]], dtype=torch.float64).cuda())
    return lambda: hf.fit_batch(*args)


def test_forgotten_contexts_are_made_anew(hf):
    fit = batch(hf)
    want = fit()
    ctx, pool = dict(hf._ctx), dict(hf._pool)
    try:
        hf._ctx.clear()
        hf._pool.clear()
        got = fit()
        assert len(hf._ctx) == 1 and all(len(p) == hf.POOL_SIZE for p in hf._pool.values())
        assert not {h.value for h in hf._ctx.values()} & {h.value for h in ctx.values()}
    finally:
        for d, was in ((hf._ctx, ctx), (hf._pool, pool)):
            d.clear()
            d.update(was)
    assert got.theta.equal(want.theta)


def test_calls_use_the_context_that_is_set(hf):
    """A cache of counts that no kernel can hold is refused by fit_batch: set
    on the context of the current stream alone, it shows which one a call
    takes."""
    import torch
    fit = batch(hf)
    fit()
    L = hf.load()
    dev = torch.cuda.current_device()
    key = (dev, torch.cuda.current_stream().cuda_stream)
    was, other = hf._ctx[key], ctypes.c_void_p()
    assert L.hf_ctx_create(ctypes.byref(other), dev) == 0
    try:
        assert L.hf_fit_set_tuning(other, 2, 1 << 20, 256) == 0
        hf._ctx[key] = other
        with pytest.raises(hf.HistfitError, match="LDS cache"):
            fit()
    finally:
        hf._ctx[key] = was
        L.hf_ctx_destroy(other)
    fit()
