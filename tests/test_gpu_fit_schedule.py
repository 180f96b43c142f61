"""The schedule of small histograms as a setting: its automatic state can be
read, set and restored, and does what it says."""
import ctypes

import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu


def test_new_contexts_are_automatic(hf):
    """A context made through the C interface, which no other test has set."""
    import torch
    L = hf.load()
    h = ctypes.c_void_p()
    torch.cuda.init()
    assert L.hf_ctx_create(ctypes.byref(h), torch.cuda.current_device()) == 0
    try:
        assert L.hf_fit_get_wave_bins(h) == hf.WAVE_AUTO
        for wb in (0, 512, hf.WAVE_AUTO, 0):
            assert L.hf_fit_set_wave_bins(h, wb) == 0
            assert L.hf_fit_get_wave_bins(h) == wb
        assert L.hf_fit_set_wave_bins(h, -1) == -1
    finally:
        L.hf_ctx_destroy(h)


def test_setting_is_restored(hf):
    was = hf.fit_get_wave_bins()
    try:
        for wb in (hf.WAVE_AUTO, 0, 256, hf.WAVE_AUTO):
            hf.fit_set_wave_bins(wb)
            assert hf.fit_get_wave_bins() == wb
    finally:
        hf.fit_set_wave_bins(was)
    assert hf.fit_get_wave_bins() == was


@pytest.mark.parametrize("B", [1023, 1024, 1500])
def test_automatic_choice(hf, B):
    """512 workgroups: from 1024 histograms on the automatic setting gives the
    bits of wave_bins 2048, below it those of 0.  The two differ in the order
    of a fit's sums, so that in hundreds of fits some objective differs in its
    last bits."""
    import torch
    th = [500.0, 0.4, 0.1, 4.0, -0.7]
    spec = datagen.model_spec(2, 1, -1, 0.0, 1.0)
    rng = np.random.default_rng(B)
    sizes = rng.choice([300, 700, 2047, 2048, 2049, 5000], B)
    lam = {n: datagen.intensity_1d(spec, np.array(th), int(n), 0.0, 1.0) for n in set(sizes)}
    c = torch.from_numpy(np.concatenate([datagen.poisson_counts(lam[n], rng) for n in sizes]).view(np.int32)).cuda()
    off = torch.as_tensor(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)).cuda()
    th0 = torch.as_tensor(np.array([datagen.perturb(th, 0.02, rng) for _ in sizes])).cuda()
    rg = torch.tensor([[0.0, 1.0]], dtype=torch.float64).repeat(B, 1).cuda()
    m = hf.Model.from_spec(spec)
    was, shape = hf.fit_get_wave_bins(), hf.fit_get_tuning()
    got = {}
    try:
        hf.fit_set_tuning(2, 0, 256)
        for wb in (hf.WAVE_AUTO, 0, 2048):
            hf.fit_set_wave_bins(wb)
            r = hf.fit_batch(c, off, rg, m, th0)
            torch.cuda.synchronize()
            got[wb] = np.concatenate([r.theta.cpu().numpy(), r.nll.cpu().numpy()[:, None]], axis=1)
    finally:
        hf.fit_set_wave_bins(was)
        hf.fit_set_tuning(*shape)
    assert not np.array_equal(got[0], got[2048])
    np.testing.assert_array_equal(got[hf.WAVE_AUTO], got[2048 if B >= 1024 else 0])


@pytest.mark.parametrize("B, on", [(600, False), (1023, False), (1024, True)])
def test_automatic_choice_counts_waves(hf, B, on):
    """512 threads, of which one workgroup fits a CU: as many waves as at the
    default shape, so the same 1024 histograms."""
    import torch
    th = [500.0, 0.4, 0.1, 4.0, -0.7]
    spec = datagen.model_spec(2, 1, -1, 0.0, 1.0)
    rng = np.random.default_rng(B)
    lam = datagen.intensity_1d(spec, np.array(th), 700, 0.0, 1.0)
    c = torch.from_numpy(np.concatenate([datagen.poisson_counts(lam, rng) for _ in range(B)]).view(np.int32)).cuda()
    off = torch.arange(0, 700 * B + 1, 700).cuda()
    th0 = torch.as_tensor(np.array([datagen.perturb(th, 0.02, rng) for _ in range(B)])).cuda()
    rg = torch.tensor([[0.0, 1.0]], dtype=torch.float64).repeat(B, 1).cuda()
    m = hf.Model.from_spec(spec)
    was, shape = hf.fit_get_wave_bins(), hf.fit_get_tuning()
    got = {}
    try:
        hf.fit_set_tuning(2, 0, 512)
        for wb in (hf.WAVE_AUTO, 0, 2048):
            hf.fit_set_wave_bins(wb)
            got[wb] = hf.fit_batch(c, off, rg, m, th0).nll.cpu().numpy()
    finally:
        hf.fit_set_wave_bins(was)
        hf.fit_set_tuning(*shape)
    assert not np.array_equal(got[0], got[2048])
    np.testing.assert_array_equal(got[hf.WAVE_AUTO], got[2048 if on else 0])
