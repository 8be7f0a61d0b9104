"""Band split and band series of the chi^2 test where the launches divide: edges found
from sums in another order equal the sequential rule's, also where a share falls exactly on
a bin, and band series made in several batches add up to the reference series."""
import numpy as np
import pytest

import synth
from oracle import chisq as ocq

pytestmark = pytest.mark.gpu


def _plan(rfd, n, psd, f_low=20.0, fs=2048.0):
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    info = rfd.rfd_plan_info_get(plan)
    w = np.zeros(n // 2 + 1)
    w[info["i_low"]:info["i_high"] + 1] = 4.0 * (fs / n) / psd[info["i_low"]:info["i_high"] + 1]
    return plan, info, w


def _series(rfd, plan, n, h, bands, seed):
    import torch
    data = torch.from_numpy(np.random.default_rng(seed).standard_normal(n)).to("cuda")
    hd = torch.from_numpy(h).to("cuda")
    rfd.rfd_dechirp(plan, data, hd)
    return rfd.rfd_dechirp_bands(plan, hd, 0, bands)


# one chunk of bins, a few, and 512 of them; the fewest and the most bands
@pytest.mark.parametrize("n", [1 << 10, 1 << 13, 1 << 20])
@pytest.mark.parametrize("bands", [2, 3, 16, 64])
def test_edges_follow_the_sequential_rule(rfd, n, bands):
    psd = synth.psd_array(n, 2048.0)
    plan, info, w = _plan(rfd, n, psd)
    rng = np.random.default_rng(n + bands)
    h = (rng.standard_normal(n // 2 + 1) + 1j * rng.standard_normal(n // 2 + 1)).astype(np.complex128) * psd ** 0.5
    try:
        want = ocq.band_edges(h, w, info["i_low"], info["i_high"], bands)
    except ValueError:
        with pytest.raises(rfd.RfdError):
            _series(rfd, plan, n, h, bands, 1)
    else:
        np.testing.assert_array_equal(_series(rfd, plan, n, h, bands, 1), want)
    rfd.rfd_plan_destroy(plan)


# equal power in every bin: with 992 * 4 bins each share ends exactly on one
@pytest.mark.parametrize("bands", [2, 4, 31, 62])
def test_shares_that_end_on_a_bin(rfd, bands):
    n = 1 << 13                                       # df = 1/4: 4 df / psd = 1
    plan, info, w = _plan(rfd, n, np.ones(n // 2 + 1), f_low=32.0)
    h = np.ones(n // 2 + 1, dtype=np.complex128)
    assert set(w) == {0.0, 1.0}
    np.testing.assert_array_equal(_series(rfd, plan, n, h, bands, 2),
                                  ocq.band_edges(h, w, info["i_low"], info["i_high"], bands))
    rfd.rfd_plan_destroy(plan)


def test_batched_bands_add_up_to_the_reference_series(rfd):
    """2^20 samples take 8 bands a batch: 11 bands are two batches.  Band series are only read by
    the test statistic, so they are compared through it: with one tap and shares f_b, chi^2 at a trigger
    is sum_b |z_b - f_b z|^2 / f_b from numpy's band series."""
    import torch
    from paper_2601_18835_amd.driver import RatioFilterSearch, SubBankSpec
    n, bands, fs, f_low = 1 << 20, 11, 2048.0, 20.0
    psd = synth.psd_array(n, fs)
    w_ = synth.Workload("bands", 9, n, fs, f_low, 0, 1, 0, "fp32", "nonspin")
    h = synth.taylorf2(synth.WaveformParams(2.0, 1.8), n, fs, f_low)
    s = RatioFilterSearch(psd, f_low, fs, n, [SubBankSpec(0, 1, 0, 1)])
    s.set_reference(0, h)
    s.make_taps(0, h[None])
    data = synth.spectrum_to_time(synth.make_noise_spectrum(w_, np.random.default_rng(3)), n, fs)
    s.set_segment(data)
    s.dechirp_all()
    edges = s.bands(bands)[0]
    buf, k = s.filter("fp32", 4.0, 2048, 4096)
    trig = rfd.triggers_to_numpy(buf, k)
    assert k > 3
    got = s.chisq(buf, k)
    info = s.info
    w = np.zeros(n // 2 + 1)
    w[info["i_low"]:info["i_high"] + 1] = 4.0 * (fs / n) / psd[info["i_low"]:info["i_high"] + 1]
    np.testing.assert_array_equal(edges, ocq.band_edges(h, w, info["i_low"], info["i_high"], bands))
    zb = ocq.reference_band_series(np.fft.rfft(data) / fs, h, w, edges)[:, trig["sample"]]
    f = ocq.band_fractions(h, w, np.ones(1), 0, edges)
    want = ocq.chisq(zb, f)
    # FP32 band values of up to max |z_b| (2^-23 each, 11 of them squared over a share of 1/11)
    tol = 2.0 ** -23 * 4 * bands * np.max(np.abs(zb)) * np.sqrt(np.max(want))
    assert np.max(np.abs(got - want)) <= tol
    s.close()
