"""A band split that is refused leaves the band series of the slot's last good one in use, also where the refused one's
column pass has already run."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1 << 10, 1 << 13])
def test_refused_split_keeps_the_series(rfd, n):
    import torch
    from paper_2601_18835_amd.driver import RatioFilterSearch, SubBankSpec
    fs, f_low = 2048.0, 30.0
    h = synth.taylorf2(synth.WaveformParams(2.0, 1.8), n, fs, f_low)
    psd = synth.psd_array(n, fs)
    s = RatioFilterSearch(psd, f_low, fs, n, [SubBankSpec(0, 1, 0, 1)])
    band = slice(s.info["i_low"], s.info["i_high"] + 1)
    power = np.abs(h) ** 2 / psd
    loud = n // 16                                        # three fifths of the power: three bands are too many
    h[loud] *= np.sqrt(1.5 * (power[band].sum() - power[loud]) / power[loud])
    s.set_reference(0, h)
    s.make_taps(0, h[None])
    w = synth.Workload("order", 9, n, fs, f_low, 0, 1, 0, "fp32", "nonspin")
    s.set_segment(synth.spectrum_to_time(synth.make_noise_spectrum(w, np.random.default_rng(3)), n, fs))
    s.dechirp_all()
    edges = s.bands(2)[0]
    buf, k = s.filter("fp32", 0.0, n // 8, 8)
    want = s.chisq(buf, k)
    assert k == 8 and np.all(np.isfinite(want))
    dev = torch.from_numpy(h).cuda()
    for bands in (3, 64):
        with pytest.raises(rfd.RfdError):
            rfd.rfd_dechirp_bands(s.plan, dev, 0, bands)
        np.testing.assert_array_equal(s.chisq(buf, k), want)
    np.testing.assert_array_equal(rfd.rfd_dechirp_bands(s.plan, dev, 0, 2), edges)
    np.testing.assert_array_equal(s.chisq(buf, k), want)
    s.close()
