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
    loud = n // 16
    h[loud] *= 1e3 * np.sqrt(n) * np.abs(h).max() / np.abs(h[loud])     # nearly all the power: three bands are too many
    s = RatioFilterSearch(synth.psd_array(n, fs), f_low, fs, n, [SubBankSpec(0, 1, 0, 1)])
    s.set_reference(0, h)
    s.make_taps(0, h[None])
    s.set_segment(np.random.default_rng(3).standard_normal(n))
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
