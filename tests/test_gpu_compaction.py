"""Trigger compaction where its launches change shape: one block of slots (no counts),
a few (each block adds the counts before it), more than 4096 blocks (scanned counts),
and window maps of a range; against the slots' own peaks of the threshold-free call."""
import numpy as np
import pytest

import gpu_cases as gc
import synth

pytestmark = pytest.mark.gpu


def _search(n, count):
    fs, f_low = 2048.0, 30.0
    w = synth.Workload("compaction", 9, n, fs, f_low, 0, 1, 0, "fp32", "nonspin")
    rng = np.random.default_rng(n + count)
    ref = synth.taylorf2(synth.WaveformParams(6.0, 5.0), n, fs, f_low)
    H = synth.template_batch(w, [synth.WaveformParams(*m) for m in rng.uniform(5.0, 7.0, size=(count, 2))])
    s = synth.make_noise_spectrum(w, rng)
    return gc.gpu_search(gc.Case("compaction", n, fs, f_low, synth.psd_array(n, fs), synth.spectrum_to_time(s, n, fs),
                                 {0: ref}, [gc.SB(0, 32, -16, H)]))


# slots = 5 n / window: 5, 4095, 4100 (block edge), 8196, 20480, 16.8 million and one template's more than 4096 blocks
@pytest.mark.parametrize("n,window,count", [(1 << 12, 1 << 12, 5), (1 << 13, 10, 5), (1 << 12, 5, 5), (1 << 13, 5, 5),
                                            (1 << 12, 1, 5), (1 << 19, 1, 32), (1 << 19, 1, 33)])
def test_triggers_are_the_louder_slots_in_order(rfd, n, window, count):
    s = _search(n, count)
    nwin = -(-n // window)
    buf, k = s.filter("fp32", 0.0, window, count * nwin)
    every = rfd.triggers_to_numpy(buf, k)
    assert k == count * nwin
    key = every["tmpl"].astype(np.int64) * nwin + every["sample"] // window
    np.testing.assert_array_equal(key, np.arange(k))
    theta = float(np.sort(every["rho"])[-max(3, k // 7)])
    near = np.abs(every["rho"] - theta) <= 1e-6 * theta
    buf, m = s.filter("fp32", theta, window, k)
    got = rfd.triggers_to_numpy(buf, m)
    at = got["tmpl"].astype(np.int64) * nwin + got["sample"] // window
    assert np.all(np.diff(at) > 0)
    for name in ("sample", "tmpl", "subbank", "rho", "z_re", "z_im", "flags"):
        np.testing.assert_array_equal(got[name], every[name][at])
    np.testing.assert_array_equal(np.setdiff1d(np.flatnonzero((every["rho"] > theta) & ~near), at), [])
    assert np.all(every["rho"][at] >= theta * (1 - 1e-6))
    # too small a buffer: the count, and the first triggers
    out, full = s.filter("fp32", theta, window, m // 2, raise_overflow=False)
    assert full == m
    np.testing.assert_array_equal(rfd.triggers_to_numpy(out, m // 2), got[:m // 2])
    # a range reports the windows that it meets
    lo, length = n // 4, n // 2
    buf, r = s.filter_range("fp32", 0.0, window, lo, length, count * nwin)
    part = rfd.triggers_to_numpy(buf, r)
    inside = (every["sample"] // window * window >= lo) & ((every["sample"] // window + 1) * window <= lo + length)
    whole = (part["sample"] // window * window >= lo) & ((part["sample"] // window + 1) * window <= lo + length)
    for name in ("sample", "tmpl", "rho"):
        np.testing.assert_array_equal(part[name][whole], every[name][inside])
    s.close()
