"""Window peaks of the direct forms over the windows at which their epilogue changes: shorter than, equal to and not
dividing a 16-sample block or a tile, one window per workgroup and one per segment; exactly the peaks (first of equal
ones) of the same call's sample by sample values."""
import numpy as np
import pytest

import gpu_cases as gc
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["fp32", "bf16x3", "fp16x3"])
@pytest.mark.parametrize("n,count", [(1 << 12, 9), (1 << 15, 35)])
def test_window_peaks_are_the_samples_peaks(rfd, form, n, count):
    fs, f_low = 2048.0, 30.0
    w = synth.Workload("epilogue", 9, n, fs, f_low, 0, 1, 0, form, "nonspin")
    rng = np.random.default_rng(n + count)
    ref = synth.taylorf2(synth.WaveformParams(6.0, 5.0), n, fs, f_low)
    H = synth.template_batch(w, [synth.WaveformParams(*m) for m in rng.uniform(5.0, 7.0, size=(count, 2))])
    s = gc.gpu_search(gc.Case("epilogue", n, fs, f_low, synth.psd_array(n, fs),
                              synth.spectrum_to_time(synth.make_noise_spectrum(w, rng), n, fs), {0: ref},
                              [gc.SB(0, 24, -12, H)]))
    buf, k = s.filter(form, 0.0, 1, count * n)
    assert k == count * n
    rho = rfd.triggers_to_numpy(buf, k)["rho"].reshape(count, n)
    for window in (2, 7, 15, 16, 17, 31, 32, 100, 127, 128, 129, 256, 1000, 2048, 2049, n - 1, n):
        starts = range(0, n, window)
        peak = np.array([[a + int(np.argmax(rho[j, a:a + window])) for a in starts] for j in range(count)])
        for theta in (0.0, float(np.quantile(rho, 0.999)), 1e3):
            buf, m = s.filter(form, theta, window, peak.size)
            t = rfd.triggers_to_numpy(buf, m)
            j, q = np.nonzero(np.take_along_axis(rho, peak, 1) > theta)
            np.testing.assert_array_equal(t["tmpl"], j, err_msg=f"W={window} theta={theta}")
            np.testing.assert_array_equal(t["sample"], peak[j, q])
            np.testing.assert_array_equal(t["rho"], rho[j, peak[j, q]])
    s.close()
