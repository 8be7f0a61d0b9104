"""Epilogue of the overlap-save FIR: the test that lets a wave skip its window
keys never changes which windows fire, at every block shape the rule chooses."""
import numpy as np
import pytest

import synth
import gpu_cases as gc

pytestmark = pytest.mark.gpu


def _case(T, n=1 << 14):
    fs, f_low = 2048.0, 30.0
    w = synth.Workload("epilogue", 9, n, fs, f_low, 0, 1, 0, "fp32", "nonspin")
    rng = np.random.default_rng(T)
    ref = synth.taylorf2(synth.WaveformParams(6.0, 5.0), n, fs, f_low)
    H = synth.template_batch(w, [synth.WaveformParams(*m) for m in rng.uniform(5.0, 7.0, size=(5, 2))])
    s = synth.make_noise_spectrum(w, rng)
    return gc.Case("epilogue", n, fs, f_low, synth.psd_array(n, fs), synth.spectrum_to_time(s, n, fs), {0: ref},
                   [gc.SB(0, T, -(T // 2), H)])


def _peaks(s, threshold, window):
    from paper_2601_18835_amd import rfd
    buf, k = s.filter("ols32", threshold, window, s.n_templates * s.n)
    t = rfd.triggers_to_numpy(buf, k)
    return {(int(x["tmpl"]), int(x["sample"]) // window): (int(x["sample"]), float(x["rho"])) for x in t}


# K = 1024 general, 1024 in groups, 2048 in groups, 4096 general and in groups (12 and 14), the longest taps
@pytest.mark.parametrize("T", [33, 257, 256, 900, 1024, 512, 2048])
@pytest.mark.parametrize("window", [2048, 100])
def test_threshold_selects_exactly_the_louder_windows(T, window):
    case = _case(T)
    s = gc.gpu_search(case)
    every = _peaks(s, 0.0, window)
    assert len(every) == case.n_templates * -(-case.n // window)
    rho = np.sort([r for _, r in every.values()])
    for theta in (rho[len(rho) // 4], rho[len(rho) // 2], rho[-3], 0.999 * rho[-1]):
        got = _peaks(s, float(theta), window)
        for key, (sample, r) in every.items():
            if r > theta * (1 + 1e-6):      # rho^2 > theta^2 whatever the roundings of sqrt and square
                assert got.get(key) == (sample, r), (key, theta)
            elif r < theta * (1 - 1e-6):
                assert key not in got, (key, theta)
    s.close()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_data_fire_nothing(bad):
    case = _case(256)
    case.data = case.data.copy()
    case.data[1000] = bad
    s = gc.gpu_search(case)
    assert _peaks(s, 0.0, 2048) == {}
    s.close()
