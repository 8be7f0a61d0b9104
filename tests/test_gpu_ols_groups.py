"""Overlap-save over many sub-banks, whose launches are shared by block size, up to 32 of them and 128 MiB of block spectra
at a time: exactly the triggers of each sub-bank filtered by itself."""
import numpy as np
import pytest

import gpu_cases as gc
import synth

pytestmark = pytest.mark.gpu


# mixed block sizes and forms; more of one than a launch takes; more block spectra than one takes; one launch each
@pytest.mark.parametrize("n,taps", [(1 << 13, [40, 256, 257, 700, 1024, 40, 300, 256, 1300, 64]), (1 << 12, [100] * 35),
                                    (1 << 20, [1024] * 14), (1 << 13, [100, 1024])])
def test_shared_launches_equal_single_sub_banks(rfd, n, taps):
    fs, f_low = 2048.0, 30.0
    w = synth.Workload("groups", 9, n, fs, f_low, 0, 1, 0, "ols32", "nonspin")
    rng = np.random.default_rng(n + len(taps))
    refs = {r: synth.taylorf2(synth.WaveformParams(6.0 + 0.05 * r, 5.0), n, fs, f_low) for r in range(len(taps))}
    banks = [synth.template_batch(w, [synth.WaveformParams(*m) for m in rng.uniform(5.0, 7.0, size=(1 + r % 3, 2))])
             for r in range(len(taps))]
    psd = synth.psd_array(n, fs)
    data = synth.spectrum_to_time(synth.make_noise_spectrum(w, rng), n, fs)
    window, theta = 500, 1.0
    nwin = -(-n // window)

    def run(refs, sbs):
        s = gc.gpu_search(gc.Case("groups", n, fs, f_low, psd, data, refs, sbs))
        cap = nwin * sum(len(b.H) for b in sbs)
        buf, k = s.filter("ols32", theta, window, cap)
        whole = rfd.triggers_to_numpy(buf, k)
        buf, k = s.filter_range("ols32", theta, window, n // 4, n // 2, cap)
        part = rfd.triggers_to_numpy(buf, k)
        s.close()
        return whole, part

    got = run(refs, [gc.SB(r, T, -(T // 2), H) for r, (T, H) in enumerate(zip(taps, banks))])
    first = 0
    for r, (T, H) in enumerate(zip(taps, banks)):
        for all_, one in zip(got, run({0: refs[r]}, [gc.SB(0, T, -(T // 2), H)])):
            mine = all_[all_["subbank"] == r]
            np.testing.assert_array_equal(mine["tmpl"] - first, one["tmpl"])
            for name in ("sample", "rho", "z_re", "z_im", "flags"):
                np.testing.assert_array_equal(mine[name], one[name], err_msg=f"sub-bank {r} {name}")
        first += len(H)
