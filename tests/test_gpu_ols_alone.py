"""Overlap-save with a sub-bank of a million block transforms among small ones of its shape: it takes a launch of its own, the
others share theirs, and the triggers are those of one launch per sub-bank."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("less", [0, 1])
def test_a_large_sub_bank_beside_shared_launches(rfd, less):
    import torch
    n, fs, f_low, T = 1 << 18, 2048.0, 30.0, 16
    w = synth.Workload("alone", 9, n, fs, f_low, 0, 1, 0, "ols32", "nonspin")
    rng = np.random.default_rng(3)
    psd = synth.psd_array(n, fs)
    data = torch.from_numpy(synth.spectrum_to_time(synth.make_noise_spectrum(w, rng), n, fs)).cuda()
    ref = torch.from_numpy(synth.taylorf2(synth.WaveformParams(6.0, 5.0), n, fs, f_low)).cuda()
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    L = rfd.rfd_ols_shape(plan, T)[1]
    large = -(-(1 << 20) // -(-n // L)) - less          # on either side of 2^20 transforms
    counts = [3, large, 5, 2]
    taps = rfd.rfd_taps_create(plan, np.concatenate([[0], np.cumsum(counts)]), [0] * 4, [T] * 4, [-8] * 4)
    H = torch.from_numpy(synth.template_batch(w, [synth.WaveformParams(*m) for m in rng.uniform(5.0, 7.0, size=(5, 2))])).cuda()
    H = H.repeat(100, 1) * torch.exp(0.01j * torch.arange(500, device="cuda"))[:, None]
    for b, c in enumerate(counts):
        for a in range(0, c, 500):
            rfd.rfd_make_taps(plan, taps, b, ref, H[:min(500, c - a)], a)
    rfd.rfd_dechirp(plan, data, ref, 0)
    window, theta, cap = 1 << 14, 3.5, 1 << 17
    buf, k = rfd.rfd_filter_bank(plan, taps, "ols32", theta, window, cap)
    out = torch.empty(cap * 32, dtype=torch.uint8, device="cuda")
    _, m = rfd.rfd_filter_bank_noalloc(plan, taps, "ols32", theta, window, cap, out)
    assert k == m > 0
    assert np.array_equal(rfd.triggers_to_numpy(buf, k), rfd.triggers_to_numpy(out, m))
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)
