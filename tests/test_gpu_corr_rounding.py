"""The FP64 correlations that the taps are made from, against sums in extended precision: with a ridge of 1e30 least-squares taps
are the correlation at their lags over the ridge."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# column transforms of 256, 256 and 512 points; few lags and lags in many turns of a workgroup
@pytest.mark.parametrize("log2n", [16, 17, 18])
@pytest.mark.parametrize("T", [128, 2048])
@pytest.mark.parametrize("centre", [False, True])
def test_correlations_carry_the_rounding_of_a_transform(rfd, log2n, T, centre):
    import torch
    n, fs, f_low = 1 << log2n, 2048.0, 30.0
    nb, lo = n // 2 + 1, int(np.ceil(f_low / (fs / n)))
    rng = np.random.default_rng(log2n + T)
    i = np.arange(nb, dtype=np.int64)
    sq = 0.0
    picked = 48
    for k0 in (-(T // 2), n // 5):
        psd = rng.uniform(0.5, 2.0, nb)
        h = rng.standard_normal((2, nb)) + 1j * rng.standard_normal((2, nb))
        w = np.zeros(nb)
        w[lo:n // 2] = 4.0 * (fs / n) / psd[lo:n // 2]
        x = w.astype(np.longdouble) * (h[1].astype(np.clongdouble) * np.conj(h[0].astype(np.clongdouble)))
        plan = rfd.rfd_plan_create(psd, f_low, fs, n)
        taps = rfd.rfd_taps_create(plan, [0, 1], [0], [T], [k0])
        rfd.rfd_make_taps(plan, taps, 0, torch.from_numpy(h[0]).cuda(), torch.from_numpy(h[1:]).cuda(),
                          method=rfd.RFD_TAPS_LS | (rfd.RFD_TAPS_CENTRE if centre else 0), ridge_eps=1e30)
        a, _, _, first = rfd.rfd_taps_get(taps, 0)
        rfd.rfd_taps_destroy(taps)
        rfd.rfd_plan_destroy(plan)
        lags = rng.choice(T, picked, replace=False)
        want = np.empty(picked, np.clongdouble)
        for j, l in enumerate(lags):
            turn = ((i * (first + int(l))) % n).astype(np.longdouble) * (np.longdouble("6.283185307179586476925286766559") / n)
            c, s = np.cos(turn), np.sin(turn)
            want[j] = np.sum(x.real * c - x.imag * s) + 1j * np.sum(x.real * s + x.imag * c)
        got = a[lags].astype(np.clongdouble)
        got *= np.sum(np.conj(got) * want) / np.sum(np.abs(got) ** 2)     # the ridge's own rounding is one factor for all
        sq += float(np.sum(np.abs(got - want) ** 2) / np.sum(np.abs(x) ** 2))
    # log2 N layers of independent roundings, each of at most 2^-53 (rms) of the values
    assert np.sqrt(sq / (2 * picked)) <= 2.0 ** -53 * np.sqrt(log2n)
