"""Least-squares taps where the blocked solve changes shape: tap counts around its 64-row blocks
and around 1024 (eight and four templates per workgroup), template counts around those
groups, small and vanishing ridges; against FP64 solves on the host."""
import numpy as np
import pytest

import synth
from oracle import taps as otaps

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    n, fs, f_low = 1 << 13, 2048.0, 30.0
    w = synth.Workload("blocks", 9, n, fs, f_low, 0, 1, 0, "fp32", "nonspin")
    rng = np.random.default_rng(11)
    ref = synth.taylorf2(synth.WaveformParams(6.0, 5.0), n, fs, f_low)
    H = synth.template_batch(w, [synth.WaveformParams(*m) for m in rng.uniform(5.0, 7.0, size=(17, 2))])
    psd = synth.psd_array(n, fs)
    i_low = int(np.ceil(f_low / (fs / n)))
    wts = np.zeros(n // 2 + 1)
    wts[i_low:n // 2] = 4.0 * (fs / n) / psd[i_low:n // 2]
    return n, fs, f_low, psd, wts, ref, H


@pytest.mark.parametrize("T", [1, 2, 63, 64, 65, 128, 200, 1023, 1024, 1025, 2048])
@pytest.mark.parametrize("count", [1, 8, 17])
def test_taps_solve_the_normal_equations(rfd, setup, T, count):
    import torch
    n, fs, f_low, psd, wts, ref, H = setup
    eps = 1e-4
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, count], [0], [T], [-(T // 2)])
    rfd.rfd_make_taps(plan, taps, 0, torch.from_numpy(ref).cuda(), torch.from_numpy(H[:count]).cuda(), ridge_eps=eps)
    M = otaps.gram(ref, wts, T)
    lam = eps * M[0, 0].real
    A = M + lam * np.eye(T)
    k = np.arange(n // 2 + 1)[None]
    lags = (np.arange(T) - T // 2)[:, None]
    turn = np.exp(2j * np.pi * ((k * lags) % n) / n)
    for j in {0, count // 2, count - 1}:
        a, sig, t, k0 = rfd.rfd_taps_get(taps, j)
        assert (t, k0) == (T, -(T // 2))
        b = turn @ (wts * H[j] * np.conj(ref))
        # backward error of the solve and of the correlations, in units of |A| |a| + |b|
        res = np.linalg.norm(A @ a - b) / (A[0, 0].real * T * np.linalg.norm(a) + np.linalg.norm(b))
        assert res <= 1e-14 * max(T, 64)
        want = np.sqrt(np.real(np.conj(a) @ M @ a))
        # the two forms of the norm differ by rounding of |M| |a|^2
        tol = 1e-15 * T * A[0, 0].real * T * np.linalg.norm(a) ** 2 / want ** 2 + 1e-12
        assert abs(sig / want - 1) <= tol
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)


@pytest.mark.parametrize("T", [48, 320])
def test_another_ridge_refactors(rfd, setup, T):
    import torch
    n, fs, f_low, psd, wts, ref, H = setup
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, 3], [0], [T], [-(T // 2)])
    r, h = torch.from_numpy(ref).cuda(), torch.from_numpy(H[:3]).cuda()
    M = otaps.gram(ref, wts, T)
    turn = np.exp(2j * np.pi * ((np.arange(n // 2 + 1)[None] * (np.arange(T) - T // 2)[:, None]) % n) / n)
    b = turn @ (wts * H[1] * np.conj(ref))
    for eps in (1e-4, 1e-2, 1e-6):
        rfd.rfd_make_taps(plan, taps, 0, r, h, ridge_eps=eps)
        a = rfd.rfd_taps_get(taps, 1)[0]
        want = np.linalg.solve(M + eps * M[0, 0].real * np.eye(T), b)
        # forward error: condition (at most T / eps) times rounding
        assert np.linalg.norm(a - want) <= 64 * 2.0 ** -52 * T / eps * np.linalg.norm(want)
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)
