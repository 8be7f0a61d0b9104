"""Least-squares taps on both sides of the line between one launch for the whole solve and one per block row: tap counts
around 512 and above 1024, template counts around 256."""
import numpy as np
import pytest

from oracle import taps as otaps
from test_gpu_taps_blocks import setup  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [511, 512, 577, 1030])
@pytest.mark.parametrize("count", [255, 256, 257])
def test_taps_solve_the_normal_equations(rfd, setup, T, count):  # noqa: F811
    import torch
    n, fs, f_low, psd, wts, ref, H = setup
    H = np.tile(H, (16, 1))[:count] * np.exp(0.1j * np.arange(count))[:, None]
    eps = 1e-4
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, count], [0], [T], [-(T // 2)])
    rfd.rfd_make_taps(plan, taps, 0, torch.from_numpy(ref).cuda(), torch.from_numpy(H).cuda(), ridge_eps=eps)
    M = otaps.gram(ref, wts, T)
    A = M + eps * M[0, 0].real * np.eye(T)
    k = np.arange(n // 2 + 1)[None]
    turn = np.exp(2j * np.pi * ((k * (np.arange(T) - T // 2)[:, None]) % n) / n)
    for j in (0, 7, 8, count // 2, count - 1):
        a, sig, t, k0 = rfd.rfd_taps_get(taps, j)
        b = turn @ (wts * H[j] * np.conj(ref))
        # backward error of the solve and of the correlations, in units of |A| |a| + |b|
        res = np.linalg.norm(A @ a - b) / (A[0, 0].real * T * np.linalg.norm(a) + np.linalg.norm(b))
        assert res <= 1e-14 * T
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)
