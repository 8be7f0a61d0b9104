"""Least-squares taps made again by one taps object after what the cached Cholesky factor was made from has
changed, against FP64 solves on the host."""
import numpy as np
import pytest

import synth
from oracle import taps as otaps
from test_gpu_taps_blocks import setup  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _weights(n, fs, f_low, psd):
    w = np.zeros(n // 2 + 1)
    i_low = int(np.ceil(f_low / (fs / n)))
    w[i_low:n // 2] = 4.0 * (fs / n) / psd[i_low:n // 2]
    return w


def _check(rfd, taps, ref, wts, H, T, eps):
    """Every template's taps solve the normal equations and sigma_fit is their norm."""
    n = 2 * (ref.size - 1)
    M = otaps.gram(ref, wts, T)
    A = M + eps * M[0, 0].real * np.eye(T)
    for j in range(len(H)):
        a, sig, _, k0 = rfd.rfd_taps_get(taps, j)
        b = otaps.crosscorr(H[j], ref, wts, T, k0)
        # backward error of the solve and of the correlations, in units of |A| |a| + |b|
        res = np.linalg.norm(A @ a - b) / (A[0, 0].real * T * np.linalg.norm(a) + np.linalg.norm(b))
        assert res <= 1e-14 * max(T, 64)
        want = np.sqrt(np.real(np.conj(a) @ M @ a))
        # rounding of |M| |a|^2
        tol = 1e-15 * T * A[0, 0].real * T * np.linalg.norm(a) ** 2 / want ** 2 + 1e-12
        assert abs(sig / want - 1) <= tol


@pytest.mark.parametrize("T", [48, 320])
@pytest.mark.parametrize("centre", [False, True])
def test_factor_follows_the_psd_and_the_reference(rfd, setup, T, centre):  # noqa: F811
    import torch
    n, fs, f_low, psd, _, ref, H = setup
    H, eps = H[:3], 1e-4
    other = synth.taylorf2(synth.WaveformParams(6.4, 5.2), n, fs, f_low)
    f = np.arange(n // 2 + 1) * (fs / n)
    method = rfd.RFD_TAPS_LS | (rfd.RFD_TAPS_CENTRE if centre else 0)
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, 3], [0], [T], [-(T // 2)])
    h = torch.from_numpy(H).cuda()
    first = None
    for p, r in ((psd, ref), (2.0 * psd, ref), (np.where(f < 60.0, 3.0, 1.0) * psd, ref), (psd, other), (psd, ref)):
        rfd.rfd_plan_set_psd(plan, p)
        rfd.rfd_make_taps(plan, taps, 0, torch.from_numpy(r).cuda(), h, method=method, ridge_eps=eps)
        _check(rfd, taps, r, _weights(n, fs, f_low, p), H, T, eps)
        if first is None:
            first = [rfd.rfd_taps_get(taps, j) for j in range(3)]
    for j in range(3):                      # back to the first inputs: the first bits
        a, sig, _, k0 = rfd.rfd_taps_get(taps, j)
        assert np.array_equal(a, first[j][0]) and (sig, k0) == (first[j][1], first[j][3])
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)


def test_another_reference_in_the_same_buffer(rfd, setup):  # noqa: F811
    import torch
    n, fs, f_low, psd, wts, ref, H = setup
    T, eps = 100, 1e-4
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, 3], [0], [T], [-(T // 2)])
    r, h = torch.from_numpy(ref).cuda(), torch.from_numpy(H[:3]).cuda()
    rfd.rfd_make_taps(plan, taps, 0, r, h, ridge_eps=eps)
    # a reference without power in band is refused, and the taps that stand keep their lag windows
    before = [rfd.rfd_taps_get(taps, j) for j in range(3)]
    with pytest.raises(rfd.RfdError) as e:
        rfd.rfd_make_taps(plan, taps, 0, torch.zeros_like(r), h, method=rfd.RFD_TAPS_LS | rfd.RFD_TAPS_CENTRE,
                          ridge_eps=eps)
    assert e.value.code == rfd.RFD_E_INVALID
    for j in range(3):
        a, sig, _, k0 = rfd.rfd_taps_get(taps, j)
        assert np.array_equal(a, before[j][0]) and (sig, k0) == (before[j][1], before[j][3])
    other = synth.taylorf2(synth.WaveformParams(6.4, 5.2), n, fs, f_low)
    r.copy_(torch.from_numpy(other))
    rfd.rfd_make_taps(plan, taps, 0, r, h, ridge_eps=eps)
    _check(rfd, taps, other, wts, H[:3], T, eps)
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)


@pytest.mark.parametrize("T", [48, 320])
def test_a_refused_ridge_leaves_no_factor_behind(rfd, setup, T):  # noqa: F811
    import torch
    n, fs, f_low, psd, wts, ref, H = setup
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, 3], [0], [T], [-(T // 2)])
    r, h = torch.from_numpy(ref).cuda(), torch.from_numpy(H[:3]).cuda()
    rfd.rfd_make_taps(plan, taps, 0, r, h, ridge_eps=1e-4)
    first = [rfd.rfd_taps_get(taps, j) for j in range(3)]
    def refused():
        with pytest.raises(rfd.RfdError) as e:      # the band ends below fs / 2: M alone is singular to rounding
            rfd.rfd_make_taps(plan, taps, 0, r, h, ridge_eps=0.0)
        assert e.value.code == rfd.RFD_E_INVALID

    refused()
    rfd.rfd_make_taps(plan, taps, 0, r, h, ridge_eps=1e-4)
    for j in range(3):
        a, sig, _, k0 = rfd.rfd_taps_get(taps, j)
        assert np.array_equal(a, first[j][0]) and (sig, k0) == (first[j][1], first[j][3])
    refused()
    with pytest.raises(rfd.RfdError) as e:          # nothing to whiten training taps with
        rfd.rfd_surrogate_create(plan, taps, 0, 2, 32, 1)
    assert e.value.code == rfd.RFD_E_STATE
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)


def _norms(a, M):
    """sqrt(a^H M a) in extended precision, and the error that rounding sums of |a| |M| |a| can leave."""
    al, Ml = a.astype(np.clongdouble), M.astype(np.clongdouble)
    sq = np.real(np.einsum("jl,jl->j", np.conj(al), al @ Ml.T)).astype(np.float64)
    T, g0 = M.shape[0], M[0, 0].real
    # 2 T products in a row, and g itself good to a few roundings of g[0] on either side
    return np.sqrt(sq), 2.0 ** -52 * (2 * T + 32) * g0 * np.sum(np.abs(a), axis=1) ** 2 / sq


@pytest.mark.parametrize("T,count", [(1, 3), (15, 8), (16, 9), (17, 3), (128, 3), (129, 3), (256, 17), (257, 3), (500, 3)])
@pytest.mark.parametrize("eps", [1e-8, 1e-4, 1.0, 1e4, 1e8, 1e16])
def test_norm_at_every_ridge(rfd, setup, T, count, eps):  # noqa: F811
    import torch
    n, fs, f_low, psd, wts, ref, H = setup
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, count], [0], [T], [-(T // 2)])
    rfd.rfd_make_taps(plan, taps, 0, torch.from_numpy(ref).cuda(), torch.from_numpy(H[:count]).cuda(), ridge_eps=eps)
    got = [rfd.rfd_taps_get(taps, j)[:2] for j in range(count)]
    want, tol = _norms(np.array([a for a, _ in got]), otaps.gram(ref, wts, T))
    assert np.all(np.abs(np.array([s for _, s in got]) / want - 1) <= tol)
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)


@pytest.mark.parametrize("T", [100, 144, 260])
def test_norms_of_more_templates_than_a_batch(rfd, T):
    import torch
    n, fs, f_low, count = 1 << 10, 1024.0, 20.0, 4101
    rng = np.random.default_rng(5)
    draw = lambda m: rng.standard_normal((m, n // 2 + 1)) + 1j * rng.standard_normal((m, n // 2 + 1))  # noqa: E731
    ref, H = draw(1)[0], draw(count)
    psd = rng.uniform(0.5, 2.0, n // 2 + 1)
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, count], [0], [T], [-(T // 2)])
    rfd.rfd_make_taps(plan, taps, 0, torch.from_numpy(ref).cuda(), torch.from_numpy(H).cuda())
    picked = [0, 7, 8, 4095, 4096, 4099, 4100]
    got = [rfd.rfd_taps_get(taps, j)[:2] for j in picked]
    want, tol = _norms(np.array([a for a, _ in got]), otaps.gram(ref, _weights(n, fs, f_low, psd), T))
    assert np.all(np.abs(np.array([s for _, s in got]) / want - 1) <= tol)
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)


@pytest.mark.parametrize("T,count", [(16, 3), (64, 3), (100, 9), (200, 3), (512, 3), (600, 512), (600, 513), (1100, 513)])
@pytest.mark.parametrize("eps", [1e-10, 1e-8, 1e-4])
def test_solve_is_backward_stable_at_small_ridges(rfd, setup, T, count, eps):  # noqa: F811
    import torch
    n, fs, f_low, psd, wts, ref, H = setup
    H = np.tile(H, (32, 1))[:count] * np.exp(0.1j * np.arange(count))[:, None]
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, count], [0], [T], [-(T // 2)])
    rfd.rfd_make_taps(plan, taps, 0, torch.from_numpy(ref).cuda(), torch.from_numpy(H).cuda(), ridge_eps=eps)
    M = otaps.gram(ref, wts, T)
    A = M + eps * M[0, 0].real * np.eye(T)
    for j in {0, count // 2, count - 1}:
        a = rfd.rfd_taps_get(taps, j)[0]
        b = otaps.crosscorr(H[j], ref, wts, T, -(T // 2))
        # two substitutions leave a few roundings of |L| |L^H| |a|, at most T A[0,0] |a|; M, b and the products
        # here as many again
        res = np.linalg.norm(A @ a - b) / (A[0, 0].real * T * np.linalg.norm(a) + np.linalg.norm(b))
        assert res <= 64 * 2.0 ** -53
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)


def test_taps_do_not_depend_on_earlier_calls(rfd):
    import torch
    n, fs, f_low = 1 << 10, 1024.0, 20.0
    rng = np.random.default_rng(6)
    draw = lambda m: torch.from_numpy(rng.standard_normal((m, n // 2 + 1)) + 1j * rng.standard_normal((m, n // 2 + 1))).cuda()  # noqa: E731,E501
    ref, H, more = draw(1)[0], draw(256), draw(600)
    plan = rfd.rfd_plan_create(rng.uniform(0.5, 2.0, n // 2 + 1), f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, 256, 856], [0, 0], [512, 100], [-256, -50])
    rfd.rfd_make_taps(plan, taps, 0, ref, H)
    first = [rfd.rfd_taps_get(taps, j)[:2] for j in (0, 100, 255)]
    rfd.rfd_make_taps(plan, taps, 1, ref, more)      # more scratch than the first call had
    rfd.rfd_make_taps(plan, taps, 0, ref, H)
    for (a, sig), j in zip(first, (0, 100, 255)):
        got = rfd.rfd_taps_get(taps, j)
        assert np.array_equal(got[0], a) and got[1] == sig
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)


def test_calls_queued_behind_each_other(rfd, setup):  # noqa: F811
    """Many calls in a row without a wait: each finds out about its factor while the ones before it still run."""
    import torch
    n, fs, f_low, psd, wts, ref, H = setup
    T, count = 64, 1500
    plan = rfd.rfd_plan_create(psd, f_low, fs, n)
    taps = rfd.rfd_taps_create(plan, [0, count], [0], [T], [-(T // 2)])
    other = synth.taylorf2(synth.WaveformParams(6.4, 5.2), n, fs, f_low)
    h = torch.from_numpy(np.tile(H, (100, 1))[:count]).cuda()
    r = [torch.from_numpy(x).cuda() for x in (ref, other)]
    for k in range(40):
        rfd.rfd_make_taps(plan, taps, 0, r[k // 20], h, method=rfd.RFD_TAPS_LS | rfd.RFD_TAPS_CENTRE)
    M = otaps.gram(other, wts, T)
    A = M + 1e-4 * M[0, 0].real * np.eye(T)
    for j in (0, 700, count - 1):
        a, _, _, k0 = rfd.rfd_taps_get(taps, j)
        b = otaps.crosscorr(H[j % len(H)], other, wts, T, k0)
        res = np.linalg.norm(A @ a - b) / (A[0, 0].real * T * np.linalg.norm(a) + np.linalg.norm(b))
        assert res <= 1e-14 * T
    rfd.rfd_taps_destroy(taps)
    rfd.rfd_plan_destroy(plan)
