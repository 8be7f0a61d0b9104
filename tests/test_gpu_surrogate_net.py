"""Gradients of the surrogate's network over the widths and row counts at which their kernels change: hidden widths in
32s (one pass over the layers, one or two strips of columns per wave) and others (layer by layer), coefficient
counts around a 32-column strip, rows around a workgroup (16) and a chunk of the row sums (256)."""
import numpy as np
import pytest

import synth
from oracle import surrogate as osg
from test_gpu_surrogate import U32, bf16_round

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def search(rfd):
    from paper_2601_18835_amd.driver import RatioFilterSearch, SubBankSpec
    n, fs, f_low, taps = 1 << 13, 2048.0, 30.0, 160
    w = synth.Workload("network", 9, n, fs, f_low, 0, 1, taps, "fp32", "nonspin")
    s = RatioFilterSearch(synth.psd_array(n, fs), f_low, fs, n, [SubBankSpec(0, taps, -(taps // 2), 3)], max_refs=1)
    s.set_reference(0, synth.taylorf2(synth.WaveformParams(6.0, 5.0), n, fs, f_low))
    bank = [synth.WaveformParams(5.9 + 0.1 * j, 5.0) for j in range(3)]
    s.make_taps(0, s.to_dev(synth.template_batch(w, bank)))
    yield s
    s.close()


@pytest.mark.parametrize("hidden,coefs", [(32, 1), (64, 33), (256, 64), (256, 300), (288, 31), (512, 64), (40, 16),
                                          (544, 8)])
def test_gradients_at_every_width_and_row_count(rfd, search, hidden, coefs):
    import torch
    sur = rfd.rfd_surrogate_create(search.plan, search.taps, 0, coefs, hidden, 7)
    rng = np.random.default_rng(hidden + coefs)
    shapes = [(hidden, 4), (hidden,), (hidden, hidden), (hidden,), (coefs, hidden), (coefs,)]
    parts = [bf16_round(rng.uniform(-1, 1, q) * np.sqrt((6.0 if len(q) > 1 else 0.1) / q[-1])) for q in shapes]
    rfd.rfd_surrogate_set_state(sur, weights=np.concatenate([q.ravel() for q in parts]))
    params = [(a.astype(np.float64), b.astype(np.float64)) for a, b in zip(parts[::2], parts[1::2])]
    for n in (1, 15, 16, 17, 47, 255, 256, 257, 511, 1024):
        x = rng.uniform(-1, 1, size=(n, 4)).astype(np.float32)
        c = (0.3 * rng.standard_normal((n, coefs))).astype(np.float32)
        loss, g = rfd.rfd_surrogate_loss_grad(sur, torch.from_numpy(x).cuda(), torch.from_numpy(c).cuda())
        lo, go = osg.loss_and_grads(params, x.astype(np.float64), c.astype(np.float64))
        # FP32 sums of at most max(n, hidden) products through three layers, and the exponential of SiLU (a few
        # roundings of an argument of a few units); where an output comes close to its target, its error counts against the small difference
        y = osg.forward(params, x.astype(np.float64))[0]
        tol = (3 * max(n, hidden) + 32) * U32 * max(1.0, np.max(np.abs(y)) / np.max(np.abs(y - c)))
        assert abs(loss - lo) <= tol * lo
        o = 0
        for name, want in zip(("W1", "b1", "W2", "b2", "W3", "b3"), [q for pair in go for q in pair]):
            got = g[o:o + want.size].astype(np.float64)
            o += want.size
            err = np.max(np.abs(got - want.ravel())) / np.max(np.abs(want))
            assert err <= tol, (n, name, err)
        assert o == g.size
    rfd.rfd_surrogate_destroy(sur)
