"""Complex SNR of FINDCHIRP's triggers against the FP64 oracle where the way it is evaluated changes: peak windows
around 256 samples (the listed row sums and the sums over the filters), 4096 firing slots and one batch more, capacities
below the trigger count, a ragged last window, and the smallest and largest column lengths."""
import numpy as np
import pytest

from oracle import pipeline as orc
from test_gpu_findchirp import F_LOW, FS, _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,count,threshold,window,capacity", [
    (1 << 13, 4096, 5.0, 256, 8192), (1 << 19, 64, 0.0, 8192, 4096), (1 << 19, 65, 0.0, 8192, 8192),
    (1 << 19, 64, 0.0, 8192, 100), (1 << 19, 64, 4.5, 3000, 4096), (1 << 19, 63, 4.5, 3000, 4096),
    (1 << 20, 33, 5.0, 256, 4096), (1 << 20, 33, 5.0, 255, 4096), (1 << 21, 18, 5.5, 1 << 21, 4096),
    (1 << 13, 3, 2.5, 300, 4096), (1 << 12, 4, 3.0, 512, 4096)])
def test_trigger_snr_matches_oracle(rfd, n, count, threshold, window, capacity):
    import torch
    psd, data, H, want, _ = _case(n, count, seed=n % 1009 + count)
    p = orc.prepare(psd, data, FS, F_LOW)
    plan = rfd.rfd_plan_create(psd, F_LOW, FS, n)
    filt, _ = rfd.rfd_findchirp_prepare(plan, torch.from_numpy(H).cuda())
    for _ in range(2):                       # the second call finds the first one's list
        buf = torch.zeros(capacity * 32, dtype=torch.uint8, device="cuda")
        buf, m = rfd.findchirp_filter(plan, torch.from_numpy(data).cuda(), filt, threshold, window, capacity, buf,
                                      raise_overflow=False)
        t = rfd.triggers_to_numpy(buf, min(m, capacity))
        near = np.abs(want - threshold).min() < 1e-5
        assert near or m == sum((want[:, a:a + window] > threshold).any(axis=1).sum() for a in range(0, n, window))
        assert len(t) > 0
        t = t[:4096]
        assert not t["flags"].any()
        z = np.array([orc.findchirp_snr(p, H[j]) for j in range(t["tmpl"].max() + 1)])[t["tmpl"], t["sample"]]
        # an FP32 transform of at most 2^21 points: 21 stages' roundings of values up to the largest SNR
        tol = 21 * 2.0 ** -24 * max(14.0, want.max())
        err = np.abs(t["z_re"] + 1j * t["z_im"] - z).max()
        print(f"[findchirp z N={n} W={window}] {len(t)} triggers, max |dz| {err:.2e} (tol {tol:.1e})")
        assert err <= tol
    rfd.rfd_plan_destroy(plan)
