"""Performance cases: what a search built on this library has it do, per segment and at set-up.

Inputs are synthetic and seeded: coloured Gaussian noise in an analytic detector PSD with one injected signal, and
stationary-phase inspiral templates grouped in sub-banks around reference templates.  `exact` evaluates the same
quantities in complex128 with torch.fft and dense solves.
"""
import math

import numpy as np
import torch

from paper_2601_18835_amd import rfd
from paper_2601_18835_amd.driver import RatioFilterSearch, SubBankSpec

FS = 2048.0
MSUN_S = 4.925490947641267e-6
RIDGE = 1e-4


# ------------------------------------------------------------------ cases
def listed():
    return [
        # one reference, 16 short-filter templates: the smallest search call, made of launches and latency
        dict(name="small_fp32", kind="bank", n=1 << 17, refs=1, per_ref=16, taps=64, uneven=False, form="fp32",
             graph=False, f_low=30.0),
        # short filters on the matrix cores (hi/lo 16-bit operands), where they beat the FFT blocks
        dict(name="short_bf16x3", kind="bank", n=1 << 18, refs=1, per_ref=250, taps=48, uneven=False, form="bf16x3",
             graph=False, f_low=30.0),
        # a spinning bank on one reference, 256 s segment, 256 taps
        dict(name="spin_t256", kind="bank", n=1 << 19, refs=1, per_ref=4096, taps=256, uneven=False, form="ols32",
             graph=False, f_low=20.0),
        # long filters on a 512 s segment, the whole segment replayed as one graph: an offline search's inner loop
        dict(name="ecc_t1024", kind="bank", n=1 << 20, refs=8, per_ref=512, taps=1024, uneven=False, form="ols32",
             graph=True, f_low=15.0),
        # uneven sub-banks with ragged tap counts, 256 s segment
        dict(name="tidal_uneven", kind="bank", n=1 << 19, refs=16, per_ref=250, taps=1024, uneven=True, form="ols32",
             graph=False, f_low=20.0),
        # the reference series of a new segment alone
        dict(name="dechirp_32refs", kind="dechirp", n=1 << 20, refs=32, fp64=False, f_low=15.0),
        # low latency: a stream primed with a window, then fed one second at a time
        dict(name="stream_1s", kind="stream", n=1 << 20, refs=32, per_ref=64, taps=1024, increment=2048, pushes=4,
             f_low=15.0),
        # set-up of a sub-bank with lag windows on each template's correlation peak, and its first filtering
        dict(name="taps_centred_t1024", kind="taps", n=1 << 20, per_ref=256, taps=1024, centre=True, window=False,
             f_low=15.0),
        # the same for a shorter filter with lag windows on zero
        dict(name="taps_t256", kind="taps", n=1 << 19, per_ref=500, taps=256, centre=False, window=False, f_low=20.0),
        # the one-FFT-per-template search that the ratio filter is compared with
        dict(name="findchirp", kind="findchirp", n=1 << 20, templates=250, f_low=15.0),
        # a segment with the chi-squared test at its triggers
        dict(name="chisq_16bands", kind="chisq", n=1 << 19, refs=4, per_ref=64, taps=256, bands=16, f_low=20.0),
        # one gradient of the learned tap generator's network, forward and backward
        dict(name="surrogate_grad", kind="surrogate", n=1 << 13, taps=64, basis=64, hidden=256, rows=1024, f_low=30.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["bank", "bank", "bank", "bank", "dechirp", "stream", "taps", "taps", "findchirp", "chisq",
                       "surrogate"])
    f_low = rng.choice([15.0, 20.0, 30.0])
    log2n = rng.randint(15, 20)
    if kind == "bank":
        form = rng.choice(["ols32", "ols32", "ols32", "fp32", "bf16x3", "fp16x3"])
        taps = _log_int(rng, 32, 1500) if form == "ols32" else _log_int(rng, 16, 160)
        refs = rng.choice([1, 1, 2, 5, 8, 16])
        # templates x samples: at most those of the largest listed case, a tenth of them for the direct forms
        most = (1 << 32) // (1 << log2n) // refs // (1 if form == "ols32" else 10)
        return dict(kind=kind, n=1 << log2n, refs=refs, per_ref=_log_int(rng, 8, max(9, min(4096, most))), taps=taps,
                    uneven=refs > 1 and rng.random() < 0.5, form=form, graph=rng.random() < 0.5, f_low=f_low)
    if kind == "dechirp":
        return dict(kind=kind, n=1 << log2n, refs=_log_int(rng, 1, 32), fp64=rng.random() < 0.25, f_low=f_low)
    if kind == "stream":
        return dict(kind=kind, n=1 << rng.randint(17, 20), refs=_log_int(rng, 1, 32), per_ref=_log_int(rng, 8, 64),
                    taps=_log_int(rng, 64, 1200), increment=256 * rng.choice([2, 4, 8, 8, 16]),
                    pushes=rng.randint(1, 4), f_low=f_low)
    if kind == "taps":
        return dict(kind=kind, n=1 << log2n, per_ref=_log_int(rng, 8, 250), taps=_log_int(rng, 32, 1024),
                    centre=rng.random() < 0.5, window=rng.random() < 0.2, f_low=f_low)
    if kind == "findchirp":
        return dict(kind=kind, n=1 << log2n, templates=_log_int(rng, 8, 250), f_low=f_low)
    if kind == "chisq":
        return dict(kind=kind, n=1 << rng.randint(15, 19), refs=rng.randint(1, 4), per_ref=_log_int(rng, 8, 64),
                    taps=_log_int(rng, 32, 512), bands=rng.randint(4, 20), f_low=f_low)
    return dict(kind=kind, n=1 << 13, taps=rng.randint(32, 100), basis=rng.choice([16, 32, 64]),
                hidden=rng.choice([64, 128, 256]), rows=_log_int(rng, 64, 1024), f_low=30.0)


# ----------------------------------------------------------------- inputs
def _band(case):
    n = case["n"]
    return int(math.ceil(case["f_low"] / (FS / n))), n // 2 - 1


def _psd(n):
    f = np.arange(n // 2 + 1) * (FS / n)
    f[0] = f[1]
    x = f / 215.0
    return 1e-46 * (x ** -4.14 - 5.0 / x ** 2 + 111.0 * (1.0 - x ** 2 + 0.5 * x ** 4) / (1.0 + 0.5 * x ** 2))


def _coefficients(p):
    """Phase coefficients [count, 10] on the frequency powers of _waveforms: post-Newtonian to 3.5 orders with aligned
    spin, leading eccentric and tidal terms.  p: columns m1, m2, chi, e0, tidal."""
    m1, m2, chi, e0, lam = p.T
    m = m1 + m2
    eta = m1 * m2 / m ** 2
    pi, g = math.pi, math.pi * m * MSUN_S
    beta = 113.0 / 12.0 * ((m1 / m) ** 2 + (m2 / m) ** 2) * chi + 25.0 * eta / 2.0 * chi
    k3 = -16.0 * pi + 4.0 * beta
    k2 = 3715.0 / 756.0 + 55.0 * eta / 9.0
    k4 = 15293365.0 / 508032.0 + 27145.0 * eta / 504.0 + 3085.0 * eta ** 2 / 72.0 - 79.0 / 0.8 * eta * chi ** 2
    k5 = pi * (38645.0 / 756.0 - 65.0 * eta / 9.0)
    k6 = (11583231236531.0 / 4694215680.0 - 640.0 * pi ** 2 / 3.0 - 6848.0 / 21.0 * (0.5772156649015329 + math.log(4.0))
          + (-15737765635.0 / 3048192.0 + 2255.0 * pi ** 2 / 12.0) * eta + 76055.0 * eta ** 2 / 1728.0
          - 127825.0 * eta ** 3 / 1296.0)
    k7 = pi * (77096675.0 / 254016.0 + 378515.0 * eta / 1512.0 - 74045.0 * eta ** 2 / 756.0)
    lv = np.log(g) / 3.0                                    # log v = lv + log(f) / 3
    a = 3.0 / (128.0 * eta)

    def v(k):
        return g ** (k / 3.0)

    return np.stack([a * v(-5), -a * v(-5) * 2355.0 / 1462.0 * e0 ** 2 * 10.0 ** (19.0 / 9.0), a * k2 * v(-3),
                     a * k3 * v(-2), a * k4 * v(-1), a * k5 * (1.0 + 3.0 * (lv + 0.5 * math.log(6.0))) - pi / 4.0,
                     a * k5, a * v(1) * (k6 - 6848.0 / 21.0 * lv), -a * v(1) * 6848.0 / 63.0,
                     a * (k7 * v(2) - 19.5 * lam * v(5))], axis=1)


def _waveforms(case, p):
    """complex128 [count, N/2 + 1] on the GPU: f^(-7/6) exp(-i psi) from f_low to the last stable orbit."""
    n = case["n"]
    lo, hi = _band(case)
    f = torch.arange(lo, hi + 1, dtype=torch.float64, device="cuda") * (FS / n)
    lf = torch.log(f)
    powers = torch.stack([f ** (-5.0 / 3.0), f ** (-34.0 / 9.0), f ** -1.0, f ** (-2.0 / 3.0), f ** (-1.0 / 3.0),
                          torch.ones_like(f), lf, f ** (1.0 / 3.0), lf * f ** (1.0 / 3.0), f ** (2.0 / 3.0)])
    psi = torch.zeros((len(p), f.numel()), dtype=torch.float64, device="cuda")
    c = torch.from_numpy(_coefficients(p)).cuda()
    for k in range(powers.shape[0]):
        psi.addcmul_(c[:, k:k + 1], powers[k][None])
    isco = torch.from_numpy(1.0 / (6.0 ** 1.5 * math.pi * (p[:, 0] + p[:, 1]) * MSUN_S)).cuda()
    out = torch.zeros((len(p), n // 2 + 1), dtype=torch.complex128, device="cuda")
    amp = torch.where(f[None] <= isco[:, None], f ** (-7.0 / 6.0), 0.0)
    band = torch.view_as_real(out)[:, lo:hi + 1]
    torch.mul(amp, torch.cos(psi), out=band[..., 0])
    torch.mul(amp, -torch.sin(psi), out=band[..., 1])
    return out


def _masses(mc, eta):
    m = mc * eta ** -0.6
    d = np.sqrt(np.maximum(0.0, 1.0 - 4.0 * eta))
    return m * (1.0 + d) / 2.0, m * (1.0 - d) / 2.0


def _templates_around(rng, mc, count, spread):
    """Parameters of `count` templates near an equal-mass, circular reference of chirp mass mc."""
    m1, m2 = _masses(mc * (1.0 + rng.uniform(-spread, spread, count)), rng.uniform(0.235, 0.25, count))
    return np.stack([m1, m2, rng.uniform(-0.02, 0.02, count), rng.uniform(0.0, 0.05, count),
                     rng.uniform(0.0, 500.0, count)], axis=1)


class _Inputs:
    """Host parameters of a case (drawn from the seed alone) and the waveforms made from them on the GPU."""

    def __init__(self, case, seed):
        self.case, self.n = case, case["n"]
        rng = np.random.default_rng([seed, 26011])
        refs = case.get("refs", 1)
        self.mc = np.geomspace(1.0, 1.6, refs) * rng.uniform(1.0, 1.02)
        per = case.get("per_ref", case.get("templates", 0))
        self.counts, self.taps = [per] * refs, [case.get("taps", 0)] * refs
        if case.get("uneven"):
            self.counts = [max(1, int(per * rng.uniform(0.25, 1.75))) for _ in range(refs)]
            self.taps = [int(rng.integers(min(32, t), t + 1)) for t in self.taps]
        # a bank of thousands covers a wider strip of chirp mass around its reference
        self.params = [_templates_around(rng, mc, c, 1e-3 if c < 400 else 1e-2)
                       for mc, c in zip(self.mc, self.counts)]
        m1, m2 = _masses(self.mc, np.full(refs, 0.25))
        self.refs = np.stack([m1, m2, np.zeros(refs), np.zeros(refs), np.full(refs, 250.0)], axis=1)
        self.inject = (int(rng.integers(refs)), rng.uniform(0.3, 0.7))
        self.rng = rng
        self.psd = _psd(self.n)
        lo, hi = _band(case)
        self.w = np.zeros(self.n // 2 + 1)
        self.w[lo:hi + 1] = 4.0 * (FS / self.n) / self.psd[lo:hi + 1]

    def noise(self):
        """Spectrum on the rfft grid of one stretch of detector noise."""
        lo, hi = _band(self.case)
        g = self.rng.standard_normal((hi - lo + 1, 2))
        s = np.zeros(self.n // 2 + 1, dtype=np.complex128)
        s[lo:hi + 1] = np.sqrt(self.psd[lo:hi + 1] / (4.0 * FS / self.n)) * (g[:, 0] + 1j * g[:, 1])
        return torch.from_numpy(s).cuda()

    def signal(self, at, snr=12.0):
        """Spectrum of one template of the case with optimal SNR `snr`, ending at sample `at`."""
        r = self.inject[0]
        h = _waveforms(self.case, self.params[r][:1] if len(self.params[r]) else self.refs[r:r + 1])[0]
        amp = snr / torch.sqrt((torch.from_numpy(self.w).cuda() * h.abs() ** 2).sum())
        k = torch.arange(self.n // 2 + 1, device="cuda")
        turn = ((k * at) % self.n).double() * (-2.0 * math.pi / self.n)
        return amp * h * torch.polar(torch.ones_like(turn), turn)

    def series(self, spectrum):
        return (torch.fft.irfft(spectrum, self.n) * FS).contiguous()

    def segment(self):
        """float64 [N] on the GPU: noise and one signal."""
        return self.series(self.noise() + self.signal(int(self.inject[1] * self.n)))

    def batches(self, r, size=256):
        for a in range(0, self.counts[r], size):
            yield a, _waveforms(self.case, self.params[r][a:a + size])


class _State:
    """What a program keeps between calls; library objects go back in the order that their users allow."""

    def __del__(self):
        for name, close in (("graph", rfd.rfd_graph_destroy), ("stream", rfd.rfd_stream_destroy),
                            ("sur", rfd.rfd_surrogate_destroy)):
            if getattr(self, name, None) is not None:
                close(getattr(self, name))
        if getattr(self, "search", None) is not None:
            self.search.close()
        if getattr(self, "plan", None) is not None:
            rfd.rfd_plan_destroy(self.plan)


def _window(case):
    return 2048


def _threshold(case):
    return {"taps": 6.0, "stream": 5.5, "chisq": 5.5, "findchirp": 6.0}.get(case["kind"], 6.0)


def _search(x, with_taps=True):
    search = RatioFilterSearch(x.psd, x.case["f_low"], FS, x.n,
                               [SubBankSpec(r, t, -(t // 2), c) for r, (t, c) in enumerate(zip(x.taps, x.counts))])
    for r, h in enumerate(_waveforms(x.case, x.refs)):
        search.h_ref[r] = h.clone()
    if with_taps:
        for r in range(len(x.counts)):
            for a, h in x.batches(r):
                search.make_taps(r, h, first=a, ridge_eps=RIDGE)
    return search


CAPACITY = 1 << 14


def _trigger_buffer():
    """A trigger buffer on the GPU and its fields as tensors; entries past the last trigger stay zero."""
    buf = torch.zeros(CAPACITY * 32, dtype=torch.uint8, device="cuda")
    i32, f32 = buf.view(torch.int32).view(-1, 8), buf.view(torch.float32).view(-1, 8)
    return buf, dict(sample=buf.view(torch.int64).view(-1, 4)[:, 0], tmpl=i32[:, 2], subbank=i32[:, 3], rho=f32[:, 4],
                     z_re=f32[:, 5], z_im=f32[:, 6])


def prepare(case, seed):
    x = _Inputs(case, seed)
    s = _State()
    s.case, kind = case, case["kind"]
    s.out, s.fields = _trigger_buffer()
    if kind == "bank":
        s.search = _search(x)
        s.search.set_segment(x.segment())
        s.graph = None
        if case["graph"]:
            s.graph = rfd.rfd_segment_graph_create(s.search.plan, s.search.taps, case["form"], _threshold(case),
                                                   _window(case), s.search.data, s.search.h_ref, s.out, CAPACITY)
    elif kind == "dechirp":
        x.taps, x.counts = [16] * case["refs"], [0] * case["refs"]
        s.search = _search(x, with_taps=False)
        s.search.set_segment(x.segment())
        rfd.rfd_plan_set_dechirp_fp64(s.search.plan, case["fp64"])
        s.z = torch.empty((case["refs"], x.n), dtype=torch.complex64, device="cuda")
    elif kind == "stream":
        s.search = _search(x)
        # one signal ends just before the stream starts, a second one in the data that is pushed
        d, k = case["increment"], case["pushes"]
        first = x.noise() + x.signal(x.n - 128)
        s.search.set_segment(x.series(first))
        s.stream = rfd.rfd_stream_create(s.search.plan, s.search.taps, s.search.h_ref, d)
        s.pushed = x.series(first + x.signal(d * k // 3)).reshape(-1, d)[:k].clone()
        s.outs = [_trigger_buffer() for _ in range(k)]
    elif kind == "taps":
        s.search = _search(x, with_taps=False)
        s.search.set_segment(x.segment())
        s.search.dechirp_all()
        s.h = _waveforms(case, x.params[0])
        s.method = ((rfd.RFD_TAPS_WINDOW if case["window"] else rfd.RFD_TAPS_LS)
                    | (rfd.RFD_TAPS_CENTRE if case["centre"] else 0))
    elif kind == "findchirp":
        s.plan = rfd.rfd_plan_create(x.psd, case["f_low"], FS, x.n)
        s.data = x.segment()
        info = rfd.rfd_plan_info_get(s.plan)
        s.filt = torch.empty((case["templates"], info["n_band"]), dtype=torch.complex64, device="cuda")
        for a, h in x.batches(0):
            rfd.rfd_findchirp_prepare(s.plan, h, filt=s.filt[a:a + len(h)])
    elif kind == "chisq":
        s.search = _search(x)
        for r in range(case["refs"]):
            rfd.rfd_taps_band_fractions(s.search.plan, s.search.taps, r, s.search.h_ref[r], case["bands"])
        s.search.set_segment(x.segment())
    elif kind == "surrogate":
        x.counts, x.params = [case["basis"]], [_templates_around(x.rng, x.mc[0], case["basis"], 1e-3)]
        s.search = _search(x)
        s.sur = rfd.rfd_surrogate_create(s.search.plan, s.search.taps, 0, case["basis"], case["hidden"], 2601)
        p = _network(case, seed)
        basis = np.linalg.qr(x.rng.standard_normal((2 * case["taps"], case["basis"])))[0].T
        rfd.rfd_surrogate_set_state(s.sur, p["flat"], basis)
        s.x, s.c = torch.from_numpy(p["x"]).cuda(), torch.from_numpy(p["c"]).cuda()
    return s


def _network(case, seed):
    """Weights (float32, the library's order), scaled inputs and target coefficients of a trained network's size."""
    rng = np.random.default_rng([seed, 77])
    h, k = case["hidden"], case["basis"]
    sizes = [(h, 4), (h,), (h, h), (h,), (k, h), (k,)]
    parts = [(rng.uniform(-1, 1, q) * math.sqrt((6.0 if len(q) > 1 else 0.1) / q[-1])).astype(np.float32)
             for q in sizes]
    c = rng.standard_normal((case["rows"], k)) / np.arange(1, k + 1)
    c /= np.linalg.norm(c, axis=1, keepdims=True)
    return dict(parts=parts, flat=np.concatenate([q.ravel() for q in parts]), c=c.astype(np.float32),
                x=rng.uniform(-1, 1, (case["rows"], 4)).astype(np.float32))


# -------------------------------------------------------------------- run
def run(s):
    case, kind = s.case, s.case["kind"]
    thr, win = _threshold(case), _window(case)
    if kind == "bank":
        if s.graph is not None:
            n = rfd.rfd_segment_graph_launch(s.graph)
        else:
            s.search.dechirp_all()
            _, n = s.search.filter(case["form"], thr, win, CAPACITY, s.out)
        return dict(s.fields, n=n)
    if kind == "dechirp":
        sigma = rfd.rfd_dechirp_refs(s.search.plan, s.search.data, s.search.h_ref)
        for r in range(case["refs"]):
            rfd.rfd_get_zref(s.search.plan, r, s.z[r])
        return dict(z=s.z, sigma=np.array([sigma[r] for r in range(case["refs"])]))
    if kind == "stream":
        rfd.rfd_stream_prime(s.stream, s.search.data)
        got = []
        for data, (out, fields) in zip(s.pushed, s.outs):
            _, n, start = rfd.rfd_stream_push(s.stream, data, "ols32", thr, win, CAPACITY, out)
            got.append(dict(fields, n=n, start=start))
        return got
    if kind == "taps":
        s.search.make_taps(0, s.h, method=s.method, ridge_eps=RIDGE)
        _, n = s.search.filter("ols32", thr, win, CAPACITY, s.out)
        return dict(s.fields, n=n)
    if kind == "findchirp":
        _, n = rfd.findchirp_filter(s.plan, s.data, s.filt, thr, win, CAPACITY, s.out)
        return dict(s.fields, n=n)
    if kind == "chisq":
        s.search.dechirp_all()
        _, n = s.search.filter("ols32", thr, win, CAPACITY, s.out)
        edges = [rfd.rfd_dechirp_bands(s.search.plan, h, r, case["bands"]) for r, h in s.search.h_ref.items()]
        chisq = np.zeros(CAPACITY, dtype=np.float32)
        chisq[:n] = s.search.chisq(s.out, n)
        return dict(s.fields, n=n, chisq=chisq, edges=np.stack(edges))
    loss, grad = rfd.rfd_surrogate_loss_grad(s.sur, s.x, s.c)
    return dict(loss=loss, grad=grad)


# ------------------------------------------------------------------- work
def work(case):
    n, kind = case["n"], case["kind"]
    lo, hi = _band(case)
    m = hi - lo + 1
    lg = math.log2(n)
    refs = case.get("refs", 1)
    count = refs * case.get("per_ref", case.get("templates", 0))
    taps = case.get("taps", 0)

    def filter_flops(outputs, t):
        # FFT blocks of the best power of two, product and squared modulus included; or the direct sum where less
        best = min((5.0 * k + 14.0) * 2 ** k / (2 ** k - t + 1) for k in range(6, 16) if 2 ** k > t)
        return count * outputs * min(best, 8.0 * t + 4.0)

    t_mid = taps if not case.get("uneven") else (taps + 32) // 2
    segment = 8 * n + refs * 16 * m                     # data and reference spectra
    transforms = (1 + refs) * 5.0 * n * lg
    if kind == "bank":
        return dict(bytes=segment + 8 * count * t_mid, flops=transforms + filter_flops(n, t_mid))
    if kind == "dechirp":
        return dict(bytes=segment + refs * 16 * n, flops=transforms)        # the series, and their copies out
    if kind == "stream":
        d = case["increment"]
        k = case["pushes"]
        return dict(bytes=segment + refs * 8 * n + k * (8 * d + refs * 16 * m + 8 * count * taps),
                    flops=transforms + k * (5.0 * n * lg + refs * (8.0 * m + 5.0 * n * lg) + filter_flops(d, taps)))
    if kind == "taps":
        solve = 0 if case["window"] else 16.0 * taps ** 2
        return dict(bytes=count * (16 * m + 16 * taps) + 16 * m + 8 * n,
                    flops=count * (5.0 * n * lg + solve + 20.0 * taps * math.log2(2 * taps)) + filter_flops(n, taps))
    if kind == "findchirp":
        return dict(bytes=8 * n + count * 8 * m, flops=(count + 1) * 5.0 * n * lg + count * 9.0 * n)
    if kind == "chisq":
        return dict(bytes=segment + refs * 16 * m + 8 * count * taps,
                    flops=transforms + refs * case["bands"] * 5.0 * n * lg + filter_flops(n, taps))
    h, k, rows = case["hidden"], case["basis"], case["rows"]
    weights = 4 * h + h * h + h * k
    return dict(bytes=8 * weights + 4 * rows * (4 + k), flops=6.0 * rows * weights)


# ------------------------------------------------------------------ exact
def exact(case, seed):
    x = _Inputs(case, seed)
    if case["kind"] == "surrogate":
        return _exact_gradient(case, seed)
    if case["kind"] == "stream":
        return None             # rings of several pushes; the same series and filters as the other cases
    dev = torch.device("cuda")
    w = torch.from_numpy(x.w).to(dev)
    n = x.n

    def series(q):              # sum_i q_i e^{2 pi i i n / N} over the one-sided bins
        return torch.fft.ifft(q, n=n, dim=-1) * n

    data = x.segment()
    s = torch.fft.rfft(data) / FS
    if case["kind"] == "findchirp":
        found = []
        for a, h in x.batches(0, 32):
            sig = torch.sqrt((w * h.abs() ** 2).sum(1))
            z = series(w * s * h.conj()) / sig[:, None]
            found.append(_peaks(case, z))
        return _exact_triggers(found)
    href = _waveforms(case, x.refs)
    sigma = torch.sqrt((w * href.abs() ** 2).sum(1))
    if case["kind"] == "dechirp":
        return dict(z=torch.stack([series(w * s * h.conj()) / g for h, g in zip(href, sigma)]), sigma=sigma)
    found, chis = [], []
    for r in range(len(x.counts)):
        t = x.taps[r]
        k0 = -(t // 2)
        u = w * href[r].abs() ** 2
        g = series(u)[:t]
        idx = torch.arange(t, device=dev)
        d = idx[:, None] - idx[None]
        gram = torch.where(d >= 0, g[d.abs()], g[d.abs()].conj())
        zf = torch.fft.fft(series(w * s * href[r].conj()) / sigma[r])
        if case["kind"] == "chisq":
            edges = _exact_edges(x, u, case["bands"])
            zb = torch.stack([series(_only(w * s * href[r].conj(), edges, b)) / sigma[r]
                              for b in range(case["bands"])])
            gb = torch.stack([series(_only(u.to(torch.complex128), edges, b))[:t] for b in range(case["bands"])])
        for a, h in x.batches(r, 32):
            if case.get("window"):
                v = w * h * href[r].conj()
                ratio = torch.where(u > 0, h * href[r].conj() / href[r].abs().clamp_min(1e-300) ** 2, 0.0)
                rhs = series(ratio) / n
            else:
                rhs = v = series(w * h * href[r].conj())
            lag = torch.full((len(h),), k0, device=dev)
            if case.get("centre"):
                full = series(v) if case.get("window") else rhs
                peak = full.abs().argmax(1)
                lag = torch.where(peak > n // 2, peak - n, peak) - t // 2
            b = torch.gather(rhs, 1, (lag[:, None] + idx) % n)
            if case.get("window"):
                taps = b * _tukey(t).to(dev)
            else:
                m = (gram + RIDGE * g[0].real * torch.eye(t, device=dev)).cpu()
                taps = torch.linalg.solve(m, b.cpu().T).T.contiguous().to(dev)
            fit = torch.sqrt((taps.conj() * (taps @ gram.T)).sum(1).real)
            c = taps.conj() * (sigma[r] / fit)[:, None]
            kernel = torch.zeros((len(h), n), dtype=torch.complex128, device=dev)
            kernel[:, (k0 + idx) % n] = c                # on the filter index m = n + lag - k0
            z = torch.fft.ifft(zf * torch.fft.ifft(kernel, dim=1) * n, dim=1)
            peaks = _peaks(case, z)
            found.append(peaks)
            if case["kind"] == "chisq":
                toep = torch.where(d >= 0, gb[:, d.abs()], gb[:, d.abs()].conj())
                num = torch.stack([(taps.conj() * (taps @ q.T)).sum(1) for q in toep]).real
                f = num / num.sum(0)
                for j, at in zip(peaks[0].tolist(), peaks[1].tolist()):
                    zj = (zb[:, (at + k0 + idx) % n] * c[j]).sum(1)
                    chis.append(((zj - f[:, j] * zj.sum()).abs() ** 2 / f[:, j]).sum())
    got = _exact_triggers(found)
    if case["kind"] == "chisq":
        got.update(chisq=_padded(torch.stack(chis) if chis else torch.zeros(0, dtype=torch.float64)), edges=None)
    return got


def _only(q, edges, b):
    out = torch.zeros_like(q)
    out[edges[b]:edges[b + 1]] = q[edges[b]:edges[b + 1]]
    return out


def _exact_edges(x, u, bands):
    lo, hi = _band(x.case)
    prefix = np.concatenate([[0.0], np.cumsum(u.cpu().numpy()[lo:hi + 1])])
    inner = [lo + int(np.searchsorted(prefix, prefix[-1] * b / bands)) for b in range(1, bands)]
    return [lo] + inner + [hi + 1]


def _tukey(t):
    y = torch.arange(t, dtype=torch.float64) / max(1, t - 1)
    edge = torch.minimum(y, 1.0 - y) / 0.125
    return torch.where(edge < 1.0, 0.5 * (1.0 - torch.cos(math.pi * edge)), 1.0) if t > 1 else torch.ones(1)


def _peaks(case, z):
    """(row, index, z) of the largest |z| of each window where it exceeds the threshold."""
    win = _window(case)
    rho = z.abs().reshape(z.shape[0], -1, win)
    top, at = rho.max(2)
    row, q = torch.nonzero(top > _threshold(case), as_tuple=True)
    m = q * win + at[row, q]
    return row, m, z[row, m]


def _padded(v):
    return torch.nn.functional.pad(v, (0, CAPACITY - v.numel()))


def _exact_triggers(found):
    z = torch.cat([f[2] for f in found])
    return dict(sample=None, tmpl=None, subbank=None, n=None, rho=_padded(z.abs()), z_re=_padded(z.real),
                z_im=_padded(z.imag))


def _exact_gradient(case, seed):
    p = _network(case, seed)
    wts = []
    for k, q in enumerate(p["parts"]):      # the forward pass reads the weight matrices rounded to bfloat16
        v = torch.from_numpy(q)
        v = v.bfloat16().double() if v.dim() > 1 else v.double()
        wts.append(v.requires_grad_(True))
    x, c = torch.from_numpy(p["x"]).double(), torch.from_numpy(p["c"]).double()
    h1 = torch.nn.functional.silu(x @ wts[0].T + wts[1])
    h2 = torch.nn.functional.silu(h1 @ wts[2].T + wts[3])
    loss = ((h2 @ wts[4].T + wts[5] - c) ** 2).sum() / case["rows"]
    loss.backward()
    return dict(loss=loss.detach(), grad=torch.cat([q.grad.reshape(-1) for q in wts]))
