"""Timed cases of the SPIIR library: the calls that a search program makes.

Banks are random first-order complex IIR filter banks of the shapes that the
benchmark, the tests and the workload generators use (radii, frequencies,
delays and gains drawn the same way), strain is unit white noise, raw strain is
noise through a resonant low-pass, and the trigger series is chi-square noise
with bumps. Streaming objects are warmed with enough strain in prepare() that
every filter of the bank sees input, as in the middle of a stream.

Kinds:
  rows       SpiirBank.filter_block: the SNR rows of the next block
  z          SpiirBank.filter_block_z: the complex template sums of the next block
  multirate  SpiirMultiRate.filter_block_z: the full-rate sums of a multi-rate bank
  adjoint    SpiirBank.forward_z with its tape, then SpiirBank.backward
  whiten     Whitener.process of the next block (train > 0: the PSD is estimated first)
  cluster    TriggerClusterer.run
  pipeline   raw strain: Whitener.process, SpiirBank.trigger_max, TriggerStream.push_into
"""
import math

import numpy as np
import torch

FS = 4096.0


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    wide = dict(r_lo=0.99, r_hi=1.0 - 1e-5)
    return [
        # an eighth of a second of one detector through a handful of templates: latency
        dict(name="rows_4x128_512", kind="rows", T=4, k_lo=128, k_hi=128, r_lo=0.99, r_hi=0.9999,
             dmax=2047, n=512, max_block=16384),
        # the same bank over four seconds at once
        dict(name="rows_4x128_16384", kind="rows", T=4, k_lo=128, k_hi=128, r_lo=0.99, r_hi=0.9999,
             dmax=2047, n=16384, max_block=16384),
        # the search bank, one second per call: every template's SNR
        dict(name="rows_1024_4096", kind="rows", T=1024, k_lo=100, k_hi=800, dmax=16384, n=4096,
             max_block=4096, **wide),
        # one stream's bank of the batched search, a ragged call
        dict(name="rows_256_3001", kind="rows", T=256, k_lo=200, k_hi=600, dmax=16384, n=3001,
             max_block=4096, **wide),
        # offline run of long filters (poles next to the unit circle), long calls
        dict(name="z_64x1000_65536", kind="z", T=64, k_lo=1000, k_hi=1000, r_lo=1.0 - 1e-4, r_hi=1.0 - 1e-6,
             dmax=2047, n=65536, max_block=16384),
        # the multi-rate chirp bank, one second per call
        dict(name="multirate_1024_4096", kind="multirate", T=1024, k_lo=100, k_hi=800, levels=5, dmax=2047,
             n=4096),
        # a fit step of the whole chirp-fit bank: template sums and coefficient gradients
        dict(name="adjoint_256x400", kind="adjoint", T=256, k=400, chirp=True, n=65536),
        # gradients of a small random bank over a short stretch of strain
        dict(name="adjoint_32x100", kind="adjoint", T=32, k=100, chirp=False, n=4001),
        # one second of raw strain per call; about a minute at once, after re-estimating the PSD on 32 seconds
        dict(name="whiten_4096", kind="whiten", frame=4096, train=0, n=4096),
        dict(name="whiten_train_262144", kind="whiten", frame=4096, train=131072, n=262144),
        # clustering of a stored series of 17 minutes
        dict(name="cluster_4194304", kind="cluster", n=4194304, window=4096, quantile=0.9999),
        # the whole chain on raw strain, one second per call
        dict(name="pipeline_1024_4096", kind="pipeline", T=1024, k_lo=100, k_hi=800, dmax=16384, n=4096,
             frame=4096, window=1024, **wide),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rows", "rows", "z", "multirate", "adjoint", "whiten", "cluster"])
    if kind in ("rows", "z"):
        T = _log_int(rng, 1, 1024)
        k_lo = _log_int(rng, 1, 500)
        k_hi = min(1000, k_lo + rng.randrange(0, 301))
        most = min(32768, int(4.0e9 / (T * 0.5 * (k_lo + k_hi))), int(3.0e7 / T))
        n = max(64, min(most, _log_int(rng, 100, 32768)))
        return dict(kind=kind, T=T, k_lo=k_lo, k_hi=k_hi, r_lo=rng.choice([0.98, 0.99, 1.0 - 1e-4]),
                    r_hi=rng.choice([0.9999, 1.0 - 1e-5, 1.0 - 1e-6]), dmax=_log_int(rng, 1, 16384), n=n,
                    max_block=rng.choice([4096, 16384]))
    if kind == "multirate":
        levels = rng.randrange(2, 6)
        n = (1 << (levels - 1)) * _log_int(rng, 32, 8192 >> (levels - 1))
        k_lo = _log_int(rng, 20, 300)
        return dict(kind=kind, T=_log_int(rng, 16, 1024), k_lo=k_lo, k_hi=k_lo + rng.randrange(0, 301),
                    levels=levels, dmax=_log_int(rng, 64, 2047), n=n)
    if kind == "adjoint":
        return dict(kind=kind, T=_log_int(rng, 2, 128), k=_log_int(rng, 8, 300), chirp=False,
                    n=_log_int(rng, 500, 9000))
    if kind == "whiten":
        frame = 1 << rng.randrange(8, 14)
        n = (frame // 2) * _log_int(rng, 1, max(2, 524288 // frame))
        train = rng.choice([0, 0, frame * rng.randrange(4, 33) + rng.randrange(0, frame)])
        return dict(kind=kind, frame=frame, train=train, n=n)
    return dict(kind=kind, n=_log_int(rng, 2000, 4194304), window=_log_int(rng, 16, 8192),
                quantile=rng.choice([0.99, 0.999, 0.9999]))


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------

class Bank:
    """Filters of template j: offsets[j]:offsets[j+1] of a, b, d."""

    def __init__(self, offsets, a, b, d, dmax):
        self.offsets = np.ascontiguousarray(offsets, np.int64)
        self.a = np.ascontiguousarray(a, np.complex128)
        self.b = np.ascontiguousarray(b, np.complex128)
        self.d = np.ascontiguousarray(d, np.int32)
        self.dmax = int(dmax)

    @property
    def n_templates(self):
        return len(self.offsets) - 1

    @property
    def n_filters(self):
        return int(self.offsets[-1])


def _offsets(k):
    return np.concatenate([[0], np.cumsum(k)]).astype(np.int64)


def _random_bank(rng, k, r_lo, r_hi, dmax):
    """|a| and arg a uniform, b circular complex normal / sqrt(K), delays uniform."""
    F = int(k.sum())
    r = rng.uniform(r_lo, r_hi, F) if r_hi > r_lo else np.full(F, min(r_lo, r_hi))
    a = r * np.exp(1j * rng.uniform(0.001 * math.pi, 0.5 * math.pi, F))
    b = (rng.standard_normal(F) + 1j * rng.standard_normal(F)) * np.repeat(np.sqrt(0.5 / np.maximum(k, 1)), k)
    return Bank(_offsets(k), a, b, rng.integers(0, dmax + 1, F), dmax)


def _bank_of(case, rng):
    k = rng.integers(case["k_lo"], case["k_hi"] + 1, case["T"])
    return _random_bank(rng, k, case["r_lo"], case["r_hi"], case["dmax"])


def _multirate_banks(case, rng):
    """Filter frequencies with p(f) ~ f^(-11/3) on 20 - 1,024 Hz, each filter on the
    lowest rate FS / 2^r (r < levels) that keeps f below a quarter of the rate."""
    T, levels = case["T"], case["levels"]
    k = rng.integers(case["k_lo"], case["k_hi"] + 1, T)
    F = int(k.sum())
    tpl = np.repeat(np.arange(T), k)
    e = -8.0 / 3.0
    lo, hi = 20.0 ** e, 1024.0 ** e
    f = (lo - rng.random(F) * (lo - hi)) ** (1.0 / e)
    lev = np.zeros(F, np.int64)
    for r in range(1, levels):
        lev[f < FS / 2.0 ** (r + 2)] = r
    om = 2.0 * math.pi * f * 2.0 ** lev / FS
    a = rng.uniform(0.98, 0.999, F) * np.exp(1j * om)
    b = (rng.standard_normal(F) + 1j * rng.standard_normal(F)) * np.repeat(np.sqrt(0.5 / k), k)
    u = rng.random(F)
    banks = []
    for r in range(levels):
        s = lev == r
        dm = case["dmax"] >> r
        banks.append(Bank(_offsets(np.bincount(tpl[s], minlength=T)), a[s], b[s],
                          np.floor(u[s] * (dm + 1)).astype(np.int32), dm))
    return banks


def _taps(n=24):
    """Halving taps h (sum 1) and doubling taps g (each polyphase half sums to 1)."""
    i = np.arange(n)
    base = 0.5 * np.sinc(0.5 * (i - (n - 1) / 2.0)) * (0.5 - 0.5 * np.cos(2.0 * np.pi * (i + 1) / (n + 1)))
    g = np.empty(n)
    g[0::2] = base[0::2] / base[0::2].sum()
    g[1::2] = base[1::2] / base[1::2].sum()
    return base / base.sum(), g


def _chirp_bank(case, rng):
    """k filters per template at equal steps along a time-reversed leading-order
    chirp: delay = start of the step, rotation and gain of the chirp there, decay
    over about one step (the starting point of a chirp fit)."""
    T, k, n = case["T"], case["k"], case["n"]
    a, b, d = (np.empty(T * k, t) for t in (np.complex128, np.complex128, np.int32))
    for j, mc in enumerate(rng.uniform(1.0, 30.0, T)):
        m = mc * 4.925491025543576e-06
        tau0 = (5.0 / 256.0) * (math.pi * 1000.0) ** (-8.0 / 3.0) * m ** (-5.0 / 3.0)
        tau = tau0 + np.arange(n) / FS
        f = (5.0 / (256.0 * tau)) ** 0.375 * m ** -0.625 / math.pi
        size = max(k, int(np.count_nonzero(f >= 30.0)))
        at = np.floor(np.linspace(0, min(size, n), k + 1)[:-1]).astype(np.int64)
        ph = 2.0 * (tau / (5.0 * m)) ** 0.625
        w = np.minimum(ph[np.minimum(at + 1, n - 1)] - ph[at], 0.5 * math.pi)
        s = slice(j * k, (j + 1) * k)
        a[s] = min(math.exp(-k / float(min(size, n))), 1.0 - 1e-6) * np.exp(1j * w)
        b[s] = f[at] ** (2.0 / 3.0) * np.exp(1j * ph[at])
        d[s] = at
    return Bank(np.arange(T + 1) * k, a, b, d, n - 1)


def _raw_strain(rng, n):
    """White noise through 1 / (1 - 1.8 z^-1 + 0.85 z^-2) plus a white floor."""
    m = 1 << int(n + 512 - 1).bit_length()
    w = np.exp(-2j * np.pi * np.arange(m // 2 + 1) / m)
    x = np.fft.irfft(np.fft.rfft(rng.standard_normal(m)) / (1.0 - 1.8 * w + 0.85 * w * w), m)
    return (x[:n] + 0.1 * rng.standard_normal(n)).astype(np.float32)


def _psd_model(frame):
    """PSD of _raw_strain at the frame's frequencies 0 .. frame / 2."""
    w = np.exp(-2j * np.pi * np.arange(frame // 2 + 1) / frame)
    return 1.0 / np.abs(1.0 - 1.8 * w + 0.85 * w * w) ** 2 + 0.01


def _warm(case):
    """Samples fed before the timed block: every delay filled, and some memory."""
    n = case["dmax"] + 4096
    return (n + 4095) // 4096 * 4096


def _inputs(case, seed):
    rng = np.random.default_rng([1602, 77, seed])
    kind = case["kind"]
    if kind in ("rows", "z"):
        bank = _bank_of(case, rng)
        return bank, rng.standard_normal(_warm(case) + case["n"]).astype(np.float32)
    if kind == "multirate":
        banks = _multirate_banks(case, rng)
        return banks, rng.standard_normal(2 * case["n"]).astype(np.float32)
    if kind == "adjoint":
        n, T = case["n"], case["T"]
        if case["chirp"]:
            bank = _chirp_bank(case, rng)
            x = np.zeros(n, np.float32)
            x[0] = 1.0
        else:
            bank = _random_bank(rng, np.full(T, case["k"]), 0.99, 0.9999, 1000)
            x = rng.standard_normal(n).astype(np.float32)
        g = rng.standard_normal((T, 2 * n), dtype=np.float32) / math.sqrt(n)
        return bank, x, g.view(np.complex64)
    if kind == "whiten":
        warm = case["frame"]
        return _raw_strain(rng, max(case["train"], 1)), _raw_strain(rng, warm + case["n"])
    if kind == "pipeline":
        bank = _bank_of(case, rng)
        return bank, _raw_strain(rng, 32 * 4096), _raw_strain(rng, _warm(case) + case["n"])
    raise ValueError(kind)


# ---------------------------------------------------------------------------
# what a program has in hand, and one pass
# ---------------------------------------------------------------------------

def _cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def prepare(case, seed):
    import paper_1602_05573_amd as lib
    kind = case["kind"]
    if kind == "cluster":
        return _prepare_cluster(case, seed, lib)
    if kind in ("rows", "z"):
        bank, x = _inputs(case, seed)
        bk = lib.SpiirBank(bank.offsets, bank.a, bank.b, bank.d, max_delay=bank.dmax, max_block=case["max_block"])
        w = _warm(case)
        xd = _cuda(x)
        out = torch.empty((case["T"], case["n"]), device="cuda",
                          dtype=torch.float32 if kind == "rows" else torch.complex64)
        for i in range(0, w, 4096):
            bk.trigger_max(xd[i:i + 4096])
        return dict(case=case, bank=bk, x=xd[w:].contiguous(), out=out)
    if kind == "multirate":
        banks, x = _inputs(case, seed)
        h, g = _taps()
        n = case["n"]
        mr = lib.SpiirMultiRate(banks, h, g, max_block=n)
        xd = _cuda(x)
        out = torch.empty((case["T"], n), device="cuda", dtype=torch.complex64)
        mr.filter_block_z(xd[:n].contiguous(), out)
        return dict(case=case, bank=mr, x=xd[n:].contiguous(), out=out)
    if kind == "adjoint":
        bank, x, g = _inputs(case, seed)
        bk = lib.SpiirBank(bank.offsets, bank.a, bank.b, bank.d, max_delay=bank.dmax)
        return dict(case=case, bank=bk, x=_cuda(x), g=_cuda(g))
    if kind == "whiten":
        train, x = _inputs(case, seed)
        wh = lib.Whitener(case["frame"])
        wh.set_psd(_psd_model(case["frame"]))
        w = len(x) - case["n"]
        wh.process(_cuda(x[:w]))
        return dict(case=case, wh=wh, train=_cuda(train), x=_cuda(x[w:]),
                    out=torch.empty(case["n"], device="cuda", dtype=torch.float32))
    bank, train, x = _inputs(case, seed)
    n, w = case["n"], len(x) - case["n"]
    bk = lib.SpiirBank(bank.offsets, bank.a, bank.b, bank.d, max_delay=bank.dmax, max_block=n)
    wh = lib.Whitener(case["frame"])
    wh.estimate_psd(_cuda(train))
    xd = _cuda(x)
    for i in range(0, w, 4096):
        mx, _ = bk.trigger_max(wh.process(xd[i:i + 4096]))
    ts = lib.TriggerStream(float(torch.quantile(mx, 0.99)), case["window"], n)
    triggers = [torch.zeros(c, device="cuda", dtype=t) for c, t in
                ((ts.capacity, torch.int64), (ts.capacity, torch.int32), (ts.capacity, torch.float32),
                 (1, torch.int64))]
    return dict(case=case, bank=bk, wh=wh, ts=ts, triggers=triggers, x=xd[w:].contiguous())


def _prepare_cluster(case, seed, lib):
    n = case["n"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    mx = -2.0 * torch.log(torch.rand(n, device="cuda", generator=gen).clamp_min(1e-12))
    am = torch.randint(0, 1024, (n,), device="cuda", generator=gen, dtype=torch.int32)
    rng = np.random.default_rng([1602, 78, seed])
    for c, h, w in zip(rng.integers(0, n, 64), rng.uniform(10.0, 100.0, 64), rng.integers(1, 200, 64)):
        lo, hi = max(0, int(c - 3 * w)), min(n, int(c + 3 * w + 1))
        t = torch.arange(lo, hi, device="cuda") - int(c)
        mx[lo:hi] = torch.maximum(mx[lo:hi], h * torch.exp(-0.5 * (t / float(w)) ** 2).float())
    at = torch.sort(mx).values[min(n - 1, int(case["quantile"] * n))]
    cl = lib.TriggerClusterer(n, n // (case["window"] + 1) + 1)
    for t in (cl.index, cl.template, cl.snr):
        t.zero_()
    return dict(case=case, cl=cl, mx=mx, am=am, threshold=float(at))


def run(state):
    kind = state["case"]["kind"]
    if kind == "rows":
        return state["bank"].filter_block(state["x"], snr=state["out"])
    if kind in ("z", "multirate"):
        return state["bank"].filter_block_z(state["x"], state["out"])
    if kind == "adjoint":
        z, tape = state["bank"].forward_z(state["x"], want_tape=True)
        ga, gb = state["bank"].backward(tape, state["g"])
        tape.close()
        return dict(z=z, grad_a=ga, grad_b=gb)
    if kind == "whiten":
        if state["case"]["train"]:
            state["wh"].estimate_psd(state["train"])
        return state["wh"].process(state["x"], out=state["out"])
    if kind == "cluster":
        c = state["case"]
        cl = state["cl"]
        cl.run(state["mx"], state["am"], state["threshold"], c["window"])
        return dict(index=cl.index, template=cl.template, snr=cl.snr, total=cl.count)
    white = state["wh"].process(state["x"])
    mx, am = state["bank"].trigger_max(white)
    state["ts"].push_into(mx, am, *state["triggers"])
    index, template, snr, total = state["triggers"]
    return dict(white=white, max=mx, index=index, template=template, snr=snr, total=total)


# ---------------------------------------------------------------------------
# the least that a pass has to do
# ---------------------------------------------------------------------------

def _filters(case):
    if case["kind"] == "adjoint":
        return case["T"] * case["k"]
    return case["T"] * 0.5 * (case["k_lo"] + case["k_hi"])


def work(case):
    kind, n = case["kind"], case["n"]
    if kind in ("rows", "z", "pipeline"):
        F, T = _filters(case), case["T"]
        # a*y 6, b*x 2, the sums 4 FLOP per filter and sample; |z|^2 3 per template and sample.
        # Coefficients (a, b complex64, delay) and state (complex64 in and out) per filter
        out = {"rows": 4.0 * T * n, "z": 8.0 * T * n, "pipeline": 12.0 * n}[kind]
        flops = 12.0 * F * n + 3.0 * T * n
        if kind == "pipeline":
            flops += (n / (case["frame"] / 2)) * 10.0 * case["frame"] * math.log2(case["frame"])
        return dict(bytes=4.0 * n + out + 36.0 * F, flops=flops)
    if kind == "multirate":
        F, T = _filters(case), case["T"]
        # share of the filters per level from the frequency law, at that level's rate
        e = -8.0 / 3.0
        lo, hi = 20.0 ** e, 1024.0 ** e
        edge = [1024.0] + [FS / 2.0 ** (r + 2) for r in range(1, case["levels"])] + [20.0]
        share = [(edge[r + 1] ** e - edge[r] ** e) / (lo - hi) for r in range(case["levels"])]
        updates = sum(F * s * n / 2.0 ** r for r, s in enumerate(share))
        # 12-tap interpolation of complex sums per template and output sample, all levels
        interp = 4.0 * 12.0 * T * n * (2.0 - 2.0 ** (2 - case["levels"]))
        return dict(bytes=4.0 * n + 8.0 * T * n + 36.0 * F, flops=12.0 * updates + interp)
    if kind == "adjoint":
        F, T = _filters(case), case["T"]
        return dict(bytes=4.0 * n + 16.0 * T * n + 36.0 * F, flops=(12.0 + 24.0) * F * n)
    if kind == "whiten":
        frame = case["frame"]
        fft = 5.0 * frame * math.log2(frame)
        frames = n / (frame / 2.0)
        return dict(bytes=8.0 * n + 4.0 * case["train"],
                    flops=frames * 2.0 * fft + (case["train"] / (frame / 2.0)) * fft)
    return dict(bytes=4.0 * n, flops=2.0 * n)


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------

def _z64(bank, x, n, dev, reduce=None):
    """Template sums of the last n samples: each template's impulse response over
    the whole stream, by an FFT convolution in complex128. reduce: applied to
    each template's row in turn instead of keeping it."""
    N = len(x)
    M = 1 << int(2 * N - 1).bit_length()
    X = torch.fft.fft(torch.as_tensor(np.asarray(x, np.float64), device=dev).to(torch.complex128), n=M)
    t = torch.arange(N, device=dev, dtype=torch.float64)
    loga = torch.log(torch.as_tensor(bank.a, device=dev))
    b = torch.as_tensor(bank.b, device=dev)
    d = torch.as_tensor(bank.d, device=dev, dtype=torch.float64)
    rows = []
    step = max(1, (1 << 23) // N)
    for j in range(bank.n_templates):
        h = torch.zeros(N, dtype=torch.complex128, device=dev)
        for k in range(int(bank.offsets[j]), int(bank.offsets[j + 1]), step):
            e = min(int(bank.offsets[j + 1]), k + step)
            s = t[None, :] - d[k:e, None]
            v = torch.exp(loga[k:e, None] * s.clamp_min(0.0)) * b[k:e, None]
            h += torch.where(s >= 0, v, torch.zeros((), dtype=v.dtype, device=dev)).sum(0)
        z = torch.fft.ifft(torch.fft.fft(h, n=M) * X)[N - n:N]
        rows.append(z if reduce is None else None)
        if reduce is not None:
            reduce(z)
    return torch.stack(rows) if reduce is None else None


def _psd64(s, N):
    w = np.sin(np.pi * np.arange(N) / N) ** 2
    frames = [np.abs(np.fft.rfft(w * s[i:i + N])) ** 2 for i in range(0, len(s) - N + 1, N // 2)]
    return np.mean(frames, axis=0) / np.sum(w * w)


def _whiten64(x, psd, N):
    """Whole-stream frame-wise whitening; output delayed by N / 2."""
    H = N // 2
    w = np.sin(np.pi * np.arange(N) / N) ** 2
    inv = np.where(psd > 0, 1.0 / np.sqrt(np.where(psd > 0, psd, 1.0)), 0.0)
    p = np.concatenate([np.zeros(H), np.asarray(x, np.float64)])
    out = np.zeros(len(p))
    for i in range(0, len(p) - N + 1, H):
        out[i:i + N] += np.fft.irfft(np.fft.rfft(w * p[i:i + N]) * inv, N)
    return out[:len(x)]


def _adjoint64(bank, x, g, dev):
    """z, and the gradients sum_m G[m] conj(dz[m]/da), sum_m G[m] conj(dz[m]/db)."""
    n = len(x)
    M = 1 << int(2 * n - 1).bit_length()
    t = torch.arange(n, device=dev, dtype=torch.float64)
    X = torch.fft.fft(torch.as_tensor(np.asarray(x, np.float64), device=dev).to(torch.complex128), n=M)
    impulse = bool(x[0] == 1.0 and not np.any(x[1:]))
    ga, gb, zs = [], [], []
    for j in range(bank.n_templates):
        lo, hi = int(bank.offsets[j]), int(bank.offsets[j + 1])
        G = torch.as_tensor(g[j], device=dev).to(torch.complex128)
        z = torch.zeros(n, dtype=torch.complex128, device=dev)
        for k in range(lo, hi, max(1, (1 << 23) // n)):
            e = min(hi, k + max(1, (1 << 23) // n))
            a, b = (torch.as_tensor(v[k:e], device=dev)[:, None] for v in (bank.a, bank.b))
            s = t[None, :] - torch.as_tensor(bank.d[k:e], device=dev, dtype=torch.float64)[:, None]
            zero = torch.zeros((), dtype=torch.complex128, device=dev)
            w = torch.where(s >= 0, torch.exp(torch.log(a) * s.clamp_min(0.0)), zero)
            v = torch.where(s >= 1, s * torch.exp(torch.log(a) * (s - 1).clamp_min(0.0)), zero)
            if not impulse:
                w, v = (torch.fft.ifft(torch.fft.fft(u, n=M) * X)[:, :n] for u in (w, v))
            gb.append((G * w.conj()).sum(1))
            ga.append((G * v.conj()).sum(1) * b[:, 0].conj())
            z += (b * w).sum(0)
        zs.append(z)
    return dict(z=torch.stack(zs), grad_a=torch.cat(ga), grad_b=torch.cat(gb))


def _multirate64(banks, h, g, x, dev):
    xs = [np.asarray(x, np.float64)]
    for _ in banks[1:]:
        xs.append(np.convolve(xs[-1], h)[:len(xs[-1])][1::2])
    G = torch.as_tensor(g, device=dev, dtype=torch.float64)
    w = None
    for bank, xr in zip(reversed(banks), reversed(xs)):
        z = _z64(bank, xr, len(xr), dev)
        if w is not None:
            up = torch.zeros_like(z)
            up[:, 0::2] = w
            for i in range(len(G)):
                z[:, i:] += G[i] * up[:, :z.shape[1] - i]
        w = z
    return w


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    kind, n = case["kind"], case["n"]
    if kind == "cluster":
        return None
    if kind in ("rows", "z"):
        bank, x = _inputs(case, seed)
        z = _z64(bank, x, n, dev)
        return z if kind == "z" else z.real ** 2 + z.imag ** 2
    if kind == "multirate":
        banks, x = _inputs(case, seed)
        h, g = _taps()
        return _multirate64(banks, h, g, x, dev)[:, n:].contiguous()
    if kind == "adjoint":
        bank, x, g = _inputs(case, seed)
        return _adjoint64(bank, x, g, dev)
    if kind == "whiten":
        train, x = _inputs(case, seed)
        w = len(x) - n
        before = _psd_model(case["frame"])
        if not case["train"]:
            return _whiten64(x, before, case["frame"])[w:]
        # the first half-frame of the block still overlaps the last frame of the
        # stretch before it, which was whitened with the earlier PSD
        H = case["frame"] // 2
        p = np.concatenate([np.zeros(H), np.asarray(x, np.float64)])
        psd = _psd64(np.asarray(train, np.float64), case["frame"])
        win = np.sin(np.pi * np.arange(2 * H) / (2 * H)) ** 2
        out = np.zeros(len(p))
        for i in range(0, len(p) - 2 * H + 1, H):
            s = before if i + 2 * H <= w + H else psd
            out[i:i + 2 * H] += np.fft.irfft(np.fft.rfft(win * p[i:i + 2 * H]) / np.sqrt(s), 2 * H)
        return out[w:w + n]
    bank, train, x = _inputs(case, seed)
    white = _whiten64(x, _psd64(np.asarray(train, np.float64), case["frame"]), case["frame"])
    best = torch.zeros(n, dtype=torch.float64, device=dev)

    def keep(z):
        torch.maximum(best, z.real ** 2 + z.imag ** 2, out=best)

    _z64(bank, white, n, dev, keep)
    return dict(white=white[len(white) - n:].copy(), max=best, index=None, template=None, snr=None, total=None)
