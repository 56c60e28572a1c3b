"""The calls that users of this library make, as timed and checked cases.

Each case names one of seven kinds of program (`kind`) and its sizes:

* ``pair``      forward transform and canonical-dual inverse of a batch;
* ``forward``   forward transform alone (offline analysis of many segments);
* ``sweep``     several Q over one batch from one spectrum, each with its inverse;
* ``bank``      composite bank: forward with row statistics, best plane per segment;
* ``dense``     forward, then full-rate tiles of every row;
* ``denoise``   training step of the gain x soft-threshold denoiser;
* ``gradients`` backward pass through forward and inverse to the input.

``listed()`` holds one case for each way the library is used at the sizes of
its benchmark, its tests and the paper; ``draw`` spreads the same kinds over
the ranges of lengths, rows, Q, windows, envelope lengths, batches and
precisions they stand for. ``exact`` computes the same results in 64 bits with
plain torch from the definitions of the transform.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_29785_amd as qt
from paper_2603_29785_amd.autograd import GainThresholdDenoiser, qtam_forward, qtam_inverse

DEV = "cuda"


def listed():
    return [
        # One segment as it arrives: 4 s at 4096 Hz, 64 rows (latency; the
        # benchmark's one-segment workload).
        dict(name="one_segment", kind="pair", fs=4096.0, n=16384, batch=1, q="8", rows=64, f_min=20.0, f_max=1000.0,
             window="bisquare", n_out=0, cap="cover", precision="fp32"),
        # A few 16 s segments at once, as a serving bucket launches them.
        dict(name="serving_bucket", kind="pair", fs=4096.0, n=65536, batch=8, q="16", rows=128, f_min=10.0,
             f_max=2048.0, window="bisquare", n_out=0, cap="cover", precision="fp32"),
        # The batched benchmark: 256 x 32 s, the Q set 4 / 8 / 16 as one
        # sweep over each segment's spectrum, and the three inverses.
        dict(name="q_sweep_batch", kind="sweep", fs=4096.0, n=131072, batch=256, q="4,8,16", rows=256, f_min=10.0,
             f_max=2048.0, window="bisquare", n_out=0, cap="cover", precision="fp32"),
        # The same segments in double precision (reconstruction checks).
        dict(name="batch_fp64", kind="pair", fs=4096.0, n=131072, batch=64, q="8", rows=256, f_min=10.0,
             f_max=2048.0, window="bisquare", n_out=0, cap="cover", precision="fp64"),
        # Long segments (256 s at 8192 Hz, 512 rows of 32768 values), the
        # precision study's shape, in both precisions.
        dict(name="long_fp32", kind="pair", fs=8192.0, n=2097152, batch=32, q="12", rows=512, f_min=5.0, f_max=4096.0,
             window="bisquare", n_out=0, cap="cover", precision="fp32"),
        dict(name="long_fp64", kind="pair", fs=8192.0, n=2097152, batch=8, q="12", rows=512, f_min=5.0, f_max=4096.0,
             window="bisquare", n_out=0, cap="cover", precision="fp64"),
        # The paper's glitch tensors: 6 s at 4096 Hz (24576 = 3 * 2^13
        # samples), 62 rows; the minimal envelope ceil(T df_max) + 1 (an odd
        # length) over about a thousand segments, and the standard one of
        # N/2 + 1 = 12289 values.
        dict(name="glitch_minimal", kind="forward", fs=4096.0, n=24576, batch=1024, q="8", rows=62, f_min=10.0,
             f_max=2048.0, window="bisquare", n_out=-1, cap="paper", precision="fp32"),
        dict(name="glitch_standard", kind="pair", fs=4096.0, n=24576, batch=128, q="8", rows=62, f_min=10.0,
             f_max=2048.0, window="bisquare", n_out=12289, cap="cover", precision="fp32"),
        # Full-rate tiles of the same segments (the spectrogram a user plots).
        dict(name="glitch_dense", kind="dense", fs=4096.0, n=24576, batch=16, q="8", rows=62, f_min=10.0,
             f_max=2048.0, window="bisquare", n_out=0, cap="cover", precision="fp32"),
        # Multi-Q analysis: one bank, the best plane of every segment.
        dict(name="bank_selection", kind="bank", fs=4096.0, n=131072, batch=32, q="4,8,16", rows=256, f_min=10.0,
             f_max=2048.0, window="bisquare", n_out=0, cap="cover", precision="fp32"),
        # Training step of the denoiser (64 x 8 s), and input gradients of a
        # differentiable pipeline in double precision.
        dict(name="denoiser_step", kind="denoise", fs=4096.0, n=32768, batch=64, q="8", rows=128, f_min=10.0,
             f_max=2048.0, window="bisquare", n_out=0, cap="cover", precision="fp32"),
        dict(name="gradients_fp64", kind="gradients", fs=4096.0, n=32768, batch=32, q="8", rows=128, f_min=10.0,
             f_max=2048.0, window="bisquare", n_out=0, cap="cover", precision="fp64"),
    ]


WINDOW_PARAM = {"bisquare": 0.0, "hann": 0.0, "kaiser": 8.0, "tukey": 0.5}


def draw(rng):
    kind = rng.choice(["pair", "pair", "pair", "forward", "forward", "sweep", "bank", "dense", "denoise", "gradients"])
    # segment lengths r * 2^k: 1024 samples to 2^21 (the four-minute segments)
    r = rng.choice([1, 1, 1, 3, 5])
    top = 17 if kind in ("dense", "denoise", "gradients") else 21
    n = r * 2 ** rng.randint(10, top - (0, 0, 0, 2, 0, 3)[r])
    fs = float(rng.choice([1024, 2048, 4096, 8192, 16384]))
    f_min = rng.uniform(max(10.0, 4.0 * fs / n), max(30.0, 8.0 * fs / n))
    f_max = fs * rng.choice([0.5, rng.uniform(0.2, 0.5)])
    q = rng.choice([4.0, 6.0, 8.0, 12.0, 16.0, 32.0])
    case = dict(kind=kind, fs=fs, n=n, batch=1, q="%g" % q, rows=int(round(2 ** rng.uniform(4.0, 9.0))),
                f_min=round(f_min, 3), f_max=round(f_max, 3),
                window=rng.choice(["bisquare", "bisquare", "hann", "kaiser", "tukey"]), n_out=0, cap="cover",
                precision=rng.choice(["fp32", "fp32", "fp32", "fp64"]))
    if kind in ("sweep", "bank"):
        case["q"] = ",".join("%g" % v for v in sorted(rng.sample([4.0, 6.0, 8.0, 12.0, 16.0, 32.0], rng.randint(2, 3))))
        case["rows"] = min(case["rows"], 256)
    # enough rows for neighbouring bands to overlap, as an inverse needs
    widest = max(float(v) for v in case["q"].split(","))
    case["rows"] = max(case["rows"], min(512, 2 + int(math.log(f_max / f_min) / math.log1p(1.0 / widest))))
    limit = 3e8 if kind in ("sweep", "bank", "dense") else 6e8
    if kind in ("pair", "forward") and rng.random() < 0.3 and n <= 2 ** 18:
        # an envelope length the caller chose, often not a power of two
        case["n_out"] = int(round(tables(case, float(case["q"].split(",")[0]))["max_len"] * rng.uniform(1.0, 1.6)))
        limit = 1.5e8
    # batch: from one segment to what the envelopes (or tiles) allow
    per = sum(t["rows"] * t["n_out"] for t in all_tables(case)) * 8.0 * (2 if case["precision"] == "fp64" else 1)
    if kind == "dense":
        per = case["rows"] * n * 8.0 * (2 if case["precision"] == "fp64" else 1)
    most = max(1.0, min(1024.0, limit / per))
    case["batch"] = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    return case


# ---------------------------------------------------------------------------
# Inputs: coloured noise with a chirp and two sine-Gaussian glitches in each
# segment, drawn on the device from the seed.
# ---------------------------------------------------------------------------
def signals(case, seed, clean=False):
    b, n, fs = case["batch"], case["n"], case["fs"]
    rdt = torch.float64 if case["precision"] == "fp64" else torch.float32
    rng = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(rng.integers(1 << 60)))
    freq = torch.fft.rfftfreq(n, 1.0 / fs, device=DEV, dtype=torch.float32)
    gain = torch.where(freq < 20.0, (20.0 / freq.clamp(min=1.0)) ** 2, torch.ones_like(freq))
    gain[0] = 0.0
    x = torch.empty((b, n), dtype=rdt, device=DEV)
    c = torch.zeros((b, n), dtype=rdt, device=DEV) if clean else None
    t = torch.arange(n, device=DEV, dtype=torch.float32) / fs
    T = n / fs
    step = max(1, (1 << 25) // n)
    for i in range(0, b, step):
        m = min(step, b - i)
        w = torch.randn((m, n), generator=gen, device=DEV, dtype=torch.float32)
        w = torch.fft.irfft(torch.fft.rfft(w) * gain, n=n)

        def col(lo, hi):
            return torch.tensor(rng.uniform(lo, hi, size=(m, 1)), device=DEV, dtype=torch.float32)

        sig = torch.zeros_like(w)
        d = 0.5 * T * col(0.2, 1.0)
        u = (t - (T - d) * col(0.0, 1.0)) / d
        sig += torch.where((u > 0) & (u < 1), 5.0 * torch.sin(math.pi * u.clamp(0, 1)) ** 2
                           * torch.sin(2 * math.pi * d * fs * (0.01 * u + 0.03 * u ** 3)), torch.zeros_like(w))
        for _ in range(2):
            f0, t0 = fs * col(0.02, 0.35), T * col(0.05, 0.95)
            tau = col(4.0, 20.0) / (math.sqrt(2.0) * math.pi * f0)
            sig += 5.0 * torch.exp(-((t - t0) / tau) ** 2) * torch.sin(2 * math.pi * f0 * (t - t0))
        x[i:i + m] = w + sig
        if clean:
            c[i:i + m] = sig
    return (x, c) if clean else x


def n_out_of(case, q):
    if case["n_out"] >= 0:
        return case["n_out"]
    f = grid(case)
    return math.ceil(case["n"] / case["fs"] * float(np.max(np.diff(f)))) + 1   # the paper's minimal envelope


def qs(case):
    return [float(v) for v in case["q"].split(",")]


def make_plan(case, q, planes=None):
    return qt.Plan(case["fs"], case["n"], q, case["f_min"], case["f_max"], case["rows"], window=case["window"],
                   window_param=WINDOW_PARAM[case["window"]], cap_mode=case["cap"], n_out=n_out_of(case, q),
                   precision=case["precision"], planes=planes)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind)
    if kind == "denoise":
        s["x"], s["clean"] = signals(case, seed, clean=True)
        p = make_plan(case, qs(case)[0])
        s["model"] = GainThresholdDenoiser(p, thresholds(case, p.R))
        with torch.no_grad():   # gains as they stand part way through a training
            s["model"].gain.copy_(torch.linspace(0.7, 1.3, p.R, device=DEV, dtype=s["x"].dtype))
        return s
    s["x"] = signals(case, seed)
    b = case["batch"]
    if kind == "bank":
        s["plans"] = [make_plan(case, 1.0, [(q, case["window"], WINDOW_PARAM[case["window"]]) for q in qs(case)])]
    else:
        s["plans"] = [make_plan(case, q) for q in qs(case)]
    if kind == "gradients":
        s["x"].requires_grad_(True)
        s["g"] = signals(case, seed + (1 << 40))
        return s
    if kind == "sweep":   # a long-running analysis keeps its outputs and its workspace
        cdt = torch.complex128 if case["precision"] == "fp64" else torch.complex64
        s["y"] = [torch.empty((b, p.R, p.N_out), dtype=cdt, device=DEV) for p in s["plans"]]
        s["xr"] = [torch.empty_like(s["x"]) for _ in s["plans"]]
        s["ws"] = torch.empty(max(p.workspace_bytes(b) for p in s["plans"]), dtype=torch.uint8, device=DEV)
    return s


def run(s):
    kind = s["kind"]
    if kind == "denoise":
        model = s["model"]
        model.zero_grad(set_to_none=True)
        out = model(s["x"])
        loss = torch.mean((out - s["clean"]) ** 2)
        loss.backward()
        return dict(x=out.detach(), loss=loss.detach(), gain=model.gain.grad)
    plans, x = s["plans"], s["x"]
    p = plans[0]
    if kind == "pair":
        y = p.forward(x)
        return dict(y=y, x=p.inverse(y))
    if kind == "forward":
        return dict(y=p.forward(x))
    if kind == "sweep":
        qt.forward_sweep(plans, x, outs=s["y"], ws=s["ws"])
        for pl, y, xr in zip(plans, s["y"], s["xr"]):
            pl.inverse(y, out=xr, ws=s["ws"])
        return dict(y=s["y"], x=s["xr"])
    if kind == "bank":
        y, m = p.forward_metric(x)
        score, best, yb = p.select_planes(y, m, "energy")
        return dict(y=y, metric=m, score=score, best=best, y_best=yb)
    if kind == "dense":
        y = p.forward(x)
        return dict(y=y, dense=p.dense(y))
    assert kind == "gradients"
    x.grad = None
    out = qtam_inverse(qtam_forward(x, p), p)
    out.backward(s["g"])
    return dict(x=out.detach(), grad=x.grad)


# ---------------------------------------------------------------------------
# The definitions in 64 bits: grid, supports, windows, frame (numpy), and the
# transforms (torch.fft), without the library.
# ---------------------------------------------------------------------------
def grid(case):
    R = case["rows"]
    f = [case["f_min"] * (case["f_max"] / case["f_min"]) ** (k / (R - 1)) if R > 1 else case["f_min"]
         for k in range(R)]
    return np.array(f)


def shape(window, x):
    ax = np.abs(x)
    if window == "bisquare":
        return ((1.0 - ax) * (1.0 + ax)) ** 2
    if window == "hann":
        return 0.5 + 0.5 * np.cos(math.pi * x)
    a = WINDOW_PARAM[window]
    if window == "kaiser":
        return np.i0(a * np.sqrt(np.maximum(0.0, (1.0 - ax) * (1.0 + ax)))) / np.i0(a)
    assert window == "tukey"
    return np.where(ax <= 1.0 - a, 1.0, 0.5 + 0.5 * np.cos(math.pi * (ax - (1.0 - a)) / a))


def tables(case, q, windows=False):
    """Kept bins, slots and (windows=True) weights of one plane's rows, flat."""
    n, fs = case["n"], case["fs"]
    T, half = n / fs, n // 2
    f = grid(case)
    gap = int(math.ceil(T * float(np.max(np.diff(f))))) if len(f) > 1 else None
    cap = None if gap is None else (2 * gap + 1 if case["cap"] == "cover" else 2 * (gap // 2) + 1)
    s = np.floor(f * T + 0.5).astype(np.int64)
    h = np.maximum(1, np.ceil(f * T / q).astype(np.int64) // 2)
    if cap is not None:
        h = np.maximum(1, np.minimum(h, cap // 2))
    max_len = int(2 * h.max() + 1)
    n_out = n_out_of(case, q) or 1 << (max_len - 1).bit_length()
    t = dict(rows=len(f), max_len=max_len, n_out=n_out)
    if windows:
        lo, hi = np.maximum(0, s - h), np.minimum(half, s + h)
        bins, slot, w = [], [], []
        for k in range(len(f)):
            c = np.arange(lo[k], hi[k] + 1)
            v = shape(case["window"], (c - s[k]) / float(h[k]))
            bins.append(c)
            slot.append((c - s[k]) % n_out + k * n_out)
            w.append(v / np.sqrt(np.sum(v * v)))
        t.update(bins=np.concatenate(bins), slot=np.concatenate(slot), w=np.concatenate(w))
    return t


def all_tables(case, windows=False):
    """One table per plan; the planes of a bank as one plan of all rows."""
    got = [tables(case, q, windows) for q in qs(case)]
    if case["kind"] != "bank":
        return got
    n_out = max(t["n_out"] for t in got)
    out = dict(rows=sum(t["rows"] for t in got), max_len=max(t["max_len"] for t in got), n_out=n_out)
    if windows:
        slot, first = [], 0
        for t in got:
            row, u = t["slot"] // t["n_out"], t["slot"] % t["n_out"]
            u = np.where(u > t["n_out"] // 2, u - t["n_out"], u)       # signed offset from the centre
            slot.append((first + row) * n_out + u % n_out)
            first += t["rows"]
        out.update(slot=np.concatenate(slot), bins=np.concatenate([t["bins"] for t in got]),
                   w=np.concatenate([t["w"] for t in got]))
    return [out]


class Exact:
    """Forward and canonical-dual inverse of one plan in 64 bits."""

    def __init__(self, case, t):
        self.n, self.rows, self.n_out = case["n"], t["rows"], t["n_out"]
        self.bins = torch.from_numpy(t["bins"]).to(DEV)
        self.slot = torch.from_numpy(t["slot"]).to(DEV)
        self.w = torch.from_numpy(t["w"]).to(DEV)
        P = np.bincount(t["bins"], weights=t["w"] ** 2, minlength=self.n // 2 + 1)
        M = (P > 0) & (P >= 1e-6 * P.max())
        self.mask = torch.from_numpy(M).to(DEV)
        self.dual = torch.from_numpy(np.where(M, 1.0 / np.where(M, P, 1.0), 0.0)).to(DEV)

    def forward(self, x):
        X = torch.fft.rfft(x)
        Z = torch.zeros((x.shape[0], self.rows * self.n_out), dtype=torch.complex128, device=DEV)
        Z = Z.index_copy(1, self.slot, X[:, self.bins] * self.w)
        return torch.fft.ifft(Z.view(-1, self.rows, self.n_out)) * math.sqrt(self.n_out / self.n)

    def inverse(self, y):
        Z = torch.fft.fft(y).reshape(y.shape[0], -1)[:, self.slot] * (self.w * math.sqrt(self.n / self.n_out))
        X = torch.zeros((y.shape[0], self.n // 2 + 1), dtype=torch.complex128, device=DEV)
        return torch.fft.irfft(X.index_add(1, self.bins, Z) * self.dual, n=self.n)

    def project(self, x):
        return torch.fft.irfft(torch.fft.rfft(x) * self.mask, n=self.n)

    def dense(self, x):
        X = torch.fft.rfft(x)
        Z = torch.zeros((x.shape[0], self.rows, self.n), dtype=torch.complex128, device=DEV)
        row = torch.div(self.slot, self.n_out, rounding_mode="floor")
        Z[:, row, self.bins] = X[:, self.bins] * self.w
        return torch.fft.ifft(Z)


def thresholds(case, R):
    """Soft thresholds per row, from three times the median envelope of unit
    white noise (Rayleigh of mean square 1 / N_out) up."""
    rdt = torch.float64 if case["precision"] == "fp64" else torch.float32
    n_out = tables(case, qs(case)[0])["n_out"]
    return torch.linspace(1.0, 1.5, R, device=DEV, dtype=rdt) * (3.0 * math.sqrt(math.log(2.0) / n_out))


def exact(case, seed):
    kind = case["kind"]
    ts = all_tables(case, windows=True)
    step = max(1, (1 << 26) // max(max(t["rows"] * t["n_out"] for t in ts),
                                   ts[0]["rows"] * case["n"] if kind == "dense" else 1, case["n"]))

    def each(f, *xs):
        parts = [f(*(x[i:i + step].double() for x in xs)) for i in range(0, case["batch"], step)]
        return torch.cat(parts)

    e = [Exact(case, t) for t in ts]
    if kind == "denoise":
        x, clean = signals(case, seed, clean=True)
        lam = thresholds(case, e[0].rows).double()[:, None]
        rdt = x.dtype
        gain = torch.linspace(0.7, 1.3, e[0].rows, device=DEV, dtype=rdt).double().requires_grad_(True)
        outs, loss = [], 0.0
        for i in range(0, case["batch"], step):
            with torch.no_grad():
                y = e[0].forward(x[i:i + step].double())
                y = y * (1.0 - lam / y.abs().clamp(min=1e-300)).clamp(min=0.0)
            out = e[0].inverse(y * gain[:, None])
            part = torch.sum((out - clean[i:i + step].double()) ** 2) / x.numel()
            part.backward()
            outs.append(out.detach())
            loss = loss + part.detach()
        return dict(x=torch.cat(outs), loss=loss, gain=gain.grad)
    x = signals(case, seed)
    if kind == "gradients":
        g = signals(case, seed + (1 << 40))
        return dict(x=each(e[0].project, x), grad=each(e[0].project, g))
    y = [each(p.forward, x) for p in e]
    if kind == "forward":
        return dict(y=y[0])
    if kind == "pair":
        return dict(y=y[0], x=each(e[0].project, x))
    if kind == "sweep":
        return dict(y=y, x=[each(p.project, x) for p in e])
    if kind == "dense":
        return dict(y=y[0], dense=each(e[0].dense, x))
    assert kind == "bank"
    y, planes, R = y[0], len(qs(case)), case["rows"]
    power = torch.cat([(y[i:i + step].abs() ** 2).sum(-1) for i in range(0, len(y), step)])
    peak = torch.cat([(y[i:i + step].abs() ** 2).amax(-1) for i in range(0, len(y), step)])
    score = power.view(-1, planes, R).sum(-1)
    best = score.argmax(-1)
    yb = y.view(-1, planes, R, y.shape[-1])[torch.arange(len(y), device=DEV), best]
    return dict(y=y, metric=torch.complex(power, peak), score=score, best=best, y_best=yb)


def work(case):
    """Inputs read once and outputs written once; a call that takes another
    call's result reads it. Transforms at 5 L log2 L operations."""
    b, n, kind = case["batch"], case["n"], case["kind"]
    r = 8 if case["precision"] == "fp64" else 4
    x = b * n * r
    fx = 2.5 * b * n * math.log2(n)
    ts = all_tables(case)
    y = sum(b * t["rows"] * t["n_out"] * 2 * r for t in ts)
    fy = sum(5.0 * b * t["rows"] * t["n_out"] * math.log2(t["n_out"]) for t in ts)
    if kind == "forward":
        return dict(bytes=x + y, flops=fx + fy)
    if kind == "pair":
        return dict(bytes=2 * x + 2 * y, flops=2 * (fx + fy))
    if kind == "sweep":
        return dict(bytes=x + len(ts) * x + 2 * y, flops=fx + len(ts) * fx + 2 * fy)
    if kind == "bank":
        return dict(bytes=x + y + 2 * y / len(qs(case)), flops=fx + fy)
    if kind == "dense":
        d = b * case["rows"] * n * 2 * r
        return dict(bytes=x + 2 * y + d, flops=fx + 2 * fy + 5.0 * b * case["rows"] * n * math.log2(n))
    if kind == "denoise":     # forward, masked inverse, loss, and the gradient of the gains
        return dict(bytes=5 * x + 3 * y, flops=3 * (fx + fy))
    return dict(bytes=4 * x + 4 * y, flops=4 * (fx + fy))   # gradients: both directions and their adjoints
