"""The two-group form of the row kernels where the other tests of it do not go:
both adjoints, windows other than the bisquare, rows of a regularised window
(whole band, slots modulo N_out), and dense tiles. Each batch is above the line
from which launches take that form and one segment is below it; a segment has
the same bits in both, and the batch's last segment is compared with the
definition (numpy, 64 bits). Bars: rel-L2 1e-5 FP32, 1e-12 FP64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp64": 1e-12}


def torch_or_skip():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def line(values, precision):
    row = values * (16 if precision == "fp64" else 8)
    return row, (64 if row >= 65536 else 256) << 20


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


def rows_of(p, S, table):
    """Envelopes of a spectrum: table times S at the slots about the centre."""
    Z = np.zeros((p.R, p.N_out), dtype=np.complex128)
    bins = np.arange(p.N // 2 + 1)
    for k in range(p.R):
        keep = table[k] != 0.0
        Z[k, (bins[keep] - p.centre[k]) % p.N_out] = table[k, keep] * S[keep]
    return np.fft.ifft(Z, axis=1) * np.sqrt(p.N_out / p.N)


def signal_of(p, G, table):
    """irfft of the sum over rows of table times the DFT of the envelopes."""
    F = np.fft.fft(G, axis=1) * np.sqrt(p.N / p.N_out)
    bins = np.arange(p.N // 2 + 1)
    X = sum(table[k] * F[k, (bins - p.centre[k]) % p.N_out] for k in range(p.R))
    return np.fft.irfft(X, n=p.N)


CASES = [("fp32", 4096.0, 32768, 8.0, 256, 2048, 65, "hann", 0.0, 0.0),
         ("fp32", 4096.0, 65536, 8.0, 172, 16384, 3, "tukey", 0.5, 0.0),
         ("fp64", 4096.0, 16384, 8.0, 256, 1024, 65, "kaiser", 6.0, 0.0),
         ("fp64", 4096.0, 65536, 8.0, 172, 8192, 3, "hann", 0.0, 0.0),
         ("fp32", 4096.0, 16384, 8.0, 24, 16384, 22, "bisquare", 0.0, 1e-3),
         ("fp32", 4096.0, 4096, 8.0, 24, 4096, 342, "hann", 0.0, 1e-3),
         ("fp64", 4096.0, 8192, 8.0, 24, 8192, 22, "bisquare", 0.0, 1e-3)]


@pytest.mark.parametrize("case", CASES, ids=["%s_%d_%s%s" % (c[0], c[5], c[7], "_eps" if c[9] else "") for c in CASES])
def test_adjoints_windows_and_whole_band_rows(case):
    torch = torch_or_skip()
    import paper_2603_29785_amd as qt
    precision, fs, n, q, R, n_out, B, window, param, eps = case
    print("case", case, flush=True)
    p = qt.Plan(fs, n, q, 10.0, fs / 2, R, n_out=n_out, precision=precision, window=window, window_param=param,
                window_eps=eps)
    row, least = line(n_out, precision)
    assert B * R * row >= least > R * row
    rdt, cdt = (torch.float64, torch.complex128) if precision == "fp64" else (torch.float32, torch.complex64)
    gen = torch.Generator(device="cuda").manual_seed(n_out + B)
    x = torch.randn((B, n), generator=gen, device="cuda", dtype=torch.float32).to(rdt)
    g = torch.randn((B, R, n_out), generator=gen, device="cuda", dtype=torch.complex64).to(cdt)
    calls = {"forward": (p.forward, x), "inverse": (p.inverse, g), "forward_adjoint": (p.forward_adjoint, g),
             "inverse_adjoint": (p.inverse_adjoint, x)}
    out = {k: f(a) for k, (f, a) in calls.items()}
    for k, (f, a) in calls.items():
        for i in (0, B - 1):
            assert torch.equal(f(a[i:i + 1]), out[k][i:i + 1]), (k, i)
    W = p.windows_dense()
    P = (W * W).sum(axis=0)
    keep = (P > 0.0) & (P >= 1e-6 * P.max())
    D = W * np.where(keep, 1.0 / np.where(keep, P, 1.0), 0.0)
    xh, gh = x[-1].double().cpu().numpy(), g[-1].cpu().numpy().astype(np.complex128)
    S = np.fft.rfft(xh)
    assert rel(out["forward"][-1].cpu().numpy(), rows_of(p, S, W)) <= TOL[precision]
    assert rel(out["inverse"][-1].cpu().numpy(), signal_of(p, gh, D)) <= TOL[precision]
    # adjoints under Re<.,.>: a bin inside the band stands for itself and its
    # conjugate, so the inverse's sum over bins counts it twice
    c = np.full(n // 2 + 1, 2.0)
    c[0] = c[-1] = 1.0
    assert rel(out["forward_adjoint"][-1].cpu().numpy(), signal_of(p, gh, W / c)) <= TOL[precision]
    assert rel(out["inverse_adjoint"][-1].cpu().numpy(), rows_of(p, S, D * c)) <= TOL[precision]


@pytest.mark.parametrize("precision,n,rows,B", [("fp64", 1024, 128, 129), ("fp64", 2048, 128, 65), ("fp64", 4096, 64, 17),
                                                ("fp64", 8192, 64, 9), ("fp32", 2048, 128, 129), ("fp32", 8192, 100, 11)])
def test_dense_tiles(precision, n, rows, B):
    torch = torch_or_skip()
    import paper_2603_29785_amd as qt
    print("case", precision, n, rows, B, flush=True)
    p = qt.Plan(4096.0, n, 8.0, 4096.0 / n * 20.0, 2000.0, rows, precision=precision)
    row, least = line(n, precision)
    assert rows * B * row >= least > rows * row
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((B, n), generator=gen, device="cuda", dtype=torch.float32)
    x = x.double() if precision == "fp64" else x
    D = p.dense(p.forward(x))
    for i in (0, B - 1):
        assert torch.equal(p.dense(p.forward(x[i:i + 1])), D[i:i + 1])
    Z = np.zeros((rows, n), dtype=np.complex128)
    Z[:, :n // 2 + 1] = np.fft.rfft(x[-1].double().cpu().numpy()) * p.windows_dense()
    assert rel(D[-1].cpu().numpy(), np.fft.ifft(Z, axis=1)) <= TOL[precision]
