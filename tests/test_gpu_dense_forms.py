"""Dense tiles straight from the packed entries, at the edges of their forms:
several rows per workgroup, one-workgroup and two-pass transforms, r = 1, 3, 5,
rows whose support is wider than a decimated transform, rows at DC and
Nyquist. Reference: the N-point inverse FFT (numpy, 64 bits) of the windowed
spectrum, which the tile is by definition. Bars as for every dense tile
(rel-L2 1e-5 FP32, 1e-12 FP64)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp64": 1e-12}
# (N, Q, f_min, f_max, rows, segments), 1 Hz bins
CASES = [(48, 1.5, 2.0, 24.0, 3, 5), (64, 2.0, 3.0, 32.0, 5, 3), (640, 4.0, 5.0, 320.0, 7, 3), (1536, 0.6, 20.0, 700.0, 5, 2),
         (5 * 256, 0.5, 20.0, 640.0, 3, 2), (2048, 0.5, 8.0, 1024.0, 3, 2), (3 * 16384, 1.0, 500.0, 20000.0, 3, 1),
         (5 * 16384, 0.5, 500.0, 40960.0, 3, 1), (65536, 4.0, 100.0, 32768.0, 3, 1)]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("case", CASES, ids=["N%d" % c[0] for c in CASES])
def test_dense_forms(case, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    n, q, f_min, f_max, R, B = case
    print("case", case, precision, flush=True)
    p = qt.Plan(float(n), n, q, f_min, f_max, R, cap_mode="none", precision=precision)
    x = np.random.default_rng(n).standard_normal((B, n)).astype(np.float32).astype(np.float64)
    xd = torch.from_numpy(x).to(device="cuda", dtype=torch.float64 if precision == "fp64" else torch.float32)
    D = p.dense(p.forward(xd)).cpu().numpy()
    Z = np.zeros((B, R, n), dtype=np.complex128)
    Z[:, :, :n // 2 + 1] = np.fft.rfft(x)[:, None, :] * p.windows_dense()
    T = np.fft.ifft(Z)
    err = np.linalg.norm((D - T).reshape(B, -1), axis=1) / np.linalg.norm(T.reshape(B, -1), axis=1)
    assert err.max() <= TOL[precision], err


@pytest.mark.parametrize("precision,n,rows,B", [("fp32", 24576, 62, 7), ("fp32", 16384, 100, 8), ("fp64", 24576, 40, 3),
                                                ("fp64", 5 * 4096, 64, 3), ("fp32", 4096, 200, 45)])
def test_dense_many_rows_same_bits(precision, n, rows, B):
    """A batch whose tiles take the two-group form gives each segment the bits
    it has alone."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    print("case", precision, n, rows, B, flush=True)
    p = qt.Plan(4096.0, n, 8.0, 20.0, 2000.0, rows, precision=precision)
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((B, n), generator=gen, device="cuda", dtype=torch.float64 if precision == "fp64" else torch.float32)
    D = p.dense(p.forward(x))
    for i in (0, B - 1):
        assert torch.equal(p.dense(p.forward(x[i:i + 1])), D[i:i + 1])
