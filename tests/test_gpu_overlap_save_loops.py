"""Chirp-z rows by overlap-save blocks, in both forms of each direction: few
rows (the blocks of a row in parallel: a workgroup each, forward; thread groups
of one workgroup, inverse) and many (one after the other in a workgroup). A
segment has the same bits alone and in a batch of more than 8 rows per CU, and
the batch's values are those of the definition (numpy, 64 bits). One, two and
up to sixteen blocks, transforms of 512 to 8192 values."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp64": 1e-12}
# N, Q, rows, N_out, cap
CASES = [(16384, 8.0, 16, 1537, "cover"), (16384, 8.0, 16, 4817, "cover"), (16384, 24.0, 64, 701, "cover"),
         (24576, 8.0, 62, 1028, "paper"), (24576, 8.0, 62, 7223, "cover"), (24576, 8.0, 8, 3535, "none"),
         (4096, 8.0, 16, 301, "cover"), (4096, 8.0, 8, 2501, "cover"), (131072, 16.0, 64, 6145, "cover")]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("case", CASES, ids=["M%d" % c[3] for c in CASES])
def test_alone_and_in_a_batch(case, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    n, q, R, n_out, cap = case
    print("case", case, precision, flush=True)
    p = qt.Plan(4096.0, n, q, 20.0, 2048.0, R, n_out=n_out, cap_mode=cap, precision=precision)
    B = 8 * torch.cuda.get_device_properties(0).multi_processor_count // R + 1
    rdt, cdt = (torch.float64, torch.complex128) if precision == "fp64" else (torch.float32, torch.complex64)
    gen = torch.Generator(device="cuda").manual_seed(n_out)
    x = torch.randn((B, n), generator=gen, device="cuda", dtype=torch.float32).to(rdt)
    g = torch.randn((B, R, n_out), generator=gen, device="cuda", dtype=torch.complex64).to(cdt)
    Y, X = p.forward(x), p.inverse(g)
    last = B - 1
    for i in (0, last):
        assert torch.equal(p.forward(x[i:i + 1]), Y[i:i + 1])
        assert torch.equal(p.inverse(g[i:i + 1]), X[i:i + 1])
    W = p.windows_dense()
    P = (W * W).sum(axis=0)
    keep = (P > 0.0) & (P >= 1e-6 * P.max())
    S = np.fft.rfft(x[last].double().cpu().numpy())
    G = np.fft.fft(g[last].cpu().numpy().astype(np.complex128), axis=1)
    ref = np.zeros((R, n_out), dtype=np.complex128)
    back = np.zeros(n // 2 + 1, dtype=np.complex128)
    for k in range(R):
        bins = np.nonzero(W[k])[0]
        slot = (bins - p.centre[k]) % n_out
        ref[k, slot] = W[k, bins] * S[bins]
        back[bins] += W[k, bins] * G[k, slot]
    ref = np.fft.ifft(ref, axis=1) * np.sqrt(n_out / n)
    back = np.fft.irfft(np.where(keep, back / np.where(keep, P, 1.0), 0.0), n=n) * np.sqrt(n / n_out)
    e = np.linalg.norm(Y[last].cpu().numpy() - ref) / np.linalg.norm(ref)
    ei = np.linalg.norm(X[last].cpu().numpy() - back) / np.linalg.norm(back)
    assert e <= TOL[precision] and ei <= TOL[precision], (e, ei)
