"""Chirp-z rows by overlap-save blocks (N_out not a power of two, plain
windows): the forward, the inverse and both adjoints against the FP64 oracle
where the blocks' edges fall differently. The bars are the parity bars of the
plain rows (rel-L2 1e-5 FP32, 1e-12 FP64): the rows' transforms are shorter
than one convolution over the row and the blocks add up in a fixed order, so
the error per row stays a small multiple of u log2(length)."""
import numpy as np
import pytest

from oracle import oracle as o

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp64": 1e-12}
CAP = {"cover": o.CAP_COVER, "paper": o.CAP_PAPER, "none": o.CAP_NONE}

# (fs, N, Q, f_min, f_max, rows, N_out, cap, segments, inverse too)
CASES = {
    "few_values_per_row": (256.0, 64, 4.0, 16.0, 100.0, 5, 9, "none", 3, False),
    "several_rows_per_workgroup": (1024.0, 1024, 4.0, 8.0, 400.0, 7, 117, "cover", 3, True),
    "ragged_workgroups": (1024.0, 4096, 6.0, 30.0, 100.0, 7, 333, "cover", 3, False),
    "support_from_dc_to_nyquist": (1024.0, 1024, 0.5, 8.0, 512.0, 9, 1030, "none", 2, True),
    "narrowest_envelope": (4096.0, 24576, 8.0, 10.0, 2048.0, 62, 1537, "cover", 2, True),
    "one_and_two_blocks": (4096.0, 24576, 8.0, 10.0, 2048.0, 62, 1028, "paper", 2, False),
    "many_blocks": (4096.0, 24576, 8.0, 10.0, 2048.0, 62, 12285, "cover", 1, True),
    "longest_transform": (4096.0, 131072, 6.0, 100.0, 600.0, 5, 8000, "none", 1, False),
    "one_row": (4096.0, 16384, 8.0, 300.0, 300.0, 1, 301, "none", 2, False),
}


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("name", list(CASES))
def test_overlap_save_rows(name, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    fs, n, q, f_min, f_max, R, n_out, cap, B, inverse = CASES[name]
    print("case", name, precision, flush=True)
    gp = qt.Plan(fs, n, q, f_min, f_max, R, n_out=n_out, cap_mode=cap, precision=precision)
    op = o.OraclePlan(fs=fs, n=n, q=q, f_min=f_min, f_max=f_max, rows=R, n_out=n_out, cap_mode=CAP[cap])
    assert gp.N_out == n_out and n_out & (n_out - 1)
    rng = np.random.default_rng(n_out)
    rdt = torch.float64 if precision == "fp64" else torch.float32
    cdt = torch.complex128 if precision == "fp64" else torch.complex64
    x = rng.standard_normal((B, n)).astype(np.float32).astype(np.float64)
    xd = torch.from_numpy(x).to(device="cuda", dtype=rdt)
    Y = gp.forward(xd)
    Y_ref = op.forward(x)
    assert rel(Y.cpu().numpy(), Y_ref) <= TOL[precision]
    # one segment alone gives the same bits as in the batch
    assert torch.equal(gp.forward(xd[B - 1:]), Y[B - 1:])
    # any envelope, not only one the forward gives
    G = (rng.standard_normal((B, R, n_out)) + 1j * rng.standard_normal((B, R, n_out))).astype(np.complex64)
    Gd = torch.from_numpy(G).to(device="cuda", dtype=cdt)
    if inverse:
        assert rel(gp.inverse(Gd).cpu().numpy(), op.inverse(G.astype(np.complex128))) <= TOL[precision]
        # <G^T x, G> = <x, inverse(G)> in 64-bit sums
        gy = gp.inverse_adjoint(xd)
        a = torch.sum((gy.to(torch.complex128).conj() * Gd.to(torch.complex128)).real)
        xi = gp.inverse(Gd).double()
        scale = float(torch.linalg.norm(xd.double()) * torch.linalg.norm(xi))
        assert abs(float(a - torch.sum(xd.double() * xi))) <= TOL[precision] * scale
    gx = gp.forward_adjoint(Gd).double()
    a = torch.sum((Y.to(torch.complex128).conj() * Gd.to(torch.complex128)).real)
    scale = float(torch.linalg.norm(Y.to(torch.complex128)) * torch.linalg.norm(Gd.to(torch.complex128)))
    assert abs(float(a - torch.sum(xd.double() * gx))) <= TOL[precision] * scale
