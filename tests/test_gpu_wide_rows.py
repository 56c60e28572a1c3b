"""Row kernels in their two forms (one group of butterflies per thread, or two
from a number of rows on): a batch that takes the two-group form gives each
segment the bits it has in a batch that does not, forward, inverse, row
statistics and masked inverse, at the shortest and longest rows of both
precisions; and the values are those of the oracle."""
import numpy as np
import pytest

from oracle import oracle as o

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp64": 1e-12}
# (precision, fs, N, Q, rows, N_out, segments above the line)
CASES = [("fp32", 4096.0, 32768, 8.0, 256, 2048, 65), ("fp32", 4096.0, 131072, 16.0, 256, 4096, 33),
         ("fp32", 4096.0, 262144, 8.0, 200, 8192, 6), ("fp32", 4096.0, 524288, 8.0, 250, 16384, 3),
         ("fp64", 4096.0, 16384, 8.0, 256, 1024, 65), ("fp64", 4096.0, 32768, 8.0, 256, 2048, 33),
         ("fp64", 4096.0, 131072, 16.0, 250, 4096, 5), ("fp64", 4096.0, 262144, 8.0, 200, 8192, 3)]


@pytest.mark.parametrize("case", CASES, ids=["%s_%d" % (c[0], c[5]) for c in CASES])
def test_both_forms_same_bits(case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    precision, fs, n, q, R, n_out, B = case
    print("case", case, flush=True)
    p = qt.Plan(fs, n, q, 10.0, fs / 2, R, n_out=n_out, precision=precision)
    row = n_out * (16 if precision == "fp64" else 8)
    line = (64 if row >= 65536 else 256) << 20
    assert B * R * row >= line > R * row          # the batch is above the line, a segment below
    rdt = torch.float64 if precision == "fp64" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(n_out)
    x = torch.randn((B, n), generator=gen, device="cuda", dtype=rdt)
    Y = p.forward(x)
    Ym, m = p.forward_metric(x)
    assert torch.equal(Ym, Y)
    X = p.inverse(Y)
    gain = torch.linspace(0.5, 1.5, R, device="cuda", dtype=rdt)
    lam = torch.full((R,), 0.5 / np.sqrt(n_out), device="cuda", dtype=rdt)
    Xm = p.inverse_masked(Y, gain, lam)
    for i in (0, B - 1):
        one = x[i:i + 1]
        y1 = p.forward(one)
        assert torch.equal(y1, Y[i:i + 1])
        m1 = p.forward_metric(one)[1]   # sums over a row in another order: rounding only
        assert float((m1 - m[i:i + 1]).abs().max() / m1.abs().max()) <= (1e-13 if precision == "fp64" else 1e-5)
        assert torch.equal(p.inverse(y1), X[i:i + 1])
        assert torch.equal(p.inverse_masked(y1, gain, lam), Xm[i:i + 1])
    op = o.OraclePlan(fs=fs, n=n, q=q, f_min=10.0, f_max=fs / 2, rows=R, n_out=n_out)
    xh = x[B - 1].double().cpu().numpy()
    ref = op.forward(xh)
    e = np.linalg.norm(Y[B - 1].cpu().numpy() - ref) / np.linalg.norm(ref)
    xm = op.project(xh)
    ex = np.linalg.norm(X[B - 1].cpu().numpy() - xm) / np.linalg.norm(xm)
    # the dual frame amplifies rounding by up to sqrt(kappa); the bar is stated for kappa <= 1e4
    kappa = p.info.frame_B / p.info.frame_A
    assert e <= TOL[precision] and ex <= TOL[precision] * max(1.0, (kappa / 1e4) ** 0.5), (e, ex)


@pytest.mark.parametrize("case", CASES, ids=["%s_%d" % (c[0], c[5]) for c in CASES])
def test_row_statistics_same_bits(case):
    """The row statistics of a segment have the same bits alone, in a batch
    whose rows take the two-group form, and in that batch under a workspace
    that cuts it into chunks of the one-group form."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    precision, fs, n, q, R, n_out, B = case
    print("case", case, flush=True)
    p = qt.Plan(fs, n, q, 10.0, fs / 2, R, n_out=n_out, precision=precision)
    rdt = torch.float64 if precision == "fp64" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(7 * n_out)
    x = torch.randn((B, n), generator=gen, device="cuda", dtype=rdt)
    m = p.forward_metric(x)[1]
    small = torch.empty(p.workspace_bytes(1), dtype=torch.uint8, device="cuda")
    assert torch.equal(p.forward_metric(x, ws=small)[1], m)
    for i in (0, B - 1):
        assert torch.equal(p.forward_metric(x[i:i + 1])[1], m[i:i + 1])
