"""Spectrum and synthesis of segments with N/2 = r * M2 (r = 1, 3, 5) against
the FP64 oracle at the edges of their forms: the shortest segments, several
segments per workgroup with a ragged last one, the longest that fit one
workgroup, the first that do not (decimated one-pass transforms), and the
decimated two-pass ones. Bars as for every plan without frame holes (rel-L2
1e-5 FP32, 1e-12 FP64)."""
import numpy as np
import pytest

from oracle import oracle as o

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp64": 1e-12}
#      r * 2^k samples, segments
SIZES = [(16, 3), (1024, 7), (16384, 2),
         (48, 9), (768, 11), (3 * 4096, 2), (3 * 8192, 3), (3 * 16384, 2), (3 * 65536, 2),
         (80, 9), (1280, 5), (5 * 2048, 2), (5 * 4096, 3), (5 * 8192, 2), (5 * 32768, 1)]


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,B", SIZES)
def test_segment_spectra(n, B, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    print("case", n, B, precision, flush=True)
    # rows over the whole band (1 Hz bins), so every bin of the spectrum counts
    R = 3 if n < 100 else 16
    kw = dict(q=1.5 if n < 100 else 4.0, f_min=2.0 if n < 100 else n / 256.0, f_max=n / 2.0)
    gp = qt.Plan(float(n), n, kw["q"], kw["f_min"], kw["f_max"], R, precision=precision)
    op = o.OraclePlan(fs=float(n), n=n, rows=R, **kw)
    rng = np.random.default_rng(n)
    rdt = torch.float64 if precision == "fp64" else torch.float32
    x = rng.standard_normal((B, n)).astype(np.float32).astype(np.float64)
    xd = torch.from_numpy(x).to(device="cuda", dtype=rdt)
    Y = gp.forward(xd)
    assert rel(Y.cpu().numpy(), op.forward(x)) <= TOL[precision]
    assert rel(gp.inverse(Y).cpu().numpy(), op.project(x)) <= TOL[precision]
    assert torch.equal(gp.forward(xd[B - 1:]), Y[B - 1:])   # the same bits alone
