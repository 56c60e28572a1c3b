"""The twiddles of the envelope rows' stride-16 pass, read off a transform.

A comb of P ones has a spectrum of P at the multiples of P and exact zeros
elsewhere, so a row whose support holds one such bin transforms a single value
v at the offset j of that bin. At j = r L / 256 (r = 1 .. 15) the value meets
one twiddle on its way, w = e^{2 pi i r m0 / 256}, and the outputs m0 + 256 m2
are v w without any other rounding. v is the output at 0.

Each component of such an output is then the product of v with a table entry:
two roundings, relative error at most 2 u + u^2, u = 2^-24. (A twiddle formed
by products of other twiddles misses that by far in its small component.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.mark.parametrize("n_out", [512, 1024, 2048, 4096])
def test_stride_16_twiddles_rounded_once(n_out):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    n, P = 16384, 512
    print("case", n_out, flush=True)
    r = np.arange(1, 16)
    j = r * (n_out // 256)
    s = 4096 - j                       # the tooth at bin 4096 sits at offset j of the row
    # 2 h_k + 1 <= n_out, and no other tooth in any support
    q = max(7.9, 4096.0 / (n_out - 4))
    order = np.argsort(s)
    p = qt.Plan(float(n), n, q, freqs=s[order].astype(np.float64), cap_mode="none", n_out=n_out)
    h = np.asarray(p.half_width)[np.argsort(order)]
    assert (h > j).all() and (h + j < P).all()
    x = torch.zeros((1, n), device="cuda")
    x[0, ::n // P] = 1.0
    Y = p.forward(x)[0].cpu().numpy()[np.argsort(order)]
    m0 = np.arange(16)
    for k in range(len(r)):
        v = float(Y[k, 0].real)
        assert v > 0.0 and Y[k, 0].imag == 0.0
        a = 2.0 * np.pi * (r[k] * m0 % 256) / 256.0
        for first in range(0, n_out, 256):
            got = Y[k, first:first + 16].astype(np.complex128)
            for g, e in ((got.real, np.cos(a)), (got.imag, np.sin(a))):
                zero = np.abs(e) < 1e-10
                assert np.all(np.abs(g[zero]) <= 1e-10 * v)
                err = np.abs(g[~zero] / (v * e[~zero]) - 1.0)
                assert err.max() <= 2.001 * U, (r[k], first, err.max() / U)
