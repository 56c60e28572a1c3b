"""Chirp-z rows by overlap-save blocks, FP32: no systematic scale.

The spectrum of a unit impulse at sample 0 is 1 in every bin with no rounding
(the transforms copy and add zeros), so the envelopes it gives show the rows'
transforms alone. What rounding does to them has no preferred sign: each table
entry and operation is rounded to nearest, and the projection of the error on
the exact envelopes averages over R * N_out > 10^4 values, to a few hundredths
of u = 2^-24. Constants and twiddles rounded once and used for all values do
have one, about -2e-8 per pass, which the rows' tables take out: the projection
stays within u / 2. Reference: the inverse DFT (numpy, 64 bits) of each
window about its centre bin."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R,n_out", [(24576, 62, 1539), (24576, 62, 2305), (24576, 62, 7223), (24576, 62, 12289),
                                       (16384, 16, 2357), (16384, 64, 1201), (131072, 64, 4179)])
def test_rows_have_unit_gain(n, R, n_out):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    print("case", n, R, n_out, flush=True)
    q = 16.0 if n == 131072 else 8.0
    p = qt.Plan(4096.0, n, q, 20.0, 2048.0, R, n_out=n_out)
    x = torch.zeros((1, n), device="cuda")
    x[0, 0] = 1.0
    Y = p.forward(x)[0].cpu().numpy().astype(np.complex128)
    W = p.windows_dense()
    Z = np.zeros((R, n_out))
    for k in range(R):
        bins = np.nonzero(W[k])[0]
        Z[k, (bins - p.centre[k]) % n_out] = W[k, bins]
    ref = np.fft.ifft(Z, axis=1) * np.sqrt(n_out / n)
    gain = np.vdot(ref, Y - ref).real / np.vdot(ref, ref).real
    assert abs(gain) <= 2.0 ** -25, gain
