"""Workspace sizes: each call asks for the intermediates that its passes write
and no more (host), and a call given exactly that much stays inside it and
gives the bits it gives with more (GPU)."""
import pytest

import paper_2603_29785_amd as qt
from paper_2603_29785_amd import binding

# N, whether the half spectrum fits one workgroup, four-step spectrum, two-pass tiles (FP32, FP64)
FORMS = [
    (16384, (True, True), (False, False), (False, True)),
    (24576, (True, False), (False, False), (False, False)),
    (40960, (False, False), (False, False), (False, False)),
    (49152, (False, False), (False, False), (False, True)),
    (65536, (False, False), (True, True), (True, True)),
    (3 * 32768, (False, False), (True, True), (True, True)),
]


def a256(v):
    return (v + 255) // 256 * 256


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,one,four,dense2", FORMS, ids=["N%d" % f[0] for f in FORMS])
def test_sizes_are_the_intermediates(n, one, four, dense2, precision):
    f64 = precision == "fp64"
    cb = 16 if f64 else 8
    decimated = n & (n - 1) != 0
    for B in (1, 3):
        p = qt.Plan(4096.0, n, 8.0, 20.0, 2000.0, 31, precision=precision, host_only=True)
        half = a256(B * n // 2 * cb)
        pack = a256(B * p.info.sum_len * cb)
        want = half + pack                            # spectrum, kept slots
        if four[f64]:
            want += half                              # between the two passes
        if decimated and not one[f64]:
            want += half                              # decimated rows
        assert p.workspace_bytes(B) == want
        tiles = B * p.R * n * cb if dense2[f64] else 0
        assert binding.lib.qtam_dense_workspace_size(p._h, B) == want + tiles


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [f[0] for f in FORMS])
def test_calls_stay_inside_their_workspace(n, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case", n, precision, flush=True)
    p = qt.Plan(4096.0, n, 8.0, 20.0, 2000.0, 31, precision=precision)
    B = 3
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((B, n), generator=gen, device="cuda", dtype=torch.float64 if precision == "fp64" else torch.float32)

    def exactly(need):
        buf = torch.full((need + 65536,), 0xA5, dtype=torch.uint8, device="cuda")
        return buf[:need], buf[need:]

    y = p.forward(x)
    for f, arg, need in ((p.forward, x, p.workspace_bytes(B)), (p.inverse, y, p.workspace_bytes(B)),
                         (p.forward_adjoint, y, p.workspace_bytes(B)), (p.inverse_adjoint, x, p.workspace_bytes(B)),
                         (p.dense, y, binding.lib.qtam_dense_workspace_size(p._h, B))):
        roomy = torch.zeros(4 * need + (1 << 20), dtype=torch.uint8, device="cuda")
        ws, after = exactly(need)
        assert torch.equal(f(arg, ws=ws), f(arg, ws=roomy))
        assert bool((after == 0xA5).all())
