"""Synthesis of a few segments (sibling workgroups) and of many (a workgroup
per segment): the same bits, at the lengths 3 2^k and 5 2^k whose workgroup
has more than 512 threads."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,n", [("fp32", 24576), ("fp32", 20480), ("fp64", 12288), ("fp64", 10240)])
def test_same_bits_alone_and_in_a_batch(precision, n):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_29785_amd as qt
    print("case", precision, n, flush=True)
    p = qt.Plan(float(n), n, 4.0, n / 256.0, n / 2.0, 16, precision=precision)
    B = torch.cuda.get_device_properties(0).multi_processor_count // 4 + 1    # 12 B > 3 CUs
    cdt = torch.complex128 if precision == "fp64" else torch.complex64
    gen = torch.Generator(device="cuda").manual_seed(n)
    y = torch.randn((B, 16, p.N_out), generator=gen, device="cuda", dtype=cdt)
    X, G = p.inverse(y), p.forward_adjoint(y)
    for i in (0, B - 1):
        assert torch.equal(p.inverse(y[i:i + 1]), X[i:i + 1])
        assert torch.equal(p.forward_adjoint(y[i:i + 1]), G[i:i + 1])
    assert torch.equal(p.inverse(y[:7]), X[:7])
