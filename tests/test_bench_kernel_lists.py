"""The kernel kinds that one forward + inverse launches, form by form: their
algorithmic shares in bench.py add up to what the two calls must move (host),
and the library's own timing names exactly these kinds (GPU), so neither list
can go stale alone."""
import os
import sys

import pytest

import paper_2603_29785_amd as qt

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

ROWS = ["fwd_rows", "inv_rows", "overlap_add"]
LONG = ROWS + ["fwd_rows_pass2", "inv_rows_pass2"]
ONE = ["spectrum_fft", "synthesis_fft"]
TWO = ["spectrum_fft_pass1", "spectrum_fft_pass2", "synthesis_fft_pass1", "synthesis_fft_pass2"]
RADIX = ["spectrum_radix", "synthesis_radix"]
#         plan arguments, N_out, kinds in FP32, kinds in FP64
FORMS = {
    "one workgroup, r = 1": ((4096.0, 16384, 8.0, 20.0, 1000.0, 16), 0, ONE + ROWS, ONE + ROWS),
    "one workgroup, r = 3": ((4096.0, 12288, 8.0, 20.0, 1000.0, 16), 0, ONE + ROWS, ONE + ROWS),
    "one workgroup, r = 5": ((4096.0, 10240, 8.0, 20.0, 1000.0, 16), 0, ONE + ROWS, ONE + ROWS),
    "decimated, one pass": ((4096.0, 49152, 8.0, 20.0, 1000.0, 16), 0, ONE + RADIX + ROWS, ONE + RADIX + ROWS),
    "decimated, two passes": ((4096.0, 5 * 32768, 8.0, 20.0, 1000.0, 16), 0, TWO + RADIX + ROWS, TWO + RADIX + ROWS),
    "two passes": ((4096.0, 131072, 8.0, 10.0, 2048.0, 16), 0, TWO + ROWS, TWO + LONG),
    "long rows": ((4096.0, 131072, 8.0, 10.0, 2048.0, 4), 65536, TWO + LONG, TWO + LONG),
    "chirp-z rows": ((4096.0, 24576, 8.0, 10.0, 2048.0, 62), 12289, ONE + ROWS, ONE + RADIX + ROWS),
    "long chirp-z rows": ((4096.0, 131072, 4.0, 500.0, 2048.0, 4), 65535, TWO + ROWS, TWO + ROWS),
}
CASES = [(f, pr) for f in FORMS for pr in ("fp32", "fp64")]


def kinds_of(form, precision):
    return FORMS[form][3 if precision == "fp64" else 2]


def plan_of(form, precision, host_only):
    args, n_out = FORMS[form][:2]
    return qt.Plan(*args, n_out=n_out, cap_mode="none" if n_out == 65535 else "cover", precision=precision,
                   host_only=host_only)


@pytest.mark.parametrize("form,precision", CASES)
def test_shares_of_the_launched_kernels_add_up(form, precision):
    p = plan_of(form, precision, True)
    B, b = 5, 8 if precision == "fp64" else 4
    total = sum(bench.kernel_bytes(k, p, B, b) for k in kinds_of(form, precision))
    assert total == float(B * (2 * b * p.N + 4 * b * p.R * p.N_out))


@pytest.mark.gpu
@pytest.mark.parametrize("form,precision", CASES)
def test_timed_kinds_are_the_listed_ones(form, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case", form, precision, flush=True)
    p = plan_of(form, precision, False)
    x = torch.randn((1, p.N), device="cuda", dtype=torch.float64 if precision == "fp64" else torch.float32)
    p.timing(True)
    p.inverse(p.forward(x))
    torch.cuda.synchronize()
    assert sorted(p.timing_collect()) == sorted(kinds_of(form, precision))
