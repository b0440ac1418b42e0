"""The byte models of the kernels that are launched (CPU): what the profile summaries set beside the
counters of each kernel agrees with the class figures that bench.py reports."""

import pytest

from paper_2602_14016_amd import profile_summary as ps
from paper_2602_14016_amd.roofline import CLASS_NAMES, field_bytes, kernel_bytes


@pytest.mark.parametrize("N", [128, 256, 512, 1024])
def test_classes_and_kernels_agree(N):
    Yb, Cb = field_bytes(N)
    total = lambda name: sum(ps.kernel_rw_bytes(name, N))
    # velocity pair in, products out; velocity and cotangent pairs in, products out
    assert kernel_bytes(0, N) == 4 * Yb == total(f"row_sq_kernel<{N}, 2>") == total(f"row_sq_pipe_kernel<{N}>")
    assert kernel_bytes(2, N) == 6 * Yb == total(f"row_mul_kernel<{N}, 1>") == total(f"row_mul_pipe_kernel<{N}>")
    for form in ("col_pass_kernel", "col_twin_kernel"):
        # a pair in and a pair out; compact operands and outputs by stage
        mean = lambda modes: sum(total(f"{form}<{N}, 1, {m}>") for m in modes) / 4
        assert mean((1, 2, 3, 4)) == pytest.approx(kernel_bytes(1, N)) == 4 * Yb + 2.75 * Cb
        assert mean((7, 8, 9, 10)) == pytest.approx(kernel_bytes(3, N)) == 4 * Yb + 2.5 * Cb
        assert ps.kernel_rw_bytes(f"{form}<{N}, 1, 5>", N) is None   # not a stage
    assert [CLASS_NAMES[c].split("_kernel")[0] for c in range(4)] == ["row_sq", "col_pass", "row_mul", "col_pass"]
