"""The byte models of the kernels that are launched (CPU): what the profile summaries set beside the
counters of each kernel agrees with the class figures that bench.py reports."""

import csv

import pytest

from paper_2602_14016_amd import profile_summary as ps
from paper_2602_14016_amd.roofline import CLASS_NAMES, field_bytes, kernel_bytes, read_traffic


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


def test_traffic_record_holds_every_plan_of_its_kernel(tmp_path):
    """The record of one plan also answers for the others that the counter runs hold."""
    def runs(path, counter, rows):
        with open(path, "w", newline="") as fh:
            w = csv.writer(fh)
            w.writerow(["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
            for i, (name, kib) in enumerate(rows):
                w.writerow([i, name if name.startswith("__") else f"void pa::{name}(pa::Dims, pa::RowArgs)", counter, kib])

    names = ("row_mul_kernel<256, 2>", "row_mul_kernel<256, 1>", "row_mul_pipe_kernel<256>", "row_sq_kernel<256, 2>")
    runs(tmp_path / "f.csv", "FETCH_SIZE", [("__amd_rocclr_copyBuffer", 1024.0)] + [(n, 100.0 + i) for i, n in enumerate(names)])
    runs(tmp_path / "w.csv", "WRITE_SIZE", [("__amd_rocclr_copyBuffer", 2048.0)] + [(n, 40.0) for n in names])
    out = tmp_path / "t.txt"
    ps.main(["traffic", str(tmp_path / "f.csv"), str(tmp_path / "w.csv"), "--command", "c", "--members", "64", "--N", "256",
             "--cls", "2", "--kernel", names[0], "--calib-mib", "2", "--out", str(out)])
    for i, n in enumerate(names[:3]):
        assert read_traffic(2, 256, 64, kernel=n, path=str(out)) == 1024 * (2 * (100 + i) + 40), n
    assert read_traffic(2, 256, 64, kernel=names[3], path=str(out)) is None
    assert read_traffic(2, 256, 64, kernel="row_mul_kernel<256, 0>", path=str(out)) is None
