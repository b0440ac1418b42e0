"""The library holds the kernels it can launch and no others: on grids up to 64^2, whose time loop is
one kernel, no row products and no stage columns; one copy of each plan (CPU: symbols of the built
library)."""

import collections
import os
import re
import subprocess


def test_kernels_of_each_grid():
    from paper_2602_14016_amd import build, native
    if not os.path.exists(native.LIB_PATH):
        build.build(verbose=False)
    text = subprocess.run(["nm", "-C", native.LIB_PATH], stdout=subprocess.PIPE, text=True, check=True).stdout
    found = collections.defaultdict(set)
    for name, args in re.findall(r"__device_stub__(\w+)<([\d, ]+)>", text):
        a = tuple(int(x) for x in args.split(","))
        found[a[0]].add((name,) + a[1:])
    columns = lambda n: {k[2] for k in found[n] if k[0] in ("col_pass_kernel", "col_twin_kernel")}
    plans = lambda n, kernel: {k[1] for k in found[n] if k[0] == kernel}
    assert set(found) == {8, 16, 32, 64, 128, 256, 512, 1024}
    for N in (8, 16, 32, 64):
        held = {("row_sq_pipe_kernel",), ("row_mul_pipe_kernel",)} if N == 64 else set()   # for test_lds_dma_codegen.py
        assert {k[0] for k in found[N] - held} == {"row_r2c_kernel", "row_c2r_kernel", "col_pass_kernel", "col_twin_kernel",
                                            "small_forward_kernel", "small_adjoint_kernel", "small_filter_kernel"}, N
        assert columns(N) <= {0, 5, 6, 12}, N   # init, filter, from a state, first guess
    for N in (128, 256, 512, 1024):
        assert columns(N) == set(range(13)), N
        rows = {"row_r2c_kernel", "row_c2r_kernel", "row_sq_kernel", "row_mul_kernel", "row_obs_kernel", "row_src_kernel"}
        for kernel in rows:
            assert plans(N, kernel) == {128: {0, 1, 2}, 256: {0, 1, 2}, 512: {0}, 1024: {3}}[N], (N, kernel)
        assert (("row_sq_pipe_kernel",) in found[N]) == (N <= 256)
    for N, want in ((8, {0}), (16, {0}), (32, {0}), (64, {0, 1}), (128, {0, 1, 2}), (512, {0}), (1024, {0, 1})):
        assert plans(N, "col_pass_kernel") == want, N
