"""Preconditioner calls on grids that fit a workgroup: separate, in-place and overlapping buffers,
members at 8-byte offsets, against the oracle."""

import numpy as np
import pytest
import torch

import oracle as O
from oracle.precond import Kernel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B", [(8, 1), (8, 5), (16, 3), (32, 2), (64, 1), (64, 3)])
@pytest.mark.parametrize("kind,param,metric,power", [(1, 0.1, 0, 0.5), (2, 0.7, 1, -0.5), (3, 2e-3, 2, 0.5), (0, 0.0, 0, 1.0)])
def test_preconditioner_buffers(N, B, kind, param, metric, power):
    """Two transforms of N^2 points in doubles: 1e-13 of the field."""
    from paper_2602_14016_amd import KernelSpec, Solver
    print("CASE small-filter", N, B, kind, power, flush=True)
    rng = np.random.default_rng(N + B + kind)
    x = rng.standard_normal((B, N, N))
    ref = np.stack([O.precondition(x[b], Kernel(kind, param, metric), power) for b in range(B)])
    s, k, n = Solver(N, B, nu=1e-3, dt=1e-3), KernelSpec(kind, param, metric), B * N * N
    for at, to in ((0, n), (n, 0), (0, 0), (1, 1), (0, 1), (3, 0), (0, N * N), (N * N, 0)):
        buf = torch.zeros(2 * n + N * N, dtype=torch.float64, device="cuda")
        src, dst = buf[at:at + n].view(B, N, N), buf[to:to + n].view(B, N, N)
        src.copy_(torch.from_numpy(x))
        got = s.precondition(src, k, power, out=dst).cpu().numpy()
        err = np.linalg.norm((got - ref).reshape(B, -1), axis=1)
        assert np.all(err < 1e-13 * np.linalg.norm(ref.reshape(B, -1), axis=1)), (at, to)
