"""Grids up to 64^2, whose time loop runs in one workgroup per member: the places where a run of
steps is cut into launches (observed steps, checkpoint boundaries, members that end early, the
longest launch) against the oracle, and bitwise against the same solve cut elsewhere."""

import numpy as np
import pytest
import torch

import oracle as O
from oracle.model import Obs, Physics

pytestmark = pytest.mark.gpu

FIELD_TOL = 1e-11   # fields and costs, relative
GRAD_TOL = 1e-9     # gradients, relative L2


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("N,B,osteps,K,forced", [(8, 3, [0, 1, 7], 2, False), (16, 2, [7], 7, True),
                                                 (32, 2, [0, 3, 4], 3, True), (64, 1, [2, 5], 4, False)])
def test_gradient_of_runs_cut_everywhere(N, B, osteps, K, forced):
    """Observed first, last and neighbouring steps, ragged segments, steps after the last observation."""
    from paper_2602_14016_amd import Observations, Solver
    print("CASE small-gradient", N, B, osteps, K, flush=True)
    extra = dict(mu=0.1, forcing_amp=1.0, forcing_k=4 if N > 8 else 2) if forced else {}
    steps, stride = 7, 4 if N > 8 else 2
    ph = Physics(N=N, nu=1e-3, dt=4e-3, **extra)
    w0 = O.init_field(N, list(range(1, B + 1)), kind=1, k0=2.0)
    vals = np.random.default_rng(7).standard_normal((B, len(osteps), 2, N // stride, N // stride)) * 0.3
    s = Solver(N, B, nu=ph.nu, dt=ph.dt, **extra)
    obs = Observations(stride, osteps, dev(vals))
    J, g = s.adjoint_gradient(dev(w0), steps, obs, ckpt_every=K)
    f = s.forward(dev(w0), steps, obs, want_obs=True, ckpt_every=K)
    J1, g1 = s.adjoint_gradient(dev(w0), steps, obs, ckpt_every=steps)
    assert torch.equal(J, J1) and torch.equal(g, g1) and torch.equal(J, f["J"])
    for b in range(B):
        Jr, gr = O.adjoint_gradient(w0[b], ph, steps, Obs(stride, osteps, vals[b]))
        wT, _, mo = O.forward(w0[b], ph, steps, Obs(stride, osteps))
        assert abs(float(J[b]) - Jr) <= FIELD_TOL * Jr
        assert rel(g[b].cpu().numpy(), gr) < GRAD_TOL
        assert rel(f["omega_T"][b].cpu().numpy(), wT) < FIELD_TOL
        assert rel(f["obs"][b].cpu().numpy(), mo) < FIELD_TOL


def test_longest_launch_is_split():
    """4100 steps of an 8^2 flow take three launches each way; checkpoints every 1000 cut them
    elsewhere with the same bits.  Rounding over 4100 steps stays far below the field tolerance of
    the smooth, decaying flow, so the oracle's end state is met within it."""
    from paper_2602_14016_amd import Observations, Solver
    print("CASE small-long", flush=True)
    N, steps = 8, 4100
    ph = Physics(N=N, nu=1e-3, dt=1e-3)
    w0 = O.init_field(N, [3], kind=1, k0=2.0)
    wT, _, _ = O.forward(w0[0], ph, steps, Obs(2, [0]))
    s = Solver(N, 1, nu=ph.nu, dt=ph.dt)
    obs = Observations(2, [0, steps], dev(np.zeros((1, 2, 2, 4, 4))))
    assert rel(s.forward(dev(w0), steps)["omega_T"][0].cpu().numpy(), wT) < FIELD_TOL
    a = s.adjoint_gradient(dev(w0), steps, obs, ckpt_every=steps)
    b = s.adjoint_gradient(dev(w0), steps, obs, ckpt_every=1000)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("N", [16, 64])
def test_members_ending_at_their_own_steps(N):
    """Members whose horizons end at different steps, one at step 0, give the bits of each alone."""
    from paper_2602_14016_amd import KernelSpec, Observations, Solver
    print("CASE small-members", N, flush=True)
    rng = np.random.default_rng(5)
    sets = [[0, 4, 9], [3, 5], [5], [0]]
    w0 = dev(O.init_field(N, [1, 2, 3, 4], kind=1, k0=2.0))
    obs = [Observations(4, st, dev(rng.standard_normal((1, len(st), 2, N // 4, N // 4)) * 0.3)) for st in sets]
    ker = [KernelSpec(0, 0.0), KernelSpec(1, 0.1), KernelSpec(2, 0.5), KernelSpec(0, 0.0)]
    w, H, it = Solver(N, 4, nu=1e-3, dt=4e-3).assimilate_members(w0, obs, ker, max_iter=2, ckpt_every=4)
    one = Solver(N, 1, nu=1e-3, dt=4e-3)
    for b in range(4):
        wb, Hb, ib = one.assimilate_members(w0[b:b + 1].contiguous(), [obs[b]], [ker[b]], max_iter=2, ckpt_every=2)
        assert torch.equal(w[b], wb[0]) and H[b] == Hb[0] and it[b] == ib[0], b
