"""Velocity rows at probes and their sources on the wavefront-resident row plans: every row variant
that a tile choice can name, from a probe at every point to one per field, against torch in 64 bits."""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B,variant", [(128, 2, 0), (128, 3, 1), (128, 1, 2), (256, 1, 0), (256, 2, 1),
                                         (256, 3, 2), (512, 2, 0), (512, 1, 2), (1024, 1, 1), (1024, 2, 2)])
def test_probe_values_cost_and_gradient(N, B, variant):
    """White fields, one step, observed at both ends.  Sums of at most 2 * 2 N^2 squares in a
    fixed order round to less than 1e-12 of the cost; the gradient is as far off as that of a
    dense observation, 1e-11."""
    from paper_2602_14016_amd import Observations, Solver
    dt, Kc = 1e-4, (N - 1) // 3
    g = torch.Generator(device="cuda").manual_seed(N + 7 * B + variant)
    k = torch.fft.fftfreq(N, 1.0 / N, dtype=torch.float64, device="cuda")
    ky, kx = k[:, None], k[None, :]
    k2 = kx ** 2 + ky ** 2
    mask = ((kx.abs() <= Kc) & (ky.abs() <= Kc) & (k2 > 0)).double()
    ik2 = mask / torch.where(k2 > 0, k2, torch.ones_like(k2))
    w0 = torch.randn(B, N, N, dtype=torch.float64, device="cuda", generator=g)
    w0 = torch.fft.ifft2(mask * torch.fft.fft2(w0)).real.contiguous()
    w0 /= w0.std()
    phys = lambda f: torch.fft.ifft2(f).real

    def rhs(w):
        u, v = phys(1j * ky * ik2 * w), phys(-1j * kx * ik2 * w)
        return -mask * torch.fft.fft2(u * phys(1j * kx * w) + v * phys(1j * ky * w))

    def observe(w, stride):
        uv = torch.stack([phys(1j * ky * ik2 * w), phys(-1j * kx * ik2 * w)], dim=1)
        return uv[:, :, ::stride, ::stride]

    s = Solver(N, B, nu=0.0, dt=dt)
    s.set_tiles(row_variant=variant, adj_variant=variant)
    for stride in (1, 2, N // 2, N):
        print("CASE probe-rows", N, B, variant, stride, flush=True)
        M = N // stride
        vals = torch.randn(B, 2, 2, M, M, dtype=torch.float64, device="cuda", generator=g)
        x = w0.clone().requires_grad_(True)
        w = mask * torch.fft.fft2(x)
        a = rhs(w)
        b = rhs(w + dt / 2 * a)
        c = rhs(w + dt / 2 * b)
        end = w + dt / 6 * (a + 2 * b + 2 * c + rhs(w + dt * c))
        want = torch.stack([observe(w, stride), observe(end, stride)], dim=1)
        J = 0.5 * ((want - vals) ** 2).flatten(1).sum(1)
        (gx,) = torch.autograd.grad(J.sum(), x)
        gx = phys(mask * torch.fft.fft2(gx))
        got = s.forward(w0, 1, Observations(stride, [0, 1], vals), want_obs=True)["obs"]
        Jg, gg = s.adjoint_gradient(w0, 1, Observations(stride, [0, 1], vals), ckpt_every=1)
        want, J = want.detach(), J.detach()
        for m in range(B):
            assert float((got[m] - want[m]).abs().max()) < 1e-12 * float(want[m].abs().max()) + 1e-13, (stride, m)
            assert abs(float(Jg[m] - J[m])) < 1e-12 * float(J[m]), (stride, m)
            assert float((gg[m] - gx[m]).norm() / gx[m].norm()) < 1e-11, (stride, m)
