"""Row transforms of 512 and 1024 points that live on one wavefront: every entry of the band and
every row of a workgroup, against torch's transform in 64 bits."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B", [(512, 1), (512, 3), (1024, 1), (1024, 2)])
def test_one_step_of_white_fields(N, B):
    """A field with energy at every retained wavenumber, one step with large dt * nonlinearity, and
    the adjoint of that step.  A wrong twiddle or lane in one entry changes the result by about
    1/N of its size; rounding is below 1e-13 of it (products of size |u|^2 |k|^2 against omega)."""
    from paper_2602_14016_amd import Observations, Solver
    print("CASE wave-rows", N, B, flush=True)
    dt, Kc = 1e-4, (N - 1) // 3
    g = torch.Generator(device="cuda").manual_seed(N + B)
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

    def step(x):
        w = mask * torch.fft.fft2(x)
        a = rhs(w)
        b = rhs(w + dt / 2 * a)
        c = rhs(w + dt / 2 * b)
        d = rhs(w + dt * c)
        return phys(w + dt / 6 * (a + 2 * b + 2 * c + d))

    def observe(x):
        w = mask * torch.fft.fft2(x)
        return torch.stack([phys(1j * ky * ik2 * w), phys(-1j * kx * ik2 * w)], dim=1)

    x = w0.clone().requires_grad_(True)
    end = step(x)
    J = 0.5 * (observe(end) ** 2).sum()
    (gx,) = torch.autograd.grad(J, x)
    gx = phys(mask * torch.fft.fft2(gx))
    s = Solver(N, B, nu=0.0, dt=dt)
    vals = torch.zeros(B, 1, 2, N, N, dtype=torch.float64, device="cuda")
    got = s.forward(w0, 1)["omega_T"]
    Jg, gg = s.adjoint_gradient(w0, 1, Observations(1, [1], vals), ckpt_every=1)
    for b in range(B):
        assert float((got[b] - end[b]).norm() / end[b].norm()) < 1e-12, b
        assert float((got[b] - end[b]).abs().max()) < 1e-10, b
        assert float((gg[b] - gx[b]).norm() / gx[b].norm()) < 1e-11, b
    assert abs(float(Jg.sum()) - float(J)) < 1e-11 * float(J)
    assert float((end - w0).norm() / w0.norm()) > 1e-6   # the nonlinear term is in the comparison
