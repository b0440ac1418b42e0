"""Rounding of the forward state for fields whose spectrum peaks far below the band's edge.

The passes multiply the spectra of u^2 - v^2 and u v by kx ky and kx^2 - ky^2, and with them the
rounding of those spectra.  That is white: a unit of rounding eps U^2 in each product, times about
a = sqrt(log2 N^2) for the transforms on either side of it.  Over the band, |kx|, |ky| <= K =
(N - 1) / 3, the two multipliers have a mean square of (2/5 - 2/9) K^4 and K^4 / 9 (the second one's
field, v^2 - u^2, four times the variance of the first's), the band holds 4/9 of the modes, and
the Runge-Kutta weights (1, 2, 2, 1) / 6 add four independent errors a step to sqrt(10) / 6.  H
steps of dt then leave
    0.53 K^2 * a * eps * U^2 * (sqrt(10) / 6) * dt * sqrt(H)
of noise in a vorticity of RMS W, if nothing damps it."""

import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,k0,dt,H", [(256, 4.0, 2e-3, 20), (512, 4.0, 1e-3, 20), (1024, 4.0, 5e-4, 20), (1024, 10.0, 5e-4, 20)])
def test_forward_noise_of_smooth_fields(N, k0, dt, H):
    """Within four times that, and 1e-14 for all other rounding of either side, of the advective
    form on torch's transforms in 64 bits."""
    from paper_2602_14016_amd import Solver
    print("CASE smooth", N, k0, flush=True)
    nu, K = 1e-4, (N - 1) // 3
    s = Solver(N, 1, nu=nu, dt=dt)
    w0 = s.init_field([7], kind=0, k0=k0, target=0.5)
    got = s.forward(w0, H)["omega_T"][0]
    k = torch.fft.fftfreq(N, 1.0 / N, dtype=torch.float64, device="cuda")
    ky, kx = k[:, None], k[None, :N // 2 + 1].abs()
    k2 = kx ** 2 + ky ** 2
    mask = ((kx <= K) & (ky.abs() <= K) & (k2 > 0)).double()
    ik2 = mask / torch.where(k2 > 0, k2, torch.ones_like(k2))
    phys = lambda f: torch.fft.irfft2(f, s=(N, N))

    def rhs(w):
        u, v = phys(1j * ky * ik2 * w), phys(-1j * kx * ik2 * w)
        return -mask * torch.fft.rfft2(u * phys(1j * kx * w) + v * phys(1j * ky * w))

    w = mask * torch.fft.rfft2(w0[0])
    E2, E1 = torch.exp(-nu * k2 * dt / 2), torch.exp(-nu * k2 * dt)
    u2 = float((phys(1j * ky * ik2 * w) ** 2 + phys(-1j * kx * ik2 * w) ** 2).mean())
    for _ in range(H):
        a = rhs(w)
        b = rhs(E2 * (w + dt / 2 * a))
        c = rhs(E2 * w + dt / 2 * b)
        d = rhs(E1 * w + dt * E2 * c)
        w = E1 * w + dt / 6 * (E1 * a + 2 * E2 * (b + c) + d)
    end = phys(w)
    noise = 0.53 * K ** 2 * math.sqrt(2 * math.log2(N)) * 2.0 ** -53 * u2 * math.sqrt(10) / 6 * dt * math.sqrt(H)
    rel = float((got - end).norm() / end.norm())
    allowed = 4 * noise / float(end.pow(2).mean().sqrt()) + 1e-14
    print("smooth", N, k0, "rel %.2e allowed %.2e" % (rel, allowed), flush=True)
    assert rel < allowed
    assert float((end - w0[0]).norm() / w0.norm()) > 1e-3   # the flow has moved
