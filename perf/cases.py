"""Measured workloads of the library, called as a user's program calls it.

Each case is one pass through a public entry point of the package: a forward
run with model observations, a cost gradient, an adjoint impulse response with
shell energies, the same gradient behind autograd, a preconditioner call, a
4D-Var solve and a batch of served 4D-Var requests.  Grids are 16^2 to 1024^2
(the library takes powers of two from 8 to 1024), batches 1 to 64 members, and
all data is float64, the library's only type.  A pass keeps the horizons short
(tens of steps; a gradient's cost is proportional to them) so that it can be
repeated.

A program that sets no tiles runs the library's own choice ("tiles": False:
the command-line configurations, the README's example, autograd).  The
ensemble benchmark and the request server tune a tile table once and keep it
("tiles": True): TILES holds what the autotuner finds for them.

exact() is a plain torch.fft implementation of the same scheme in 64 bits:
pseudo-spectral vorticity equation in advective form with the 2/3 rule,
Lawson RK4, gradients by reverse-mode differentiation of one step at a time.
"""

import math

import torch

from paper_2602_14016_amd import KernelSpec, Observations, Solver
from paper_2602_14016_amd.autograd import adjoint_cost

# what autotune() returns for the ensemble benchmark (64 members of 256^2) and
# for the request server's table (four members per grid, shares left to each launch)
TILES = {
    (256, 64): dict(row_variant=2, row_teams=2, adj_variant=2, adj_teams=2, col_variant=1, col_block=8, col_split=0),
    128: dict(row_variant=1, row_teams=4, adj_variant=2, adj_teams=2, col_variant=2, col_block=4, col_split=0),
    256: dict(row_variant=2, row_teams=4, adj_variant=2, adj_teams=8, col_variant=2, col_block=4, col_split=0),
    512: dict(row_variant=2, row_teams=8, adj_variant=0, adj_teams=8, col_variant=0, col_block=4, col_split=0),
    1024: dict(row_variant=3, row_teams=8, adj_variant=2, adj_teams=4, col_variant=2, col_block=2, col_split=0),
}

DECAYING, KOLMOGOROV = "decaying", "kolmogorov"
KERNELS = ((0, 0.0), (1, 0.05), (2, 0.5))   # identity, exp(-0.05 |k|), |k|^-1


def case(name, op, N, B, H, **more):
    c = dict(name=name, op=op, N=N, B=B, H=H, K=50, stride=8, times=3, flow=DECAYING, iters=0, tiles=False)
    c.update(more)
    return c


def listed():
    return [
        # one W(k) map of a small field: the smallest call, three launches
        case("precondition 64", "precondition", 64, 1, 0),
        # the small configuration c0: 64^2, 200 steps, probes at the final time, checkpoints every 50
        case("gradient 64 c0", "gradient", 64, 1, 200, stride=4, times=1),
        # a few small members with a ragged last segment, as the parity suite and small studies run them
        case("gradient 32 x 7", "gradient", 32, 7, 33, K=8, stride=4),
        # a training-style cost behind autograd on the server's smallest grid, segments recomputed
        case("autograd 128 x 5", "autograd", 128, 5, 50, K=7, times=5),
        # configuration c1: one 256^2 member, five observation times, checkpoints every 50
        case("gradient 256 c1", "gradient", 256, 1, 100, times=5),
        # c1's three kernels as one batched 4D-Var
        case("assimilate 256 x 3", "assimilate", 256, 3, 40, times=5, iters=3),
        # the README's example: a batched gradient of 64 members without tuning
        case("gradient 256 x 64", "gradient", 256, 64, 20),
        # the ensemble benchmark: impulse response of 64 members with shell energies, tuned tiles, whole tape
        case("impulse 256 x 64 tuned", "impulse", 256, 64, 40, tiles=True),
        # configuration c2: one 512^2 Kolmogorov member observed through the window
        case("gradient 512 c2", "gradient", 512, 1, 40, K=40, stride=16, times=5, flow=KOLMOGOROV),
        # a truth run with observations on the largest grid
        case("forward 1024", "forward", 1024, 1, 30, stride=16, times=5),
        # served requests: three 1024^2 problems with their own horizons and kernels in one batch
        case("members 1024 x 3 tuned", "members", 1024, 3, 16, stride=8, times=5, iters=1, tiles=True),
        # served requests on the smallest grid of the server's mix, a full batch of eight
        case("members 128 x 8 tuned", "members", 128, 8, 50, stride=4, times=5, iters=2, tiles=True),
    ]


MOST_POINT_STEPS = 64 * 256 * 256 * 40   # of the largest listed case


def draw(rng):
    op = rng.choice(("gradient", "gradient", "forward", "impulse", "autograd", "assimilate", "members",
                     "precondition"))
    N = rng.choice((16, 32, 64, 128, 256, 512, 1024))
    H = 0 if op == "precondition" else int(round(math.exp(rng.uniform(math.log(5), math.log(60)))))
    iters = rng.randint(1, 2) if op in ("assimilate", "members") else 0
    passes = max(1, 3 * iters)
    most = max(1, min(64, MOST_POINT_STEPS // (N * N * max(H, 1) * passes)))
    if op == "members":
        most = min(most, 8)
    B = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    tiles = N >= 128 and rng.random() < 0.4
    c = dict(op=op, N=N, B=B, H=H, K=rng.randint(3, 60), stride=rng.choice((4, 8)), times=rng.choice((1, 3, 5)),
             flow=rng.choice((DECAYING, KOLMOGOROV)), iters=iters, tiles=tiles)
    return c


# ------------------------------------------------------------- problems --

def physics(c):
    N = c["N"]
    if c["flow"] == DECAYING:
        nu = 1e-3 if N < 128 else 1e-4
        dt = 5e-3 if N < 128 else 2e-3 if N <= 256 else 1e-3 if N == 512 else 5e-4
        return dict(nu=nu, mu=0.0, dt=dt, forcing_amp=0.0, forcing_k=4)
    return dict(nu=1.0 / 40, mu=0.1, dt=1e-3 if N <= 512 else 5e-4, forcing_amp=1.0, forcing_k=4)


class Grid:
    """Wavenumbers, band and operators of an N x N periodic box, on the device."""

    def __init__(self, N, device):
        self.N = N
        self.kx = torch.arange(N // 2 + 1, dtype=torch.float64, device=device)[None, :]
        ky = torch.arange(N, dtype=torch.float64, device=device)
        self.ky = torch.where(ky < N / 2, ky, ky - N)[:, None]
        k2 = self.kx ** 2 + self.ky ** 2
        top = (N - 1) // 3
        self.mask = ((self.kx <= top) & (self.ky.abs() <= top) & (k2 > 0)).to(torch.float64)
        self.k2 = k2
        self.ik2 = self.mask / torch.where(k2 > 0, k2, torch.ones_like(k2))
        self.weight = torch.where((self.kx > 0) & (self.kx < N / 2), 2.0, 1.0)   # conjugate half of the real transform

    def phys(self, f):
        return torch.fft.irfft2(f, s=(self.N, self.N))

    def velocity(self, w_hat):
        psi = w_hat * self.ik2
        return self.phys(1j * self.ky * psi), self.phys(-1j * self.kx * psi)


def random_fields(N, B, k0, seed, device="cuda"):
    """Gaussian vorticity fields with energy spectrum k^4 exp(-2 (k/k0)^2), energy 0.5."""
    g = Grid(N, device)
    gen = torch.Generator(device=device).manual_seed(int(seed) % (1 << 62))
    noise = torch.fft.rfft2(torch.randn(B, N, N, dtype=torch.float64, device=device, generator=gen))
    k = torch.sqrt(g.k2)
    amp = torch.sqrt(k ** 5 * torch.exp(-2.0 * (k / k0) ** 2)) / torch.clamp(torch.sqrt(k), min=1.0) * g.mask
    w = noise * amp
    energy = 0.5 * (g.weight * g.ik2 * w.abs() ** 2).sum(dim=(1, 2)) / N ** 4
    return g.phys(w * torch.sqrt(0.5 / energy)[:, None, None])


def spectrum_peak(c):
    N = c["N"]
    return 4.0 if N <= 64 or c["flow"] == KOLMOGOROV else max(4.0, N / 25.0)


def probe_velocities(w, stride, times):
    """Velocities of fields w [B, N, N] at every stride-th point, for each observation time."""
    g = Grid(w.shape[-1], w.device)
    u, v = g.velocity(torch.fft.rfft2(w))
    o = torch.stack([u[:, ::stride, ::stride], v[:, ::stride, ::stride]], dim=1)
    return o[:, None].expand(-1, times, -1, -1, -1).contiguous()


def obs_steps(H, times):
    return [H] if times == 1 else sorted({int(round(i * H / (times - 1))) for i in range(times)})


def member_horizons(c):
    return [max(4, c["H"] - 3 * b) for b in range(c["B"])]   # longest first, as the server orders a batch


def inputs(c, seed):
    N, B = c["N"], c["B"]
    d = {"w0": random_fields(N, B, spectrum_peak(c), 2 * seed + 1)}
    if c["op"] in ("precondition", "impulse"):
        return d
    truth = random_fields(N, B, spectrum_peak(c), 2 * seed + 2)
    d["steps"] = obs_steps(c["H"], c["times"])
    d["values"] = probe_velocities(truth, c["stride"], len(d["steps"]))
    return d


def shells(N):
    return (N - 1) // 3


class State:
    pass


def prepare(c, seed):
    s = State()
    s.c = c
    N, B = c["N"], c["B"]
    s.solver = Solver(N, B, **physics(c))
    if c["tiles"]:
        s.solver.set_tiles(**TILES.get((N, B), TILES[N]))
    d = inputs(c, seed)
    s.w0 = d["w0"]
    s.obs = Observations(c["stride"], d["steps"], d["values"]) if "steps" in d else None
    if c["op"] == "members":
        s.sets = []
        for b, h in enumerate(member_horizons(c)):
            steps = obs_steps(h, c["times"])
            s.sets.append(Observations(c["stride"], steps, d["values"][b:b + 1, :len(steps)].contiguous()))
    s.kernels = [KernelSpec(*KERNELS[b % 3]) for b in range(B)]
    return s


def run(s):
    c, solver = s.c, s.solver
    op, H, K = c["op"], c["H"], c["K"]
    if op == "precondition":
        return solver.precondition(s.w0, KernelSpec(1, 0.05), 0.5)
    if op == "forward":
        return solver.forward(s.w0, H, s.obs, want_obs=True, ckpt_every=K)
    if op == "gradient":
        return solver.adjoint_gradient(s.w0, H, s.obs, ckpt_every=K)
    if op == "impulse":
        return solver.adjoint_impulse(s.w0, H, c["N"] // 2, c["N"] // 2, shells(c["N"]), ckpt_every=K, want_field=True)
    if op == "autograd":
        w = s.w0.detach().requires_grad_(True)
        J = adjoint_cost(w, solver, H, s.obs, K)
        (g,) = torch.autograd.grad(J.sum(), w)
        return J.detach(), g
    if op == "assimilate":
        w, hist, its = solver.assimilate(s.w0, H, s.obs, s.kernels, max_iter=c["iters"], ckpt_every=K)
        return w, torch.tensor(hist, dtype=torch.float64)
    w, hist, its = solver.assimilate_members(s.w0, s.sets, s.kernels, max_iter=c["iters"], ckpt_every=K)
    return w, torch.tensor(hist, dtype=torch.float64)


def work(c):
    """Inputs read and outputs written once; the real 2D transforms that a pseudo-spectral
    right-hand side (four: two velocities there, two products back) and its adjoint (six)
    need at least, 2.5 N^2 log2(N^2) operations each, for each of four Runge-Kutta stages."""
    N, B, H = c["N"], c["B"], c["H"]
    field = 8.0 * N * N * B
    fft = 2.5 * N * N * math.log2(N * N)
    if c["op"] == "precondition":
        return {"bytes": 2 * field, "flops": B * 2 * fft}
    n = len(obs_steps(H, c["times"])) * 2 * (N // c["stride"]) ** 2 * B * 8.0
    if c["op"] == "forward":
        return {"bytes": 2 * field + 2 * n, "flops": B * H * 4 * 4 * fft}
    if c["op"] == "impulse":
        return {"bytes": 2 * field + 8.0 * B * (H + 1) * shells(N), "flops": B * H * 4 * 10 * fft}
    if c["op"] in ("gradient", "autograd"):
        return {"bytes": 2 * field + n, "flops": B * H * 4 * 10 * fft}
    steps = sum(member_horizons(c)) if c["op"] == "members" else B * H
    # an iteration is a gradient and at least one more forward run
    return {"bytes": 2 * field + n, "flops": steps * 4 * (4 + c["iters"] * 10) * fft}


# ---------------------------------------------------------------- exact --

class Scheme:
    def __init__(self, c, device):
        p = physics(c)
        self.g = g = Grid(c["N"], device)
        self.h = p["dt"]
        lin = -(p["nu"] * g.k2 + p["mu"])
        self.E2, self.E1 = torch.exp(lin * self.h / 2), torch.exp(lin * self.h)
        self.f = torch.zeros(g.N, g.N // 2 + 1, dtype=torch.float64, device=device)
        nf = p["forcing_k"]
        if p["forcing_amp"] != 0.0 and nf <= (g.N - 1) // 3:
            self.f[nf, 0] = self.f[g.N - nf, 0] = -p["forcing_amp"] * nf * 0.5 * g.N * g.N

    def rhs(self, w):
        g = self.g
        u, v = g.velocity(w)
        return self.f - g.mask * torch.fft.rfft2(u * g.phys(1j * g.kx * w) + v * g.phys(1j * g.ky * w))

    def step(self, field):
        """One Lawson RK4 step of the field's band part, physical to physical."""
        h, E1, E2 = self.h, self.E1, self.E2
        w = self.g.mask * torch.fft.rfft2(field)
        a = self.rhs(w)
        b = self.rhs(E2 * (w + h / 2 * a))
        c = self.rhs(E2 * w + h / 2 * b)
        d = self.rhs(E1 * w + h * E2 * c)
        return self.g.phys(E1 * w + h / 6 * (E1 * a + 2 * E2 * (b + c) + d))

    def band(self, field):
        return self.g.phys(self.g.mask * torch.fft.rfft2(field))

    def observe(self, field, stride):
        u, v = self.g.velocity(self.g.mask * torch.fft.rfft2(field))
        return torch.stack([u[:, ::stride, ::stride], v[:, ::stride, ::stride]], dim=1)

    def pull(self, fn, at, cotangent):
        x = at.detach().requires_grad_(True)
        with torch.enable_grad():
            y = fn(x)
        (gx,) = torch.autograd.grad(y, x, cotangent)
        return gx


def exact(c, seed):
    op, N, H = c["op"], c["N"], c["H"]
    if op in ("assimilate", "members"):
        return None   # an optimiser's path: its gradients and costs are the other cases'
    with torch.no_grad():
        d = inputs(c, seed)
        w0 = d["w0"]
        sch = Scheme(c, w0.device)
        g = sch.g
        if op == "precondition":
            m = g.mask * torch.sqrt(g.k2 * torch.exp(-0.05 * torch.sqrt(g.k2)))
            return g.phys(m * torch.fft.rfft2(w0))
        path = [sch.band(w0)]
        for _ in range(H):
            path.append(sch.step(path[-1]))
        if op == "impulse":
            spot = torch.zeros(c["B"], 2, N, N, dtype=torch.float64, device=w0.device)
            spot[:, 0, N // 2, N // 2] = 1.0
            lam = sch.pull(lambda x: sch.observe(x, 1), path[H], spot)
            shell = torch.floor(torch.sqrt(g.k2) + 1e-9).to(torch.int64)
            rows = []
            for n in range(H, -1, -1):
                e = 0.5 * g.weight * g.k2 * (g.mask * torch.fft.rfft2(lam)).abs() ** 2 / float(N) ** 4
                rows.append(torch.stack([(e * (shell == k)).sum(dim=(1, 2)) for k in range(1, shells(N) + 1)], dim=1))
                if n > 0:
                    lam = sch.pull(sch.step, path[n - 1], lam)
            return torch.stack(rows, dim=1), sch.band(lam)
        steps, values = d["steps"], d["values"]
        seen = [sch.observe(path[n], c["stride"]) for n in steps]
        off = [o - values[:, i] for i, o in enumerate(seen)]
        J = sum(0.5 * (r ** 2).sum(dim=(1, 2, 3)) for r in off)
        if op == "forward":
            return {"omega_T": path[H], "J": J, "obs": torch.stack(seen, dim=1)}
        lam = torch.zeros_like(w0)
        for n in range(H, -1, -1):
            if n < H:
                lam = sch.pull(sch.step, path[n], lam)
            if n in steps:
                lam = lam + sch.pull(lambda x: sch.observe(x, c["stride"]), path[n], off[steps.index(n)])
        return J, sch.band(lam)
