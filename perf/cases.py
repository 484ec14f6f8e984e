"""The work that programs have this framework do, as cases that can be timed and checked.

A case is a dict of plain values.  `prepare` makes what a program has in hand before the call (seeded
inputs on the GPU, the context, a bound time-stepping state), `run` is one pass through the public
entry points, `exact` the same outputs from plain torch in 64 bits without this package, and `work`
the bytes and operations that a pass cannot do without.

Inputs follow the repository's workloads: depth 1 over one to three Gaussian bumps, a solitary wave
of amplitude 0.1 to 0.3 as the free surface, its velocity as the initial data or (solves) as the
solution the right-hand side is formed from.  Domains are those of the workloads at their sizes
(400 long in 1D, 200 x 200 in 2D, the closed basin 200 x 200) and shrink with the grid below that, so
that the wave stays resolved; dt = min(0.02, dx / 2), tol 1e-10 (1e-12 for the 1D flat run).

Stepping cases advance their state in place, as a program's time loop does: a pass is a few steps of
a longer run.  Kinds:

  solve      one constraint solve G u = b from a zero guess (a served solve request)
  rk4        classical RK4 steps, one Krylov solve per stage
  sbdf2      linearly implicit steps (one constant-coefficient solve per step)
  batch      many independent 1D solves of ragged sizes in one call
  batch_rk4  many independent 1D RK4 runs of ragged sizes in one call
"""
import math
import random

import numpy as np
import torch

SIZES_1D = (256, 512, 1024, 2048, 4096, 8192, 16384)
BATCH_SIZES = (512, 1024, 2048, 4096, 8192)


def listed():
    one = dict(dim=1, ny=1, bc="periodic", precision="fp64", dealias=False)
    two = dict(dim=2, bc="periodic", precision="fp64", dealias=False)
    return [
        # the smallest call: one 1D solve, all latency
        dict(one, name="solve 1d 1024", kind="solve", nx=1024),
        # the flat solitary wave of the 1D workload (N = 256 on L = 80, tol 1e-12)
        dict(one, name="rk4 1d 256 flat", kind="rk4", nx=256, steps=20, flat=True),
        # the 1D shelf's size under its own scheme
        dict(one, name="sbdf2 1d 4096", kind="sbdf2", nx=4096, steps=20),
        # the longest 1D grid (coefficient studies, served 1D requests)
        dict(one, name="solve 1d 16384", kind="solve", nx=16384),
        # the batched ensemble: 512 ragged systems in one call
        dict(name="batch 512 mixed", kind="batch", count=512, precision="mixed", mix=4),
        # served 1D RK4 requests gathered into one call
        dict(name="batch rk4 96", kind="batch_rk4", count=96, steps=5, precision="fp64", mix=5),
        # a small 2D grid, wider than high: launches and their gaps
        dict(two, name="rk4 2d 256x128", kind="rk4", nx=256, ny=128, steps=4),
        # the 2D workload in mixed precision at a served size
        dict(two, name="rk4 2d 512 mixed", kind="rk4", nx=512, ny=512, steps=4, precision="mixed"),
        # the 2D workload (1024 x 1024 on 200 x 200)
        dict(two, name="rk4 2d 1024", kind="rk4", nx=1024, ny=1024, steps=2),
        # the same with the de-aliased right-hand side (padded to 2048 x 2048)
        dict(two, name="rk4 2d 1024 dealiased", kind="rk4", nx=1024, ny=1024, steps=1, dealias=True),
        # the closed basin
        dict(two, name="solve walls 512", kind="solve", nx=512, ny=512, bc="walls"),
        # the largest 2D grid
        dict(two, name="rk4 2d 4096x1024", kind="rk4", nx=4096, ny=1024, steps=2),
    ]


def draw(rng):
    kind = rng.choice(["solve 1d", "rk4 1d", "sbdf2 1d", "batch", "batch_rk4", "rk4 2d", "rk4 2d", "solve 2d", "walls"])
    precision = rng.choice(["fp64", "mixed"])
    one = dict(dim=1, ny=1, bc="periodic", precision=precision, dealias=False)
    if kind == "solve 1d":
        return dict(one, kind="solve", nx=rng.choice(SIZES_1D))
    if kind == "rk4 1d":
        return dict(one, kind="rk4", nx=rng.choice(SIZES_1D), steps=rng.randint(2, 6))
    if kind == "sbdf2 1d":
        return dict(one, kind="sbdf2", nx=rng.choice(SIZES_1D), steps=rng.randint(5, 25), precision="fp64")
    if kind == "batch":
        return dict(kind="batch", count=int(2 ** rng.uniform(3, 9)), precision=precision, mix=rng.randrange(1 << 20))
    if kind == "batch_rk4":
        return dict(kind="batch_rk4", count=int(2 ** rng.uniform(3, 7)), steps=rng.randint(2, 6), precision=precision,
                    mix=rng.randrange(1 << 20))
    if kind == "walls":
        return dict(dim=2, kind=rng.choice(["solve", "rk4"]), nx=rng.choice([64, 128, 256, 512, 1024]), ny=rng.choice([64, 128, 256, 512]),
                    bc="walls", precision="fp64", dealias=False, steps=rng.randint(1, 3))
    nx, ny = rng.choice([128, 256, 512, 1024, 2048, 4096]), rng.choice([64, 128, 256, 512, 1024])
    two = dict(dim=2, nx=nx, ny=ny, bc="periodic", precision=precision, dealias=False)
    if kind == "solve 2d":
        return dict(two, kind="solve")
    if nx <= 1024 and rng.random() < 0.3:
        return dict(two, kind="rk4", steps=1, dealias=True, precision="fp64")
    return dict(two, kind="rk4", steps=1 if nx * ny > 1 << 20 else rng.randint(1, 3))


# ---- grids and inputs -----------------------------------------------------------------------------

def extent(dim, n):
    """The domain's length along an axis of n points."""
    return min(400.0, 0.3125 * n) if dim == 1 else 200.0 * min(1.0, n / 512.0)


def time_step(dim, nx):
    return min(0.02, 0.5 * extent(dim, nx) / nx)


def coordinates(dim, nx, ny, walls):
    off = 0.5 if walls else 0.0
    x = (torch.arange(nx, dtype=torch.float64, device="cuda") + off) * (extent(dim, nx) / nx)
    y = (torch.arange(ny, dtype=torch.float64, device="cuda") + off) * (extent(dim, ny) / ny)
    return x, y


def wrapped(x, x0, length):
    return torch.remainder(x - x0 + 0.5 * length, length) - 0.5 * length


def make_fields(dim, nx, ny, walls, flat, count, rng):
    """(h, eta, u) of `count` problems: h, eta (count, ny, nx), u (count, dim, ny, nx)."""
    lx, ly = extent(dim, nx), extent(dim, ny)
    x, y = coordinates(dim, nx, ny, walls)
    hs, etas, us = [], [], []
    for _ in range(count):
        h = torch.ones(ny, nx, dtype=torch.float64, device="cuda")
        bumps = 0 if flat else rng.integers(1, 4)
        for _ in range(bumps):
            height, width = rng.uniform(0.1, 0.5) / bumps, rng.uniform(0.04, 0.08) * min(lx, ly if dim == 2 else lx)
            width = min(width, 15.0)
            cx, cy = rng.uniform(0.3, 0.7) * lx, rng.uniform(0.3, 0.7) * ly
            r2 = wrapped(x, cx, lx)[None, :] ** 2
            if dim == 2:
                r2 = r2 + wrapped(y, cy, ly)[:, None] ** 2
            h = h - height * torch.exp(-r2 / width ** 2)
        a = rng.uniform(0.1, 0.3)
        if walls:
            cx, cy = rng.uniform(0.3, 0.7) * lx, rng.uniform(0.3, 0.7) * ly
            w = 0.075 * min(lx, ly)
            eta = h + a * torch.exp(-((x - cx)[None, :] ** 2 + (y - cy)[:, None] ** 2) / w ** 2)
            sx, sy = math.pi * x / lx, math.pi * y / ly
            u = torch.stack([a * torch.cos(sy)[:, None] * (torch.sin(sx) * (1.0 + 0.2 * torch.sin(3.0 * sx)))[None, :],
                             a * torch.sin(2.0 * sy)[:, None] * torch.cos(sx)[None, :]])
        else:
            c = math.sqrt(1.0 + a)
            zeta = a / torch.cosh(math.sqrt(3.0 * a) / (2.0 * c) * wrapped(x, rng.uniform(0.0, 1.0) * lx, lx)) ** 2
            eta = h + zeta[None, :]
            u = torch.stack([c * zeta[None, :] / eta] + [torch.zeros_like(eta)] * (dim - 1))
        hs.append(h)
        etas.append(eta)
        us.append(u)
    return torch.stack(hs), torch.stack(etas), torch.stack(us)


def fields_of(case, seed):
    return make_fields(case["dim"], case["nx"], case["ny"], case["bc"] == "walls", case.get("flat", False), 1,
                       np.random.default_rng([seed, 17]))


def batch_groups(case, seed):
    """(sizes in system order, {size: (systems, h, eta, u)})."""
    pick = random.Random(case["mix"])
    sizes = [pick.choice(BATCH_SIZES) for _ in range(case["count"])]
    groups = {}
    for n in sorted(set(sizes)):
        at = [i for i, s in enumerate(sizes) if s == n]
        groups[n] = (at, *make_fields(1, n, 1, False, False, len(at), np.random.default_rng([seed, n])))
    return sizes, groups


def packed(sizes, groups, of):
    """One packed tensor in system order of a field per group (of(size) -> (systems, n))."""
    rows = [None] * len(sizes)
    for n, (at, *_) in groups.items():
        f = of(n).reshape(len(at), n)
        for k, i in enumerate(at):
            rows[i] = f[k]
    return torch.cat(rows)


def tolerance(case):
    return 1e-12 if case.get("flat") else 1e-10


# ---- the framework's side ---------------------------------------------------------------------------

def prepare(case, seed):
    from paper_2506_16045_amd import inputs, sgn

    ctx = sgn.Context(0)
    mixed = case["precision"] == "mixed"
    opts = sgn.solve_opts(tol=tolerance(case), precision=sgn.MIXED if mixed else sgn.FP64, max_iter=5000, max_outer=40)
    if case["kind"] in ("batch", "batch_rk4"):
        sizes, groups = batch_groups(case, seed)
        state = dict(ctx=ctx, opts=opts, sizes=np.asarray(sizes, dtype=np.int32), periods=np.asarray([extent(1, n) for n in sizes]),
                     eta=packed(sizes, groups, lambda n: groups[n][2]))
        if case["kind"] == "batch":
            systems = {n: Plain(1, n, 1) for n in groups}
            slope = {n: systems[n].grad(groups[n][1]) for n in groups}
            state["grad_h"] = packed(sizes, groups, lambda n: slope[n])
            state["rhs"] = packed(sizes, groups, lambda n: systems[n].constraint(groups[n][2], slope[n], groups[n][3]))
            state["u"] = torch.zeros_like(state["eta"])
            return dict(state, call="batch")
        state["h"] = packed(sizes, groups, lambda n: groups[n][1])
        state["u"] = packed(sizes, groups, lambda n: groups[n][3])
        state["dts"] = np.asarray([time_step(1, n) for n in sizes])
        return dict(state, call="batch_rk4", steps=case["steps"])
    walls = case["bc"] == "walls"
    nx, ny, dim = case["nx"], case["ny"], case["dim"]
    lx, ly = extent(dim, nx), extent(dim, ny)
    if walls:
        g = inputs.grid2d_walls(nx, ny, lx, ly)
    else:
        g = inputs.grid1d(nx, lx) if dim == 1 else inputs.grid2d(nx, ny, lx, ly)
    h, eta, u = fields_of(case, seed)
    shape = (nx,) if dim == 1 else (ny, nx)
    h1, eta1, u1 = (f[0].reshape(s).contiguous() for f, s in ((h, shape), (eta, shape), (u, (dim,) + shape)))
    grad_h, flat = ctx.bathy_prepare(g, h1)
    if case["kind"] == "solve":
        rhs = right_side(case, h, eta, u)[0].reshape((dim,) + shape).contiguous()
        return dict(call="solve", ctx=ctx, opts=opts, g=g, eta=eta1, grad_h=grad_h, rhs=rhs, u=torch.zeros_like(u1))
    U1 = ctx.apply_constraint(g, eta1, grad_h, u1)
    st = sgn.State(ctx, g, h1, grad_h, flat, eta1, U1, u1)
    if case["dealias"]:
        st.set_dealias(True)
    return dict(call=case["kind"], st=st, opts=opts, dt=time_step(dim, nx), steps=case["steps"])


def run(state):
    call = state["call"]
    if call == "solve":
        u, _ = state["ctx"].krylov_solve(state["g"], state["eta"], state["grad_h"], state["rhs"], state["u"], opts=state["opts"])
        return {"u": u}
    if call == "batch":
        u, _, _ = state["ctx"].batch_solve(state["sizes"], state["periods"], state["eta"], state["grad_h"], state["rhs"], state["u"],
                                           opts=state["opts"])
        return {"u": u}
    if call == "batch_rk4":
        state["ctx"].batch_step_rk4(state["sizes"], state["periods"], state["dts"], state["steps"], state["h"], state["eta"], state["u"],
                                    opts=state["opts"])
        return {"eta": state["eta"], "u": state["u"]}
    st = state["st"]
    if call == "rk4":
        st.step_rk4(state["dt"], state["steps"], state["opts"])
    else:
        st.step_linimp(state["dt"], state["steps"], opts=state["opts"])
    return {"eta": st.eta, "U": st.U, "u": st.u}


# ---- the same in plain torch, 64 bits -----------------------------------------------------------------

LAMBDA = (4.0 + math.sqrt(13.0)) / 6.0


class Plain:
    """Spectral operators on `count` periodic problems at once: scalars (count, ny, nx), vectors (count, dim, ny, nx)."""

    def __init__(self, dim, nx, ny, lx=None, ly=None):
        self.dim, self.nx, self.ny = dim, nx, ny
        self.lx = extent(dim, nx) if lx is None else lx
        self.ly = extent(dim, ny) if ly is None else ly
        kx = torch.arange(nx // 2 + 1, dtype=torch.float64, device="cuda")
        kx[nx // 2] = 0.0
        ky = torch.fft.fftfreq(ny, 1.0 / ny, dtype=torch.float64, device="cuda")
        if ny % 2 == 0:
            ky[ny // 2] = 0.0
        self.kx = (2.0 * math.pi / self.lx) * kx[None, :]
        self.ky = (2.0 * math.pi / self.ly) * ky[:, None]

    def to(self, f):
        return torch.fft.rfft2(f) if self.dim == 2 else torch.fft.rfft(f)

    def back(self, F):
        return torch.fft.irfft2(F, s=(self.ny, self.nx)) if self.dim == 2 else torch.fft.irfft(F, n=self.nx)

    def grad(self, f):
        F = self.to(f)
        return torch.stack([self.back(1j * k * F) for k in (self.kx, self.ky)[: self.dim]], dim=1)

    def div(self, u):
        U = self.to(u)
        return self.back(sum(1j * (self.kx, self.ky)[c] * U[:, c] for c in range(self.dim)))

    def constraint(self, eta, gh, u):
        """G u = eta u - grad(eta^3/3 div u + eta^2/2 gh.u) + eta^2/2 gh div u + eta gh (gh.u)."""
        d, b = self.div(u), (gh * u).sum(1)
        return eta[:, None] * u - self.grad(eta ** 3 / 3.0 * d + eta ** 2 / 2.0 * b) + gh * (eta ** 2 / 2.0 * d + eta * b)[:, None]

    def coefficients(self, eta, gh, flat):
        top = eta.amax((1, 2))
        if flat:
            return top, top ** 3 / 3.0
        return (eta + LAMBDA * eta * (gh * gh).sum(1)).amax((1, 2)), LAMBDA * top ** 3

    def inverse(self, sigma, alpha, r):
        """(sigma - alpha grad div)^{-1} r, mode by mode, along the wavevector and across it."""
        R = self.to(r)
        k = (self.kx, self.ky)[: self.dim]
        k2 = sum(q * q for q in k)
        s, a = sigma[:, None, None], alpha[:, None, None]
        along = sum(k[c] * R[:, c] for c in range(self.dim)) / torch.where(k2 > 0, k2, 1.0)
        part = torch.stack([q * along for q in k], dim=1)
        return self.back((R - part) / s[:, None] + part / (s + a * k2)[:, None])

    def solve(self, eta, gh, flat, b, u):
        """Conjugate gradients from u, each problem to a relative residual of 1e-14 or until it stops falling."""
        sigma, alpha = self.coefficients(eta, gh, flat)

        def dot(p, q):
            return (p * q).sum((1, 2, 3))[:, None, None, None]

        target = 1e-28 * dot(b, b)
        r = b - self.constraint(eta, gh, u)
        z = self.inverse(sigma, alpha, r)
        p, rho, best, stale = z, dot(r, z), dot(r, r), 0
        while bool((best > target).any()) and stale < 8:
            q = self.constraint(eta, gh, p)
            pq = dot(p, q)
            live = (dot(r, r) > target) & (pq > 0)
            step = torch.where(live, rho / torch.where(pq > 0, pq, 1.0), 0.0)
            u, r = u + step * p, r - step * q
            z = self.inverse(sigma, alpha, r)
            new, rr = dot(r, z), dot(r, r)
            p = z + torch.where(rho > 0, new / torch.where(rho > 0, rho, 1.0), 0.0) * p
            rho = new
            stale = stale + 1 if not bool((rr < 0.9 * best).any()) else 0
            best = torch.minimum(best, rr)
        return u

    def slopes(self, eta, h, gh, u):
        """(eta_t, U_t)."""
        e = eta
        d, m, b = self.div(u), self.div(e[:, None] * u), (gh * u).sum(1)
        P = (u * self.grad(d)).sum(1) - d * d
        Q = (u * self.grad(b)).sum(1)
        S = e ** 3 / 3.0 * P + e ** 2 * m * d + e ** 2 / 2.0 * Q + e * m * b
        T = e ** 2 / 2.0 * P + e * m * d + e * Q + m * b
        flux = torch.stack([self.div(e[:, None] * u[:, c : c + 1] * u) for c in range(self.dim)], dim=1)
        return -m, -e[:, None] * self.grad(e - h) - flux + self.grad(S) - gh * T[:, None]

    def moved(self, f, other):
        """f on another grid of the same domain, its modes below the coarser grid's Nyquist kept."""
        F = self.to(f)
        G = torch.zeros(f.shape[:-2] + (other.ny, other.nx // 2 + 1), dtype=F.dtype, device=F.device)
        mx, my = min(self.nx, other.nx) // 2, min(self.ny, other.ny) // 2
        if my == 0:
            G[..., :mx] = F[..., :mx]
        else:
            G[..., :my, :mx] = F[..., :my, :mx]
            G[..., other.ny - my + 1 :, :mx] = F[..., self.ny - my + 1 :, :mx]
        return other.back(G) * (other.nx * other.ny / (self.nx * self.ny))


def mirrored(f, odd_x, odd_y):
    """A field of the closed basin on the periodic domain of twice the size."""
    f = torch.cat([f, -f.flip(-1) if odd_x else f.flip(-1)], dim=-1)
    return torch.cat([f, -f.flip(-2) if odd_y else f.flip(-2)], dim=-2)


def in_the_open(case, h, eta, u):
    """The operators and fields of the case's problem on a periodic domain."""
    dim, nx, ny = case["dim"], case["nx"], case["ny"]
    if case["bc"] != "walls":
        return Plain(dim, nx, ny), h, eta, u
    twin = Plain(dim, 2 * nx, 2 * ny, 2.0 * extent(dim, nx), 2.0 * extent(dim, ny))
    u = torch.stack([mirrored(u[:, 0], True, False), mirrored(u[:, 1], False, True)], dim=1)
    return twin, mirrored(h, False, False), mirrored(eta, False, False), u


def right_side(case, h, eta, u):
    P, h, eta, u = in_the_open(case, h, eta, u)
    return P.constraint(eta, P.grad(h), u)[..., : case["ny"], : case["nx"]]


def rk4_step(P, f, eta, U, u, gh, flat, dt):
    e1, U1 = f(eta, u)
    ea, Ua = eta + 0.5 * dt * e1, U + 0.5 * dt * U1
    ua = P.solve(ea, gh, flat, Ua, u)
    e2, U2 = f(ea, ua)
    ea, Ua = eta + 0.5 * dt * e2, U + 0.5 * dt * U2
    ua = P.solve(ea, gh, flat, Ua, ua)
    e3, U3 = f(ea, ua)
    ea, Ua = eta + dt * e3, U + dt * U3
    ua = P.solve(ea, gh, flat, Ua, ua)
    e4, U4 = f(ea, ua)
    eta = eta + dt / 6.0 * (e1 + 2.0 * e2 + 2.0 * e3 + e4)
    U = U + dt / 6.0 * (U1 + 2.0 * U2 + 2.0 * U3 + U4)
    return eta, U, P.solve(eta, gh, flat, U, ua)


def stepped(P, kind, h, eta, u, flat, dt, steps, fine=None):
    gh = torch.zeros_like(u) if flat else P.grad(h)
    if fine is None:
        def f(e, v):
            return P.slopes(e, h, gh, v)
    else:
        hf = P.moved(h, fine)
        ghf = fine.grad(hf)

        def f(e, v):
            return tuple(fine.moved(w, P) for w in fine.slopes(P.moved(e, fine), hf, ghf, P.moved(v, fine)))
    U = P.constraint(eta, gh, u)
    if kind != "sbdf2":
        for _ in range(steps):
            eta, U, u = rk4_step(P, f, eta, U, u, gh, flat, dt)
        return eta, U, u
    sigma, alpha = P.coefficients(eta, gh, flat)

    def lagged(e, V, v):
        return sigma[:, None, None, None] * v - alpha[:, None, None, None] * P.grad(P.div(v)) - P.constraint(e, gh, v) + V

    w0, f0, R0 = (eta, U), f(eta, u), lagged(eta, U, u)
    eta, U, u = rk4_step(P, f, eta, U, u, gh, flat, dt)
    for _ in range(steps - 1):
        f1, R1 = f(eta, u), lagged(eta, U, u)
        w1 = (eta, U)
        eta, U = ((2.0 * w1[k] - 0.5 * w0[k] + dt * (2.0 * f1[k] - f0[k])) / 1.5 for k in (0, 1))
        u = P.inverse(sigma, alpha, 2.0 * R1 - R0)
        w0, f0, R0 = w1, f1, R1
    return eta, U, u


def exact(case, seed):
    if case["kind"] in ("batch", "batch_rk4"):
        sizes, groups = batch_groups(case, seed)
        if case["kind"] == "batch":
            return {"u": packed(sizes, groups, lambda n: groups[n][3])}
        done = {n: stepped(Plain(1, n, 1), "rk4", h, eta, u, False, time_step(1, n), case["steps"])
                for n, (_, h, eta, u) in groups.items()}
        return {"eta": packed(sizes, groups, lambda n: done[n][0]), "u": packed(sizes, groups, lambda n: done[n][2])}
    dim, nx, ny = case["dim"], case["nx"], case["ny"]
    shape = (nx,) if dim == 1 else (ny, nx)
    h, eta, u = fields_of(case, seed)
    if case["kind"] == "solve":
        return {"u": u[0].reshape((dim,) + shape)}
    P, h, eta, u = in_the_open(case, h, eta, u)
    fine = Plain(dim, 2 * nx, 2 * ny if dim == 2 else 1, P.lx, P.ly) if case["dealias"] else None
    eta, U, u = (f[0, ..., :ny, :nx] for f in stepped(P, case["kind"], h, eta, u, case.get("flat", False), time_step(dim, nx),
                                                      case["steps"], fine))
    return {"eta": eta.reshape(shape), "U": U.reshape((dim,) + shape), "u": u.reshape((dim,) + shape)}


# ---- what a pass cannot do without -----------------------------------------------------------------

def work(case):
    """Inputs read once and outputs written once; operations of the transforms alone, a real transform of N points at
    2.5 N log2 N.  A Krylov iteration transforms dim + 1 fields each way; solves are counted at 20 iterations from a
    zero guess and 5 inside a stepper, a right-hand side at 6 dim + 4 transforms."""
    dim = case.get("dim", 1)
    if case["kind"] in ("batch", "batch_rk4"):
        pick = random.Random(case["mix"])
        sizes = [pick.choice(BATCH_SIZES) for _ in range(case["count"])]
    else:
        sizes = [case["nx"] * case["ny"]]
    points = sum(sizes)
    transform = sum(2.5 * n * math.log2(n) for n in sizes)
    iteration = 2 * (dim + 1) * transform
    if case["kind"] in ("solve", "batch"):
        return {"bytes": 8.0 * points * (1 + 3 * dim), "flops": 20 * iteration}
    pad = 2 ** dim if case.get("dealias") else 1
    slope = (6 * dim + 4) * transform * pad
    if case["kind"] == "sbdf2":
        return {"bytes": 8.0 * points * (2 + dim + 2 * (1 + 2 * dim)), "flops": case["steps"] * (slope + 2 * iteration)}
    held = 1 + 2 * dim if case["kind"] == "rk4" else 1 + dim
    return {"bytes": 8.0 * points * (1 + dim + 2 * held), "flops": case["steps"] * 4 * (slope + 5 * iteration)}
