"""Lines that one wave holds (64, 128 and 256 points: the waves past the first wait, and at
128 points half of the first repeats the work of the other half) in launches beside lines
that need the whole workgroup: batched solves and RK4 runs, FP64 and mixed, bit for bit
as alone and against the oracle."""
import numpy as np
import pytest

from oracle import operators as op
from oracle import stepping as ost
from paper_2506_16045_amd import inputs as I

pytestmark = pytest.mark.gpu

SIZES = (2, 64, 128, 256, 512, 2048, 8192)
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def ctx():
    from paper_2506_16045_amd import sgn
    return sgn.Context(0)


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _lines(sizes):
    """Seeded smooth lines, spacing 0.25: grid, h, eta, u, u with every mode, h_x, b = G of that."""
    out = []
    for i, n in enumerate(sizes):
        g = I.grid1d(n, 0.25 * n)
        rng = np.random.default_rng(100 * i + n)
        ph = 2 * np.pi * np.arange(n) / n + rng.uniform(0, 6)
        h = 1.0 - 0.2 * np.cos(ph) - 0.1 * np.sin(2 * ph)
        eta = h + 0.1 * np.sin(ph + 1.0)
        u = 0.2 * np.cos(ph + 0.5)[None]
        noisy = u + 0.01 * rng.standard_normal((1, n))
        gh, _ = op.bathy_gradient(h, g)
        out.append(dict(g=g, h=h, eta=eta, u=u, noisy=noisy, gh=gh, b=op.apply_G(eta, gh, noisy, g)))
    return out


def _cat(lines, key):
    return _t(np.concatenate([np.ravel(s[key]) for s in lines]))


def _split(t, lines):
    a, at = t.cpu().numpy(), np.cumsum([0] + [s["g"].nx for s in lines])
    return [a[at[i]:at[i + 1]] for i in range(len(lines))]


def _mix(lines):
    order = list(range(len(lines))) * 3
    np.random.default_rng(1).shuffle(order)
    return order


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solves(ctx, precision):
    from paper_2506_16045_amd import sgn
    lines, tol = _lines(SIZES), 1e-11
    opts = sgn.solve_opts(tol=tol, max_iter=3000, max_outer=40, precision=sgn.MIXED if precision == "mixed" else sgn.FP64)

    def run(some):
        u, res, st = ctx.batch_solve([s["g"].nx for s in some], [s["g"].Lx for s in some], _cat(some, "eta"), _cat(some, "gh"),
                                     _cat(some, "b"), opts=opts)
        assert st == sgn.OK and all(r.converged for r in res)
        return _split(u, some)

    alone = [run([s])[0] for s in lines]
    order = _mix(lines)
    for i, u in zip(order, run([lines[i] for i in order])):
        assert np.array_equal(u, alone[i]), lines[i]["g"].nx
    for s, u in zip(lines, alone):
        # the solver's own residual drifts from the true one by rounding only: each application of G
        # rounds at eps times its largest term, the second derivative's (symbol k^2 eta^3 / 3)
        kmax = np.pi * s["g"].nx / s["g"].Lx
        floor = 64 * EPS * (1.0 + kmax ** 2 * s["eta"].max() ** 3 / 3.0) * np.linalg.norm(s["noisy"])
        r = np.linalg.norm(s["b"] - op.apply_G(s["eta"], s["gh"], u[None], s["g"]))
        assert r <= 2.0 * tol * np.linalg.norm(s["b"]) + floor


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_rk4_runs(ctx, precision):
    from paper_2506_16045_amd import sgn
    lines, tol, dt, steps = _lines(SIZES[1:]), 1e-12, 0.01, 3
    opts = sgn.solve_opts(tol=tol, max_iter=3000, max_outer=40, precision=sgn.MIXED if precision == "mixed" else sgn.FP64)

    def run(some):
        eta, u = _cat(some, "eta"), _cat(some, "u")
        _, _, st = ctx.batch_step_rk4([s["g"].nx for s in some], [s["g"].Lx for s in some], dt, steps, _cat(some, "h"), eta, u, opts)
        assert st == sgn.OK
        return list(zip(_split(eta, some), _split(u, some)))

    alone = [run([s])[0] for s in lines]
    order = _mix(lines)
    for i, got in zip(order, run([lines[i] for i in order])):
        assert all(np.array_equal(a, b) for a, b in zip(got, alone[i])), lines[i]["g"].nx
    for s, (eta, u) in zip(lines, alone):
        pb = ost.Problem.from_h(s["g"], s["h"], tol=tol)
        e_r, _, u_r = ost.run_rk4(pb, s["eta"], pb.G(s["eta"], s["u"]), s["u"], dt, steps)
        assert np.linalg.norm(eta - e_r) <= 1e-10 * np.linalg.norm(e_r)
        assert np.linalg.norm(u - u_r) <= 1e-10 * np.linalg.norm(u_r)
