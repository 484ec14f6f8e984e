"""GPU parity of the one-workgroup 1D engine at every line length it takes (128 to
8192 points, each its own radix plan, thread count and exchange scheme) and at the
longest line of the short-line path beside it (64): FP64 and mixed solves from a
zero guess and from a guess, the right-hand side, RK4 steps and linearly implicit
steps of two and three levels, against the oracle."""
import numpy as np
import pytest

from oracle import linimp as L
from oracle import operators as op
from oracle import rhs as orhs
from oracle import stepping as ost
from paper_2506_16045_amd import inputs as I

pytestmark = pytest.mark.gpu

SIZES = (64, 128, 256, 512, 1024, 2048, 4096, 8192)
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def ctx():
    from paper_2506_16045_amd import sgn
    return sgn.Context(0)


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _problem(n):
    """Bathymetry of one Gaussian bump and a solitary wave, spacing at most 0.3125."""
    g = I.grid1d(n, min(400.0, 0.3125 * n))
    x = I.coords(g)
    h = 1.0 - 0.4 * np.exp(-((x - 0.55 * g.Lx) / (0.06 * g.Lx)) ** 2)
    eta_s, u = I.solitary_wave(g, 1.0, 0.25, 0.4 * g.Lx)
    gh, flat = op.bathy_gradient(h, g)
    return g, h, h + (eta_s - 1.0), u, gh, flat


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solves_at_every_length(ctx, n, precision):
    from paper_2506_16045_amd import sgn
    g, h, eta, u, gh, flat = _problem(n)
    u = u + 0.01 * np.random.default_rng(n).standard_normal((1, n))   # every mode present
    b = op.apply_G(eta, gh, u, g)
    tol = 1e-11
    opts = dict(tol=tol, max_iter=3000, max_outer=40, precision=sgn.MIXED if precision == "mixed" else sgn.FP64)
    for guess in (None, u + 1e-3 * np.random.default_rng(n + 1).standard_normal((1, n))):
        x = None if guess is None else _t(guess)
        x, res = ctx.krylov_solve(g, _t(eta), _t(gh), _t(b), x, opts=sgn.solve_opts(x0_is_guess=guess is not None, **opts))
        x = x.cpu().numpy()
        assert res.converged and res.relres <= tol
        # the solver's own residual drifts from the true one by rounding only: each application of G
        # rounds at eps times its largest term, the second derivative's (symbol k^2 eta^3 / 3)
        kmax = np.pi * n / g.Lx
        floor = 64 * EPS * (1.0 + kmax ** 2 * eta.max() ** 3 / 3.0) * np.linalg.norm(u)
        r = np.linalg.norm(b - op.apply_G(eta, gh, x, g))
        assert r <= 2.0 * tol * np.linalg.norm(b) + floor
        assert np.linalg.norm(x - u) <= 1.1 * (r + floor) / eta.min()   # |G^{-1}| <= 1 / eta_min


@pytest.mark.parametrize("n", SIZES)
def test_right_hand_side_at_every_length(ctx, n):
    g, h, eta, u, gh, flat = _problem(n)
    e_t, U_t = ctx.rhs(g, _t(eta), _t(h), _t(gh), _t(u))
    e_r, U_r = orhs.rhs(eta, u, h, gh, g)
    # rounding of the products, amplified by the derivatives: one of eta u, three in
    # (eta^3/3 u u_xx)_x
    kmax = np.pi * n / g.Lx
    s = np.sqrt(n)
    assert np.linalg.norm(e_t.cpu().numpy() - e_r) <= 16 * EPS * s * (1.0 + kmax) * np.max(np.abs(eta * u[0]))
    top = np.max(eta ** 3 / 3.0 * u[0] ** 2) * (1.0 + kmax ** 3) + np.max(eta) ** 2 * (1.0 + kmax)
    assert np.linalg.norm(U_t.cpu().numpy() - U_r) <= 16 * EPS * s * top


@pytest.mark.parametrize("n", SIZES)
def test_rk4_at_every_length(ctx, n):
    from paper_2506_16045_amd import sgn
    g, h, eta, u, gh, flat = _problem(n)
    tol, dt, steps = 1e-12, 0.01, 2
    pb = ost.Problem.from_h(g, h, tol=tol)
    U = pb.G(eta, u)
    ref = ost.run_rk4(pb, eta, U, u, dt, steps)
    e, Ud, v = _t(eta), _t(U), _t(u)
    st = sgn.State(ctx, g, _t(h), _t(gh), bool(flat), e, Ud, v)
    info = st.step_rk4(dt, steps, sgn.solve_opts(tol=tol, max_iter=3000))
    assert info.converged and info.solves == 4 * steps
    for a, r in zip((e, Ud, v), ref):
        assert np.linalg.norm(a.cpu().numpy() - r) <= 1e-10 * np.linalg.norm(r)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("scheme", ["sbdf2", "linimp3"])
def test_linearly_implicit_steps_at_every_length(ctx, n, scheme):
    from paper_2506_16045_amd import sgn
    g, h, eta, u, gh, flat = _problem(n)
    tol, dt, steps = 1e-12, 0.01, 6
    pb = ost.Problem.from_h(g, h, tol=tol)
    U = pb.G(eta, u)
    e, Ud, v = _t(eta), _t(U), _t(u)
    st = sgn.State(ctx, g, _t(h), _t(gh), bool(flat), e, Ud, v)
    opts = sgn.solve_opts(tol=tol, max_iter=3000)
    if scheme == "sbdf2":
        ref = ost.run_sbdf2(pb, eta, U, u, dt, steps)
        for k in (2, steps - 2):   # a history carried over calls
            st.step_linimp(dt, k, None, opts)
    else:
        r, th = 0.6, 0.9
        ref = L.run_linimp(pb, L.sbdf3r(r), eta, U, u, dt, steps, theta=th)
        for k in (3, steps - 3):
            st.step_linimp3(r, th, dt, k, None, opts)
    for a, b in zip((e, Ud, v), ref):
        assert np.linalg.norm(a.cpu().numpy() - b) <= 1e-10 * np.linalg.norm(b)
    st.close()
