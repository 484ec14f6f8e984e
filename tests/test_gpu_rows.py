"""GPU parity of the row and column passes at the edges of their launch rules: rows of
less than one thread group, of one wave, of several rows per wave, of the widest
blocks; columns from two points to the longest; rows that do not fill a block; and the
1D line of 16384 points.  Constraint solves (FP64 and mixed) and the right-hand side
against the oracle."""
import numpy as np
import pytest

from oracle import operators as op
from oracle import rhs as orhs
from paper_2506_16045_amd import inputs as I

pytestmark = pytest.mark.gpu

GRIDS = [(2, 2), (4, 8), (8, 1024), (16, 16), (32, 16), (64, 4), (128, 32), (256, 2), (256, 128), (512, 16),
         (1024, 4), (2048, 2), (2048, 64), (4096, 2), (4096, 32), (16384, 1)]
IDS = [f"{nx}x{ny}" for nx, ny in GRIDS]
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def ctx():
    from paper_2506_16045_amd import sgn
    return sgn.Context(0)


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _problem(nx, ny):
    """Seeded smooth depth and bathymetry, spacing 0.25, velocities with every mode."""
    g = I.grid1d(nx, 0.25 * nx) if ny == 1 else I.grid2d(nx, ny, 0.25 * nx, 0.25 * ny)
    rng = np.random.default_rng(nx + 7 * ny)
    ax = [np.arange(n) / n for n in g.shape]
    ph = 2 * np.pi * sum(np.meshgrid(*ax, indexing="ij"))
    h = 1.0 - 0.2 * np.cos(ph) - 0.1 * np.sin(ph)
    eta = h + 0.1 * np.sin(ph + 1.0)
    u = 0.2 * np.stack([np.cos(ph + c) for c in range(g.d)]) + 0.01 * rng.standard_normal((g.d,) + g.shape)
    gh, _ = op.bathy_gradient(h, g)
    return g, h, eta, u, gh


def _kmax(g):
    return np.pi * max([g.nx / g.Lx] + ([g.ny / g.Ly] if g.d == 2 else []))


@pytest.mark.parametrize("nx,ny", GRIDS, ids=IDS)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solves(ctx, nx, ny, precision):
    from paper_2506_16045_amd import sgn
    print(f"solve {nx}x{ny} {precision}", flush=True)
    g, h, eta, u, gh = _problem(nx, ny)
    b = op.apply_G(eta, gh, u, g)
    tol = 1e-11
    opts = sgn.solve_opts(tol=tol, max_iter=3000, max_outer=40,
                          precision=sgn.MIXED if precision == "mixed" else sgn.FP64)
    x, res = ctx.krylov_solve(g, _t(eta), _t(gh), _t(b), None, opts=opts)
    x = x.cpu().numpy()
    assert res.converged and res.relres <= tol
    # the solver's own residual drifts from the true one by rounding only: each application of G
    # rounds at eps times its largest term, the second derivative's (symbol k^2 eta^3 / 3)
    floor = 64 * EPS * (1.0 + _kmax(g) ** 2 * eta.max() ** 3 / 3.0) * np.linalg.norm(u)
    r = np.linalg.norm(b - op.apply_G(eta, gh, x, g))
    assert r <= 2.0 * tol * np.linalg.norm(b) + floor
    assert np.linalg.norm(x - u) <= 1.1 * (r + floor) / eta.min()   # |G^{-1}| <= 1 / eta_min


@pytest.mark.parametrize("nx,ny", GRIDS, ids=IDS)
def test_right_hand_side(ctx, nx, ny):
    print(f"rhs {nx}x{ny}", flush=True)
    g, h, eta, u, gh = _problem(nx, ny)
    e_t, U_t = ctx.rhs(g, _t(eta), _t(h), _t(gh), _t(u))
    e_r, U_r = orhs.rhs(eta, u, h, gh, g)
    # rounding of the products, amplified by the derivatives: one of eta u, three in
    # (eta^3/3 u u_xx)_x; one such term per axis
    k, s, um = _kmax(g), np.sqrt(nx * ny), np.max(np.abs(u))
    assert np.linalg.norm(e_t.cpu().numpy() - e_r) <= 16 * g.d * EPS * s * (1.0 + k) * eta.max() * um
    top = eta.max() ** 3 / 3.0 * um ** 2 * (1.0 + k ** 3) + eta.max() ** 2 * (1.0 + k)
    assert np.linalg.norm(U_t.cpu().numpy() - U_r) <= 16 * g.d ** 2 * EPS * s * top


# rows of 2048 and 4096 points on enough rows that a block holds two or four of them
# (four at 2048 x 1024): the blocks of 512 and 1024 threads that the grids above do not reach
TALL = [(2048, 512), (2048, 1024), (4096, 512)]


@pytest.mark.parametrize("nx,ny", TALL, ids=[f"{nx}x{ny}" for nx, ny in TALL])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solves_with_several_long_rows_per_block(ctx, nx, ny, precision):
    test_solves(ctx, nx, ny, precision)


@pytest.mark.parametrize("nx,ny", TALL, ids=[f"{nx}x{ny}" for nx, ny in TALL])
def test_right_hand_side_with_several_long_rows_per_block(ctx, nx, ny):
    test_right_hand_side(ctx, nx, ny)
