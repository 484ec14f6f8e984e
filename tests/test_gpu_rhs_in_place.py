"""The right-hand side written over its own inputs equals the one written elsewhere, bit
for bit, where that has always been so: on 1D lines of up to 8192 points either output
over any input (the short-line path and the one-workgroup engine beside it), on 2D grids
U_t over u (each of the three forms of the inverse row pass); and on the line of 16384
points, whose own pass reads its inputs again after it has stored eta_t."""
import numpy as np
import pytest

from paper_2506_16045_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2506_16045_amd import sgn
    return sgn.Context(0)


def _fields(ctx, nx, ny=1):
    """Grid and (eta, h, grad h, u) on the GPU: seeded, smooth, spacing 0.25."""
    import torch
    g = I.grid1d(nx, 0.25 * nx) if ny == 1 else I.grid2d(nx, ny, 0.25 * nx, 0.25 * ny)
    rng = np.random.default_rng(nx + 3 * ny)
    h = 1.0 + 0.1 * I.random_smooth_field(g, rng)
    eta = h + 0.1 * I.random_smooth_field(g, rng)
    u = 0.2 * np.stack([I.random_smooth_field(g, rng) for _ in range(g.d)])
    h, eta, u = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (h, eta, u))
    return g, eta, h, ctx.bathy_prepare(g, h)[0], u


def _check(ctx, fields, eta_t, U_t):
    """eta_t, U_t: the name of the input each output is written over, or None."""
    import torch
    g, eta, h, gh, u = fields
    ref = ctx.rhs(g, eta, h, gh, u)
    own = dict(eta=eta.clone(), gh=gh.clone(), u=u.clone())
    out = ctx.rhs(g, own["eta"], h, own["gh"], own["u"], own[eta_t].view(eta.shape) if eta_t else None,
                  own[U_t].view(u.shape) if U_t else None)
    for a, b in zip(out, ref):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n", (2, 64, 128, 256, 512, 1024, 2048, 4096, 8192))
def test_lines(ctx, n):
    fields = _fields(ctx, n)
    for eta_t in (None, "eta", "gh", "u"):
        for U_t in (None, "eta", "gh", "u"):
            if eta_t is None or eta_t != U_t:
                _check(ctx, fields, eta_t, U_t)


def test_longest_line(ctx):
    fields = _fields(ctx, 16384)
    for eta_t in (None, "eta", "gh", "u"):
        _check(ctx, fields, eta_t, None)
        if eta_t != "u":
            _check(ctx, fields, eta_t, "u")


@pytest.mark.parametrize("nx,ny", ((8, 8), (512, 16), (1024, 8), (2048, 4), (2048, 512), (4096, 4)))
def test_velocity_on_grids(ctx, nx, ny):
    _check(ctx, _fields(ctx, nx, ny), None, "u")
