"""GPU parity of the one-kernel vector-Jacobian product of the implicit stage
at the edges of its tiles: columns shorter than the transposed window, radial
points around the row groups of a thread (32, 64, 96, 128 with 4 |k| per
workgroup; 16, 32, 48, 64 with 8), |k| counts that leave a remainder in the
last tile, heated and isothermal, and the kernel sequence past 128 points.
The oracle is the forward stage, which is affine: <w, S(x) - S(0)> and
<S'^T w, x> have to agree. Bar: the forward stage's own, 1e-12 of a field up to
64 radial points and times (N_r / 64)^4 past that (the growth of the radial
operators' condition numbers), here of the product of the two norms."""
import sys

import pytest
import torch

from synthetic import direction

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _inner(a, b):
    return float((a.conj() * b).real.sum())


def _norm(a):
    return float(torch.linalg.vector_norm(a))


def _run(grid, Ra):
    import paper_1908_00587_amd as nsc
    from paper_1908_00587_amd.adjoint import radial_solve_vjp
    ctx = nsc.Context(0.6, 80.0, 10.0, Ra, 0.7, *grid, 4.0)
    ctx.set_timestep(dt=1e-3, c=0.5)
    x, a, b, w = [direction(ctx.F, *grid, s).cuda() for s in (31, 32, 33, 34)]
    z = torch.zeros_like(x)
    ds = ctx.radial_solve(x, a, b) - ctx.radial_solve(z, z, z)
    lhs = _inner(w, ds)
    xb, ab, bb = radial_solve_vjp(ctx, w)
    rhs = _inner(xb, x) + _inner(ab, a) + _inner(bb, b)
    torch.cuda.synchronize()
    err = abs(lhs - rhs) / (_norm(w) * _norm(ds))
    _say(f"  {err:.2e}")
    assert err < 1e-12 * max(1.0, (grid[0] / 64) ** 4)


# (N_r, M_theta, M_z): few modes, four |k| per workgroup
GRIDS = [(9, 1, 1), (9, 3, 7), (13, 2, 9), (14, 4, 7), (15, 3, 7), (16, 2, 9), (18, 4, 5), (32, 3, 3), (33, 2, 15),
         (64, 2, 17), (65, 3, 11), (75, 2, 9), (96, 2, 7), (97, 1, 29), (127, 2, 9), (128, 2, 11), (144, 2, 9)]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_stage_vjp_small_tiles(grid, Ra):
    _say("stage vjp", grid, Ra)
    _run(grid, Ra)


# enough tiles that a workgroup takes eight |k|
@pytest.mark.parametrize("grid,Ra", [((16, 64, 59), 0.0), ((18, 64, 49), 1.0e4), ((33, 64, 59), 1.0e4),
                                     ((49, 64, 49), 0.0), ((64, 64, 53), 0.0), ((64, 64, 49), 1.0e4)])
def test_stage_vjp_wide_tiles(grid, Ra):
    _say("stage vjp", grid, Ra)
    _run(grid, Ra)
