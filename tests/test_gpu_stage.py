"""GPU parity of the one-kernel implicit stage at the edges of its tiles:
radial points around the row groups of a thread (32, 64, 96, 128 with 4 |k|
per workgroup; 16, 32, 48, 64 with 8), the smallest grid, |k| counts that
leave a remainder in the last tile, heated, isothermal and pipe columns, with
and without the pressure, against the FP64 oracle on the same seeded inputs.
Bars as for the implicit stage elsewhere: 1e-12 of each field, 1e-10 of the
pressure (the Neumann Poisson operators' conditioning), for up to 64 radial
points; past that times (N_r / 64)^4, the growth of the second-derivative
operators' condition numbers on the clustered points, which is what bounds
the agreement of two LU orderings."""
import math
import sys

import pytest
import torch

import oracle as O
from oracle import pipe as P
from synthetic import direction

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _rel(a, b):
    a = a.detach().cpu()
    return float((a - b).abs().max() / b.abs().max())


def _run(ctx, ref, u, nn, nq, dt):
    ctx.set_timestep(dt=dt, c=0.5)
    x, p = ctx.radial_solve(u.cuda(), nn.cuda(), nq.cuda(), pressure=True)
    y = ctx.radial_solve(u.cuda(), nn.cuda(), nq.cuda())
    torch.cuda.synchronize()
    eu, ep = _rel(x, ref[0]), _rel(p, ref[1])
    _say(f"  state {eu:.2e} pressure {ep:.2e}")
    grow = max(1.0, (ctx.N_r / 64) ** 4)
    assert eu < 1e-12 * grow and ep < 1e-10 * grow
    # without the pressure: the same arithmetic (mode (0,0)'s head aside)
    assert _rel(y, ref[0]) < 1e-12 * grow


# (N_r, M_theta, M_z): few modes, four |k| per workgroup
GRIDS = [(9, 1, 1), (9, 3, 7), (16, 2, 9), (18, 4, 5), (32, 3, 3), (33, 2, 15), (64, 2, 17),
         (65, 3, 11), (75, 2, 9), (96, 2, 7), (97, 1, 29), (127, 2, 9), (128, 2, 11)]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_stage_small_tiles(grid, Ra):
    _say("stage", grid, Ra)
    import paper_1908_00587_amd as nsc
    args = (0.6, 80.0, 10.0, Ra, 0.7) + grid + (4.0,)
    p = O.Params(*args)
    u = O.base_state(p) + 1e-2 * direction(p.F, *grid, 31)
    nn, nq = 10 * direction(p.F, *grid, 32), 10 * direction(p.F, *grid, 33)
    _run(nsc.Context(*args), O.radial_solve(p, u, nn, nq, 1e-3, 0.5), u, nn, nq, 1e-3)


# enough tiles that a workgroup takes eight |k|
@pytest.mark.parametrize("grid,Ra", [((16, 64, 59), 0.0), ((18, 64, 49), 1.0e4), ((33, 64, 59), 1.0e4),
                                     ((49, 64, 49), 0.0), ((64, 64, 53), 0.0), ((64, 64, 49), 1.0e4)])
def test_stage_wide_tiles(grid, Ra):
    _say("stage", grid, Ra)
    import paper_1908_00587_amd as nsc
    args = (0.6, 80.0, 10.0, Ra, 0.7) + grid + (4.0,)
    p = O.Params(*args)
    u = O.base_state(p) + 1e-2 * direction(p.F, *grid, 31)
    nn, nq = 10 * direction(p.F, *grid, 32), 10 * direction(p.F, *grid, 33)
    _run(nsc.Context(*args), O.radial_solve(p, u, nn, nq, 1e-3, 0.5), u, nn, nq, 1e-3)


@pytest.mark.parametrize("grid", [(9, 2, 5), (33, 3, 9), (65, 2, 7), (97, 2, 5), (128, 1, 9)])
def test_stage_pipe(grid):
    _say("pipe stage", grid)
    import paper_1908_00587_amd as nsc
    args = (120.0,) + grid + (5.0,)
    p = P.PipeParams(*args)
    u = P.base_state(p) + 1e-2 * direction(3, *grid, 31)
    nn, nq = 10 * direction(3, *grid, 32), 10 * direction(3, *grid, 33)
    _run(nsc.Context.pipe(*args), P.radial_solve(p, u, nn, nq, 1e-3), u, nn, nq, 1e-3)
