"""GPU parity of the factorisation and the influence responses at the edges of
their row loops: the smallest columns, every remainder of the four-row loop,
and columns past the LDS of the influence kernel (160 points), cylinders and
pipe, against the FP64 oracle's implicit stage.  Bars as for the stage itself:
1e-12 of each field times (N_r / 64)^4 past 64 radial points, the growth of
the radial operators' condition numbers."""
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


def _check(ctx, ref, x, N_r):
    torch.cuda.synchronize()
    err = float((x.cpu() - ref).abs().max() / ref.abs().max())
    _say(f"  {err:.2e}")
    assert err < 1e-12 * max(1.0, (N_r / 64) ** 4)


@pytest.mark.parametrize("N_r", [9, 10, 11, 12, 13, 14, 15, 16, 18, 19, 20, 21, 159, 160])
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_factor_rows(N_r, Ra):
    _say("factor", N_r, Ra)
    import paper_1908_00587_amd as nsc
    grid = (N_r, 3, 9)
    args = (0.6, 80.0, 10.0, Ra, 0.7) + grid + (4.0,)
    p = O.Params(*args)
    u = O.base_state(p) + 1e-2 * direction(p.F, *grid, 31)
    nn, nq = 10 * direction(p.F, *grid, 32), 10 * direction(p.F, *grid, 33)
    ctx = nsc.Context(*args)
    ctx.set_timestep(dt=1e-3, c=0.5)
    _check(ctx, O.radial_solve(p, u, nn, nq, 1e-3, 0.5)[0], ctx.radial_solve(u.cuda(), nn.cuda(), nq.cuda()), N_r)


@pytest.mark.parametrize("N_r", [9, 10, 11, 12, 14, 20, 160])
def test_factor_rows_pipe(N_r):
    _say("pipe factor", N_r)
    import paper_1908_00587_amd as nsc
    grid = (N_r, 3, 9)
    args = (120.0,) + grid + (5.0,)
    p = P.PipeParams(*args)
    u = P.base_state(p) + 1e-2 * direction(3, *grid, 31)
    nn, nq = 10 * direction(3, *grid, 32), 10 * direction(3, *grid, 33)
    ctx = nsc.Context.pipe(*args)
    ctx.set_timestep(dt=1e-3, c=0.5)
    _check(ctx, P.radial_solve(p, u, nn, nq, 1e-3)[0], ctx.radial_solve(u.cuda(), nn.cuda(), nq.cuda()), N_r)
