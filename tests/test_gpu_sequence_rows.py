"""GPU parity of the implicit stage past 128 radial points, where it runs as a
sequence of kernels whose stencil passes take one, two or four rows per lane,
by the number of wavefronts that leaves (a row's wavefronts W = 4 ceil(modes /
256), times three field groups of the right sides if heated and two if not: four
rows where W ceil(N_r / 4) reaches 4096, two where W ceil(N_r / 2) does; the
velocity right sides from 8192 on).  The grids give every count to every pass
with a short last chunk, walking rows first (long radial rows) or not; sampled
modes against the FP64 oracle, cylinders with and without temperature and pipe.
Bars of the implicit stage past 64 points: 1e-12 of the state and 1e-10 of the
pressure times (N_r / 64)^4, the growth of the operators' condition numbers."""
import sys

import pytest
import torch

import oracle as O
from oracle import pipe as P
from synthetic import direction

pytestmark = pytest.mark.gpu

# rows per lane of right sides, divergence, velocity right sides
GRIDS = [(131, 32, 63),    # 2, 1, 1: 131 = 65 x 2 + 1
         (130, 48, 95),    # 4, 2, 1: 130 = 32 x 4 + 2
         (131, 48, 95),    # the same with a short last chunk of two rows' passes
         (131, 64, 127),   # 4, 4, 2: 131 = 32 x 4 + 3
         (131, 128, 127),  # 4, 4, 4, rows first
         (259, 64, 127)]   # 4, 4, 4: 259 = 64 x 4 + 3
DT = 1e-3


def _rel(a, b):
    return float((a - b).abs().max() / b.abs().max())


def _modes(grid):
    """(m, k + K) in the first and last tiles, |k| = 0, m = 0 and 1 among them."""
    _, mt, mz = grid
    K = (mz - 1) // 2
    return [(0, K), (0, 2), (1, K), (1, 0), (mt // 2, K + 7), (mt - 1, 0), (mt - 1, mz - 1)]


def _check(grid, x, pr, X, Pr):
    torch.cuda.synchronize()
    x, pr = x.cpu(), pr.cpu()
    grow = (grid[0] / 64) ** 4
    eu, ep = _rel(x, X), _rel(pr, Pr)
    print(f"  state {eu:.2e} pressure {ep:.2e}", flush=True)
    assert eu < 1e-12 * grow and ep < 1e-10 * grow


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_sequence_rows(grid, Ra):
    print("stage sequence", grid, Ra, flush=True)
    sys.stdout.flush()
    import paper_1908_00587_amd as nsc
    args = (0.6, 80.0, 10.0, Ra, 0.7) + grid + (4.0,)
    p = O.Params(*args)
    u = O.base_state(p) + 1e-2 * direction(p.F, *grid, 31)
    nn, nq = 10 * direction(p.F, *grid, 32), 10 * direction(p.F, *grid, 33)
    ctx = nsc.Context(*args)
    ctx.set_timestep(dt=DT, c=0.5)
    x, pr = ctx.radial_solve(u.cuda(), nn.cuda(), nq.cuda(), pressure=True)
    m, kk = (torch.tensor(v) for v in zip(*_modes(grid)))
    # the m = 0 column is averaged with its mirror (0, -k)
    mirror = torch.where(m == 0, p.M_z - 1 - kk, kk)
    solve = lambda k: O.radial_solve_modes(p, m, k, u[:, :, m, k], nn[:, :, m, k], nq[:, :, m, k], DT, 0.5)
    X, Pr = solve(kk)
    Xm, Pm = solve(mirror)
    X = torch.where(m == 0, 0.5 * (X + Xm.conj()), X)
    Pr = torch.where(m == 0, 0.5 * (Pr + Pm.conj()), Pr)
    _check(grid, x[:, :, m.cuda(), kk.cuda()], pr[:, m.cuda(), kk.cuda()], X, Pr)


@pytest.mark.parametrize("grid", GRIDS)
def test_sequence_rows_pipe(grid):
    print("pipe stage sequence", grid, flush=True)
    sys.stdout.flush()
    import paper_1908_00587_amd as nsc
    args = (120.0,) + grid + (5.0,)
    p = P.PipeParams(*args)
    u = P.base_state(p) + 1e-2 * direction(3, *grid, 31)
    nn, nq = 10 * direction(3, *grid, 32), 10 * direction(3, *grid, 33)
    ctx = nsc.Context.pipe(*args)
    ctx.set_timestep(dt=DT, c=0.5)
    x, pr = ctx.radial_solve(u.cuda(), nn.cuda(), nq.cuda(), pressure=True)
    ops = P._Ops(p)
    one = lambda m, k: P.radial_solve_mode(p, ops, m, k, u[:, :, m, k], nn[:, :, m, k], nq[:, :, m, k], DT, 0.5)
    X, Pr = [], []
    modes = _modes(grid)
    for m, k in modes:
        a, b = one(m, k)
        if m == 0:
            am, bm = one(m, p.M_z - 1 - k)
            a, b = 0.5 * (a + am.conj()), 0.5 * (b + bm.conj())
        X.append(a)
        Pr.append(b)
    m, kk = (torch.tensor(v).cuda() for v in zip(*modes))
    _check(grid, x[:, :, m, kk], pr[:, m, kk], torch.stack(X, -1), torch.stack(Pr, -1))
