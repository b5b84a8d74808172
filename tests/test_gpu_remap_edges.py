"""GPU parity of the restart remap and the probes at the edges of their loops:
target rows around the groups of sixteen, grids small enough that the weights
need their own memory, more or fewer modes than before, and probe sums over
fewer modes than lanes and over several rounds, against dense barycentric
interpolation and Fourier sums in FP64.  Bars: 1e-12 of the largest value (sums
of up to 128 weights of a well-conditioned interpolant; phases of up to 60
radians)."""
import math
import sys

import pytest
import torch

from synthetic import direction

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _ctx(grid, Ra):
    import paper_1908_00587_amd as nsc
    return nsc.Context(0.6, 80.0, 10.0, Ra, 0.7, *grid, 4.0)


def _grid(n, r_i, r_o):
    j = torch.arange(n, dtype=torch.float64)
    return 0.5 * (r_i + r_o) + 0.5 * torch.cos(math.pi * (n - 1 - j) / (n - 1))


def _interp(n0, n1, r_i, r_o):
    x0, x1 = _grid(n0, r_i, r_o), _grid(n1, r_i, r_o)
    w = (-1.0) ** torch.arange(n0, dtype=torch.float64)
    w[0] *= 0.5
    w[-1] *= 0.5
    d = x1[:, None] - x0[None, :]
    hit = d.abs() < 1e-14
    q = w / torch.where(hit, torch.ones_like(d), d)
    return torch.where(hit.any(1, keepdim=True), hit.double(), q / q.sum(1, keepdim=True))


@pytest.mark.parametrize("old,new", [((9, 1, 1), (16, 1, 1)), ((64, 1, 1), (9, 1, 1)), ((12, 3, 7), (15, 4, 9)),
                                     ((18, 4, 9), (16, 3, 5)), ((33, 2, 5), (65, 3, 7)), ((64, 4, 7), (33, 4, 7)),
                                     ((97, 2, 9), (49, 3, 11)), ((33, 3, 9), (33, 5, 15))])
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_remap(old, new, Ra):
    _say("remap", old, new, Ra)
    ctx = _ctx(new, Ra)
    src = direction(ctx.F, *old, 31)
    got = ctx.remap_state(src.cuda()).cpu()
    r = ctx.grid()
    W = _interp(old[0], new[0], float(r[0]), float(r[-1]))
    ref = torch.zeros(ctx.shape, dtype=torch.complex128)
    m, K0, K1 = min(old[1], new[1]), (old[2] - 1) // 2, (new[2] - 1) // 2
    k = min(K0, K1)
    part = src[:, :, :m, K0 - k:K0 + k + 1]
    ref[:, :, :m, K1 - k:K1 + k + 1] = torch.einsum("ij,fjmk->fimk", W.to(part.dtype), part)
    err = float((got - ref).abs().max() / ref.abs().max())
    _say(f"  {err:.2e}")
    assert err < 1e-12


@pytest.mark.parametrize("grid", [(9, 1, 1), (12, 5, 9), (16, 32, 31), (9, 48, 127)])
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_probe(grid, Ra):
    _say("probe", grid, Ra)
    ctx = _ctx(grid, Ra)
    u = direction(ctx.F, *grid, 31)
    rows, theta, z = [0, grid[0] - 1, 3], [0.0, 0.7, -2.1], [0.1, -1.3, 3.0]
    got = torch.as_tensor(ctx.probe(u.cuda(), rows, theta, z)).cpu()
    m = torch.arange(grid[1], dtype=torch.float64)[:, None]
    k = torch.arange(grid[2], dtype=torch.float64)[None, :] - (grid[2] - 1) // 2
    for i in range(3):
        ph = m * theta[i] + k * (2 * math.pi / 4.0) * z[i]
        c = torch.where(m == 0, 1.0, 2.0)
        ref = (c * (u[:, rows[i]].real * torch.cos(ph) - u[:, rows[i]].imag * torch.sin(ph))).sum((1, 2))
        scale = float((c * u[:, rows[i]].abs()).sum((1, 2)).max())
        assert float((got[i] - ref).abs().max()) < 1e-12 * scale
