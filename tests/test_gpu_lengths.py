"""GPU parity of the compile-time transform lengths: nonlinear term and its
vector--Jacobian product on grids whose padded lengths run through the
families of radices (powers of two, odd powers of three, factors of five;
one and several wavefronts per theta line set), against the FP64 oracle and
by the dot-product identity of a quadratic map.  Bars as elsewhere: FP64
1e-12 of the largest entry, mixed 2e-6; dot products 1e-11."""
import math
import sys

import pytest
import torch

import oracle as O
from synthetic import direction

pytestmark = pytest.mark.gpu

# (N_r, M_theta, K + 1): theta lengths 3 M_theta, z lengths 3 (K + 1)
GRIDS = [(9, 4, 4), (10, 8, 12), (9, 12, 20), (11, 20, 24), (9, 24, 36), (10, 36, 40), (9, 40, 48),
         (9, 60, 16), (9, 72, 8), (9, 80, 4), (9, 96, 4), (9, 100, 5), (9, 108, 4), (9, 128, 4),
         (9, 160, 3), (9, 180, 3), (9, 192, 3), (9, 200, 3), (9, 216, 3), (9, 240, 3), (9, 256, 3),
         (9, 4, 60), (9, 4, 100), (9, 4, 108), (9, 3, 128), (9, 3, 144), (9, 2, 216), (9, 2, 256)]


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _setup(grid, Ra):
    import paper_1908_00587_amd as nsc
    nr, mt, kp1 = grid
    args = (0.6, 80.0, 10.0, Ra, 0.7, nr, mt, 2 * kp1 - 1, 2 * math.pi)
    p = O.Params(*args)
    return p, nsc.Context(*args), direction(p.F, nr, mt, p.M_z, 41)


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_nonlinear_lengths(grid, Ra):
    _say("nonlinear", grid, Ra)
    p, ctx, d = _setup(grid, Ra)
    u = O.base_state(p) + 1e-2 * d
    ref, dtc = O.nonlinear(p, u)
    for prec, tol in (("fp64", 1e-12), ("mixed", 2e-6)):
        ctx.set_precision(prec)
        out, c = ctx.nonlinear(u.cuda(), cfl=True)
        torch.cuda.synchronize()
        e = float((out.cpu() - ref).abs().max() / ref.abs().max())
        _say(f"  {prec} {e:.2e}")
        assert e < tol
        assert abs(float(c.cpu()[0]) / dtc - 1) < (1e-14 if prec == "fp64" else 1e-6)


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_nonlinear_vjp_lengths(grid, Ra):
    """N is quadratic, so (N(u+d) - N(u-d))/2 is the exact Jacobian action."""
    _say("nonlinear vjp", grid, Ra)
    from paper_1908_00587_amd.adjoint import nonlinear_vjp
    p, ctx, d = _setup(grid, Ra)
    u = O.base_state(p) + 1e-1 * direction(p.F, p.N_r, p.M_theta, p.M_z, 42)
    nbar = direction(p.F, p.N_r, p.M_theta, p.M_z, 43)
    up, um = ctx.nonlinear((u + d).cuda()).cpu(), ctx.nonlinear((u - d).cuda()).cpu()
    jd = 0.5 * (up - um)
    g = nonlinear_vjp(ctx, u.cuda(), nbar.cuda()).cpu()
    a = float((nbar.conj() * jd).real.sum())
    b = float((g.conj() * d).real.sum())
    # relative to the terms' sizes: both sides are sums of that many products
    scale = float((nbar.abs() * jd.abs()).sum())
    _say(f"  {abs(a - b) / scale:.2e}")
    assert abs(a - b) < 1e-11 * scale
