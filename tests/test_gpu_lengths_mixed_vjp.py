"""The mixed-precision vector-Jacobian product of the nonlinear term over the
compile-time transform lengths, against the FP64 product of the same inputs
(itself checked by the dot-product identity), and by that identity at the
1536-point lines, which FP64 refuses.  Bar 1e-5 of the largest entry: four FP32
transforms of up to ten stages, 6e-8 each, make 2.4e-6 of the largest values of a
line, and the nine-point sums of the transposed derivative add nine such errors
of independent rows, about three times as much."""
import pytest
import torch

import test_gpu_lengths as lengths
import test_gpu_lengths_all as rest
import test_gpu_lengths_odd as odd
from synthetic import direction

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", lengths.GRIDS + odd.GRIDS + rest.GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_against_fp64(grid, Ra):
    lengths._say("mixed nonlinear vjp", grid, Ra)
    from paper_1908_00587_amd.adjoint import nonlinear_vjp
    p, ctx, _ = lengths._setup(grid, Ra)
    u = (lengths.O.base_state(p) + 1e-1 * direction(p.F, p.N_r, p.M_theta, p.M_z, 42)).cuda()
    nbar = direction(p.F, p.N_r, p.M_theta, p.M_z, 43).cuda()
    ref = nonlinear_vjp(ctx, u, nbar)
    ctx.set_precision("mixed")
    got = nonlinear_vjp(ctx, u, nbar)
    torch.cuda.synchronize()
    err = float((got - ref).abs().max() / ref.abs().max())
    lengths._say(f"  {err:.2e}")
    assert err < 1e-5


@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_odd_number_of_sets(Ra):
    lengths._say("mixed nonlinear vjp", rest.ODD_SETS, Ra)
    from paper_1908_00587_amd.adjoint import nonlinear_vjp
    p, ctx, d = lengths._setup(rest.ODD_SETS, Ra)
    u, nbar = (direction(p.F, p.N_r, p.M_theta, p.M_z, s) for s in (42, 43))
    ctx.set_precision("mixed")
    # N is quadratic: (N(u + d) - N(u - d)) / 2 is the exact Jacobian action
    jd = 0.5 * (ctx.nonlinear((u + d).cuda()) - ctx.nonlinear((u - d).cuda())).cpu()
    g = nonlinear_vjp(ctx, u.cuda(), nbar.cuda()).cpu()
    a = float((nbar.conj() * jd).real.sum())
    b = float((g.conj() * d).real.sum())
    scale = float((nbar.abs() * jd.abs()).sum())
    lengths._say(f"  {abs(a - b) / scale:.2e}")
    assert abs(a - b) < 1e-5 * scale
