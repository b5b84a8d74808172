"""GPU parity at 17 radial points, the one column length at which a column of
the radial stencils (column 8) lies in the windows of all 17 rows: implicit
stage and factors (cylinders and pipe, four and eight |k| per workgroup), its
vector-Jacobian product, and the nonlinear term with its product.  Checks and
bars are those of the same tests at other column lengths."""
import math
import sys

import pytest
import torch

import oracle as O
import test_gpu_lengths as lengths
import test_gpu_stage as stage
import test_gpu_stage_adjoint as stage_adjoint
from synthetic import direction

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(17, 1, 1), (17, 4, 5), (17, 64, 59)])
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_stage(grid, Ra):
    stage.test_stage_small_tiles(grid, Ra)


@pytest.mark.parametrize("grid", [(17, 2, 5), (17, 3, 9)])
def test_stage_pipe(grid):
    stage.test_stage_pipe(grid)


@pytest.mark.parametrize("grid", [(17, 1, 1), (17, 4, 5), (17, 64, 59)])
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_stage_vjp(grid, Ra):
    stage_adjoint.test_stage_vjp_small_tiles(grid, Ra)


@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_nonlinear(Ra):
    lengths.test_nonlinear_lengths((17, 4, 4), Ra)
    lengths.test_nonlinear_vjp_lengths((17, 4, 4), Ra)


@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_step_vjp(Ra):
    """The step's vector-Jacobian product against central differences of the
    step.  A step good to 1e-12 of a state of size 100 leaves 1e-10 / (2 h) =
    5e-7 at h = 1e-4 (the step's third derivative is of order dt^2): bar 1e-6."""
    print("step vjp at 17 points", Ra, flush=True)
    sys.stdout.flush()
    import paper_1908_00587_amd as nsc
    from paper_1908_00587_amd.adjoint import step_stages_fused, step_vjp_fused
    grid = (17, 3, 7)
    args = (0.6, 80.0, 10.0, Ra, 0.7) + grid + (2 * math.pi,)
    p = O.Params(*args)
    ctx = nsc.Context(*args)
    ctx.set_timestep(dt=1e-3)
    u = (O.base_state(p) + 1e-1 * direction(p.F, *grid, 51)).cuda()
    d, w = direction(p.F, *grid, 52).cuda(), direction(p.F, *grid, 53).cuda()
    h = 1e-4
    up, um = u + h * d, u - h * d
    ctx.step(up, 1e-3)
    ctx.step(um, 1e-3)
    a = float((w.conj() * (up - um)).real.sum()) / (2 * h)
    stages, _ = step_stages_fused(ctx, u)
    b = float((step_vjp_fused(ctx, u, stages, w).conj() * d).real.sum())
    scale = float(torch.linalg.vector_norm(w) * torch.linalg.vector_norm(up - um)) / (2 * h)
    assert abs(a - b) < 1e-6 * scale
