"""Every compile-time transform length runs once as a theta length and once as
a z length against the oracle: the lengths that the grids of the other two
length tests leave out, with the same checks and bars, and the launch shape of
the 1536-point FP32 lines (two sets of lines per workgroup if heated) with an
odd number of sets, whose last workgroup has a set to spare."""
import os
import re

import pytest
import torch

import test_gpu_lengths as lengths
import test_gpu_lengths_odd as odd

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (N_r, M_theta, K + 1): theta lengths 3 M_theta, z lengths 3 (K + 1)
GRIDS = [(9, 16, 240), (9, 32, 200), (9, 48, 72), (10, 64, 32), (9, 120, 80), (9, 144, 96), (9, 4, 120), (9, 3, 160),
         (9, 3, 180), (9, 3, 192), (11, 5, 64)]
# M_theta = 512, nine z points: 81 sets
ODD_SETS = (9, 512, 3)


def test_every_length_has_a_grid():
    """Host: the list of lengths against the grids."""
    text = open(os.path.join(ROOT, "paper_1908_00587_amd", "csrc", "nl_lengths.h")).read()
    listed = {int(x) for x in re.findall(r"\bX\((\d+)\)", text)}
    assert len(listed) >= 45
    grids = lengths.GRIDS + odd.GRIDS + GRIDS
    assert listed <= {3 * g[1] for g in grids}
    assert listed <= {3 * g[2] for g in grids}


@pytest.mark.gpu
@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_nonlinear(grid, Ra):
    lengths.test_nonlinear_lengths(grid, Ra)


@pytest.mark.gpu
@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_nonlinear_vjp(grid, Ra):
    lengths.test_nonlinear_vjp_lengths(grid, Ra)


@pytest.mark.gpu
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_nonlinear_odd_number_of_sets(Ra):
    """Mixed precision (FP64 lines of 1536 points are refused), bar 2e-6."""
    lengths._say("nonlinear", ODD_SETS, Ra, "mixed")
    p, ctx, d = lengths._setup(ODD_SETS, Ra)
    u = lengths.O.base_state(p) + 1e-2 * d
    ref, dtc = lengths.O.nonlinear(p, u)
    ctx.set_precision("mixed")
    out, c = ctx.nonlinear(u.cuda(), cfl=True)
    torch.cuda.synchronize()
    assert float((out.cpu() - ref).abs().max() / ref.abs().max()) < 2e-6
    assert abs(float(c.cpu()[0]) / dtc - 1) < 1e-6
