"""A restart remap on one stream beside steps of the same context on another:
the remap waits for its own stream only, so its weights must not lie in a
workspace that a step in flight reads and writes."""
import os
import re
import sys

import pytest
import torch

from synthetic import direction

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1908_00587_amd", "csrc")


def test_remap_weights_outside_the_step_workspaces():
    """Host: the remap names no workspace that another call uses."""
    text = open(os.path.join(CSRC, "k_restart.hip")).read()
    body = text[text.index("int nsc_remap_state("):]
    body = body[:body.index("\n}\n")]
    used = set(re.findall(r"c->(\w+)", body))
    internal = open(os.path.join(CSRC, "nsc_internal.h")).read()
    shared = set(re.findall(r"\*(s_\w+|zbuf|wbuf|cfl_part|cfl_val|e_part)\b", internal))
    assert {"s_f", "s_x", "s_mean", "zbuf"} <= shared
    assert not used & shared


# past 128 radial points the implicit stage runs as a sequence of kernels
# through the workspaces, up to 128 as one kernel
@pytest.mark.gpu
@pytest.mark.parametrize("N_r", [144, 33])
def test_remap_beside_steps(N_r):
    print("remap beside steps", N_r, flush=True)
    sys.stdout.flush()
    import paper_1908_00587_amd as nsc
    grid, old = (N_r, 24, 47), (65, 16, 31)
    ctx = nsc.Context(0.6, 80.0, 10.0, 1.0e4, 0.7, *grid, 4.0)
    ctx.set_timestep(dt=1e-5)
    src = direction(ctx.F, *old, 31).cuda()
    u0 = (1e-3 * direction(ctx.F, *grid, 32)).cuda()
    steps = 12
    ref_map = ctx.remap_state(src)
    ref = u0.clone()
    for _ in range(steps):
        ctx.step(ref, 1e-5)
    torch.cuda.synchronize()
    u = u0.clone()
    got = [torch.empty_like(u) for _ in range(steps)]
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for out in got:
        with torch.cuda.stream(a):
            ctx.step(u, 1e-5)
        with torch.cuda.stream(b):
            ctx.remap_state(src, out)
    torch.cuda.synchronize()
    assert torch.equal(u, ref)
    for out in got:
        assert torch.equal(out, ref_map)
