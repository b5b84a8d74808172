"""The pressure of the implicit stage written over an input state that is no
longer needed: only the output state may not alias the inputs, so the results
are those of separate arrays, bit for bit, wherever the pressure lies."""
import ctypes
import sys

import pytest
import torch

from synthetic import direction

pytestmark = pytest.mark.gpu


# (N_r, M_theta, M_z): the one-kernel stage with four and eight |k| per
# workgroup, and the kernel sequence; distances in complex entries, whole
# planes and not
@pytest.mark.parametrize("grid", [(16, 3, 9), (16, 64, 59), (130, 3, 9)])
@pytest.mark.parametrize("which", [0, 1, 2])
def test_pressure_over_an_input(grid, which):
    print("pressure over input", grid, which, flush=True)
    sys.stdout.flush()
    import paper_1908_00587_amd as nsc
    ctx = nsc.Context(0.6, 80.0, 10.0, 1.0e4, 0.7, *grid, 4.0)
    ctx.set_timestep(dt=1e-3)
    x = [direction(ctx.F, *grid, 31 + i).cuda() for i in range(3)]
    ref, pref = ctx.radial_solve(*x, pressure=True)
    torch.cuda.synchronize()
    plane = grid[1] * grid[2]
    n = ctx.F * grid[0] * plane
    for shift in (0, plane, 1, plane // 2 + 1, 3 * plane - 1):
        buf = torch.zeros(n + grid[0] * plane, dtype=torch.complex128, device="cuda")
        y = list(x)
        y[which] = buf[:n]
        y[which].copy_(x[which].reshape(-1))
        p = buf[shift:shift + grid[0] * plane]
        out = ctx.empty()
        torch.cuda.synchronize()
        ctx._sync_stream()
        ptr = [ctypes.c_void_p(t.data_ptr()) for t in (*y, out, p)]
        assert ctx._L.nsc_radial_solve(ctx._h, *ptr) == 0
        torch.cuda.synchronize()
        assert torch.equal(out, ref), shift
        assert torch.equal(p.reshape(pref.shape), pref), shift
