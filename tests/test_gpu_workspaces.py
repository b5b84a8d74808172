"""Device memory of a context: the workspaces of the kernel sequence (nine
fields and more) are held only where the sequence runs, past 128 radial
points."""
import gc

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["heated", "isothermal", "pipe"])
def test_sequence_workspaces_only_where_it_runs(kind):
    print("workspaces", kind, flush=True)
    import paper_1908_00587_amd as nsc
    mt, mz = 48, 95

    def held(N_r):
        gc.collect()
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        if kind == "pipe":
            ctx = nsc.Context.pipe(100.0, N_r, mt, mz, 4.0)
        else:
            ctx = nsc.Context(0.6, 80.0, 10.0, 1.0e4 if kind == "heated" else 0.0, 0.7, N_r, mt, mz, 4.0)
        after = torch.cuda.mem_get_info()[0]
        ctx.close()
        return before - after

    held(16)  # the library's code and static memory are loaded
    field = 128 * mt * mz * 16
    # one row more adds less than one field to the rest
    assert held(129) - held(128) > 8 * field
