"""Fixed iteration counts around the chunk sizes a solve runs them in."""
import numpy as np
import pytest

from gpu_common import say, to_dev
from seminputs import box_mesh, random_global_rhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fixed", [1, 2, 49, 50, 51, 64, 100, 101, 149, 151, 201])
def test_fixed_count_is_met_exactly(fixed):
    """Chunks of every size run exactly `fixed` iterations: the state, the
    histories and x are bitwise those of single-iteration polls."""
    import torch
    import paper_2108_12188_amd as sem
    say(f"fixed={fixed}")
    mesh = box_mesh(4, 3, 3, 5, perturb=0.1, seed=5, permute=True, reorient=True)
    gm = sem.Mesh.from_box(mesh)
    b = to_dev(random_global_rhs(mesh, seed=6), torch.float64)
    kw = dict(prec=sem.FP64, geom=sem.ON_THE_FLY, fixed_iters=fixed, history=fixed + 1)
    x, r = gm.cg_solve(b, **kw)
    y, q = gm.cg_solve(b, poll_every=1, use_graph=False, **kw)
    assert r["iters"] == q["iters"] == fixed
    assert torch.equal(x, y)
    np.testing.assert_array_equal(r["hist_rho"], q["hist_rho"])
    np.testing.assert_array_equal(r["hist_alpha"], q["hist_alpha"])
    gm.close()


def test_fixed_count_with_nothing_to_solve():
    """A zero right-hand side stops at once, whatever the chunks."""
    import torch
    import paper_2108_12188_amd as sem
    mesh = box_mesh(3, 2, 2, 4, seed=5)
    gm = sem.Mesh.from_box(mesh)
    b = torch.zeros(gm.n, dtype=torch.float64, device="cuda")
    for fixed in (7, 120, 500):
        x, r = gm.cg_solve(b, geom=sem.ON_THE_FLY, fixed_iters=fixed)
        y, q = gm.cg_solve(b, geom=sem.ON_THE_FLY, fixed_iters=fixed, poll_every=1)
        assert (r["iters"], r["status"]) == (q["iters"], q["status"])
        assert torch.equal(x, y) and not torch.any(x)
    gm.close()
