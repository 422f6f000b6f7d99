"""Fixed iteration counts where there is nothing to iterate on."""
import pytest

from gpu_common import say, to_dev
from seminputs import box_mesh, random_global_rhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n", [(7, (4, 4, 4)), (7, (16, 16, 16))])
def test_zero_right_hand_side_runs_no_iteration(N, n):
    """A solve of a zero right-hand side by a fixed count takes about as long
    as one by a tolerance, which looks at the state first (100 iterations past
    convergence would take 4 to 10 times as long)."""
    import torch
    import paper_2108_12188_amd as sem
    mesh = box_mesh(*n, N, perturb=0.1, seed=5)
    gm = sem.Mesh.from_box(mesh)
    for dtype in (torch.float32, torch.float64):
        b = torch.zeros(gm.n, dtype=dtype, device="cuda")

        def seconds(**kw):
            return min(gm.cg_solve(b, geom=sem.ON_THE_FLY, **kw)[1]["seconds"]
                       for _ in range(10))

        fixed, tol = seconds(fixed_iters=500), seconds(tol=1e-8)
        say(f"zero right-hand side: fixed {fixed * 1e6:.0f} us, tolerance {tol * 1e6:.0f} us")
        assert fixed < 2 * tol, dtype
    gm.close()


@pytest.mark.parametrize("fixed,poll", [(64, 0), (99, 0), (101, 0), (150, 0), (10, 7), (14, 7)])
def test_rest_of_a_count(fixed, poll):
    """Counts that are no multiple of the chunk, with and without histories
    and kernel times."""
    import torch
    import paper_2108_12188_amd as sem
    say(f"fixed={fixed} poll={poll}")
    mesh = box_mesh(5, 4, 4, 6, perturb=0.1, seed=9)
    gm = sem.Mesh.from_box(mesh)
    b = to_dev(random_global_rhs(mesh, seed=2), torch.float64)
    kw = dict(geom=sem.ON_THE_FLY, fixed_iters=fixed)
    x, r = gm.cg_solve(b, poll_every=poll, **kw)
    y, q = gm.cg_solve(b, poll_every=1, use_graph=False, history=fixed + 1, **kw)
    z, s = gm.cg_solve(b, poll_every=poll, kernel_times=True, **kw)
    assert r["iters"] == q["iters"] == s["iters"] == fixed
    assert torch.equal(x, y) and torch.equal(x, z)
    gm.close()
