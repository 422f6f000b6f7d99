"""Iterations that a chunk launches past convergence: they change nothing, in
every schedule, and end before they touch the mesh's data."""
import pytest

from gpu_common import say, to_dev
from seminputs import box_mesh, random_global_rhs

pytestmark = pytest.mark.gpu


# two launches (N = 9 and 7: matrix cores in FP32; 4: the per-point table),
# three, four
@pytest.mark.parametrize("N,n", [(7, (4, 4, 4)), (9, (4, 3, 4)), (4, (6, 5, 6)),
                                 (8, (12, 12, 13)), (7, (16, 16, 16)), (9, (12, 12, 13)),
                                 (7, (14, 14, 14))])
@pytest.mark.parametrize("jacobi", [False, True])
def test_state_is_passed_on(N, n, jacobi):
    """The iterate and the state after one chunk that converges early are
    bitwise those of a solve that looks after every iteration."""
    import torch
    import paper_2108_12188_amd as sem
    say(f"past convergence N={N} {n} jacobi={jacobi}")
    mesh = box_mesh(*n, N, perturb=0.1, seed=20 + N)
    gm = sem.Mesh.from_box(mesh)
    bh = random_global_rhs(mesh, seed=7)
    pc = sem.PRECOND_JACOBI if jacobi else sem.PRECOND_NONE
    for dtype in (torch.float64, torch.float32):
        b = to_dev(bh, dtype)
        kw = dict(geom=sem.ON_THE_FLY, precond=pc, history=40)
        for stop in (dict(max_iter=5, tol=1e-30), dict(max_iter=1000, tol=0.3)):
            x, r = gm.cg_solve(b, poll_every=37, **stop, **kw)
            y, q = gm.cg_solve(b, poll_every=1, **stop, **kw)
            assert (r["iters"], r["status"]) == (q["iters"], q["status"])
            assert r["rel_res_recursive"] == q["rel_res_recursive"]
            assert r["hist_rho"].tolist() == q["hist_rho"].tolist()
            assert torch.equal(x, y), dtype
    gm.close()


def test_costs_no_pass_over_the_data():
    """N = 7, 4.1 M points, three launches: an iteration past convergence is
    its launches (measured 0.22 of a live iteration; 0.38 with the operator's
    tiles staged and the partials summed before the stop is looked at)."""
    import torch
    import paper_2108_12188_amd as sem
    mesh = box_mesh(20, 20, 20, 7, perturb=0.1, seed=3)
    gm = sem.Mesh.from_box(mesh)
    b = to_dev(random_global_rhs(mesh, seed=8), torch.float32)

    def seconds(**kw):
        return min(gm.cg_solve(b, geom=sem.ON_THE_FLY, **kw)[1]["seconds"] for _ in range(8))

    past = seconds(max_iter=1, tol=1e-30, poll_every=210) - \
        seconds(max_iter=1, tol=1e-30, poll_every=10)
    live = seconds(max_iter=210, tol=1e-30, poll_every=210) - \
        seconds(max_iter=10, tol=1e-30, poll_every=10)
    say(f"past convergence {past / 200 * 1e6:.1f} us, live {live / 200 * 1e6:.1f} us")
    assert past < 0.3 * live
    gm.close()
