"""The two-, three- and four-launch schedules of a CG iteration: the sizes
where the choice changes, ragged block steps, groups of many copies, and a
batch whose total size changes the schedule of its members."""
import dataclasses

import numpy as np
import pytest

import oracle
from gpu_common import rel_norm, say, to_dev, to_host
from seminputs import box_mesh, random_global_rhs
from test_host_direct import tied_lines

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11])
@pytest.mark.parametrize("tied", [False, True])
def test_two_launch_matches_oracle(N, tied):
    """Small meshes (two launches; with tied edge lines the groups hold up to
    48 copies): FP64 to rounding, FP32 to the operator's bound, with
    histories."""
    import torch
    import paper_2108_12188_amd as sem
    say(f"two-launch N={N} tied={tied}")
    mesh = box_mesh(4, 3, 3, N, perturb=0.1, seed=300 + N, reorient=True, permute=True)
    if tied:
        mesh = dataclasses.replace(mesh, glob_id=tied_lines(mesh))
    b = random_global_rhs(mesh, seed=31)
    pr = oracle.Problem(mesh)
    # past convergence rho is rounding noise: stay well below the number of
    # unknowns (N = 1 with tied lines has 2 of them)
    free = np.unique(mesh.glob_id[mesh.dirichlet == 0]).size
    iters = max(1, min(6, free // 4))
    xo, _, hist = pr.cg(b, fixed=iters)
    gm = sem.Mesh.from_box(mesh, g_fp32=True, g_fp64=True)
    for geom in (0, 1):
        for dtype, tol in ((torch.float64, 1e-11), (torch.float32, iters * 1e-5)):
            x, res = gm.cg_solve(to_dev(b, dtype), geom=geom, fixed_iters=iters, history=iters + 1)
            assert res["iters"] == iters
            np.testing.assert_allclose(res["hist_rho"], hist["rho"][:iters + 1], rtol=10 * tol)
            np.testing.assert_allclose(res["hist_alpha"][1:], hist["alpha"][1:iters + 1],
                                       rtol=10 * tol)
            assert rel_norm(to_host(x), xo) <= tol, (geom, dtype)
    gm.close()


# sizes on both sides of 2^20, 2^21 (FP64) and 2^22 local points, the block
# counts between them, points that are no multiple of 4 (even N), and more
# than one step per block
@pytest.mark.parametrize("N,n", [(7, (13, 12, 13)), (7, (13, 13, 13)), (4, (20, 20, 21)),
                                 (4, (20, 21, 21)), (5, (17, 18, 17)), (8, (11, 13, 10)),
                                 (8, (14, 14, 15)), (9, (12, 13, 14)), (7, (20, 20, 20)),
                                 (7, (20, 20, 21)), (6, (23, 23, 23)), (3, (40, 40, 40))])
def test_schedules_agree_at_their_limits(N, n):
    """Each size against the paper's schedule (a gather-scatter pass of its
    own, sums by one block) on the same mesh, plain and Jacobi."""
    import torch
    import paper_2108_12188_amd as sem
    say(f"schedules N={N} {n}")
    mesh = box_mesh(*n, N, perturb=0.1, seed=400 + N)
    b = random_global_rhs(mesh, seed=32)
    gm = sem.Mesh.from_box(mesh, g_fp32=False)
    gp = sem.Mesh.from_box(mesh, g_fp32=False, gather_pass=True)
    for pc in (sem.PRECOND_NONE, sem.PRECOND_JACOBI):
        for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 1e-5)):
            bd = to_dev(b, dtype)
            x, rx = gm.cg_solve(bd, geom=1, fixed_iters=5, precond=pc, history=6)
            y, ry = gp.cg_solve(bd, geom=1, fixed_iters=5, precond=pc, history=6)
            assert rx["iters"] == ry["iters"] == 5
            np.testing.assert_allclose(rx["hist_rho"], ry["hist_rho"], rtol=10 * tol)
            assert float((x - y).double().norm()) <= tol * float(y.double().norm()), (pc, dtype)
    gm.close()
    gp.close()


def test_batch_schedule_follows_total_size():
    """Members of a batch run two launches while all of them together are
    small and three otherwise; either way each ends bitwise like alone
    (even order: the per-point table in both encodings)."""
    import torch
    import paper_2108_12188_amd as sem
    say("batch schedules")
    boxes = [box_mesh(4, 3, 3, N, perturb=0.1, seed=600 + N, reorient=True) for N in (4, 5, 7, 9)]
    big = box_mesh(13, 13, 13, 7, perturb=0.1, seed=610)       # above 2^20 points
    for members in (boxes, boxes + [big]):
        gms = [sem.Mesh.from_box(b, g_fp32=False) for b in members]
        bs = [to_dev(random_global_rhs(b, seed=33 + q), torch.float32)
              for q, b in enumerate(members)]
        batch = sem.Batch(gms)
        xs, res = batch.solve(bs, prec=sem.FP32, geom=1, fixed_iters=19)
        for q, gm in enumerate(gms):
            x, r = gm.cg_solve(bs[q], prec=sem.FP32, geom=1, fixed_iters=19)
            assert res[q]["iters"] == r["iters"] == 19
            assert res[q]["rel_res_recursive"] == r["rel_res_recursive"]
            assert torch.equal(xs[q], x), q
        batch.close()
        for gm in gms:
            gm.close()


@pytest.mark.parametrize("fp64", [True, False])
def test_stop_inside_a_chunk(fp64):
    """A solve to a tolerance stops inside a run of two-launch iterations
    (the rest of the run changes nothing), its x holds the last step, and a
    second solve on the same mesh starts afresh; a zero right-hand side and a
    NaN stop at once."""
    import torch
    import paper_2108_12188_amd as sem
    say(f"stop inside a chunk fp64={fp64}")
    mesh = box_mesh(3, 3, 2, 5, perturb=0.1, seed=620)
    gm = sem.Mesh.from_box(mesh, g_fp32=False)
    dtype = torch.float64 if fp64 else torch.float32
    b = to_dev(random_global_rhs(mesh, seed=34), dtype)
    x, r = gm.cg_solve(b, geom=1, tol=1e-3, history=200)
    assert r["converged"] == 1 and r["iters"] % 32 != 0
    assert np.sqrt(r["hist_rho"][-1] / r["hist_rho"][0]) <= 1e-3
    assert np.sqrt(r["hist_rho"][-2] / r["hist_rho"][0]) > 1e-3
    y, s = gm.cg_solve(b, geom=1, fixed_iters=r["iters"], use_graph=False)
    assert torch.equal(x, y)
    z, s = gm.cg_solve(b, geom=1, tol=1e-3, poll_every=7)
    assert s["iters"] == r["iters"] and torch.equal(x, z)
    _, s = gm.cg_solve(torch.zeros_like(b), geom=1, tol=1e-3)
    assert s["iters"] == 0 and s["converged"] == 1
    bad = b.clone()
    bad[7] = float("nan")
    _, s = gm.cg_solve(bad, geom=1, tol=1e-3)
    assert s.get("breakdown") and s["status"] == 3
    w, s = gm.cg_solve(b, geom=1, tol=1e-3)
    assert s["iters"] == r["iters"] and torch.equal(x, w)
    gm.close()


@pytest.mark.parametrize("N", [1, 3, 5, 7, 9])
def test_whole_element_steps(N):
    """Orders whose update steps hold whole elements (128, 16, 4, 2 and 1 of
    them): element counts around one step, alone, in a batch of two-launch
    iterations and in one whose total size takes four.  The partition into
    blocks is the mesh's, so all three give the same bits."""
    import torch
    import paper_2108_12188_amd as sem
    say(f"whole-element steps N={N}")
    per = {1: 128, 3: 16, 5: 4, 7: 2, 9: 1}[N]
    shapes = [(2, 2, k) for k in sorted({1, max(1, per // 4), per // 4 + 1, per // 2 + 1})]
    shapes.append((3, 3, 3))
    boxes = [box_mesh(*s, N, perturb=0.1, seed=41 + q, permute=q % 2 == 1, reorient=q % 2 == 1)
             for q, s in enumerate(shapes)]
    filler = box_mesh(15, 14, 14, 6, perturb=0.1, seed=3)
    assert filler.n_local > 1 << 19
    meshes = [sem.Mesh.from_box(b) for b in boxes + [filler]]
    second = sem.Mesh.from_box(filler)
    bs = [to_dev(random_global_rhs(b, seed=5), torch.float32) for b in boxes + [filler, filler]]
    alone = [m.cg_solve(b, geom=1, fixed_iters=3)[0] for m, b in zip(meshes, bs)]
    k = len(boxes)
    for members in (meshes[:k], meshes + [second]):
        batch = sem.Batch(members)
        xs, infos = batch.solve(bs[:len(members)], prec=sem.FP32, geom=1, fixed_iters=3)
        for x, ref, shape in zip(xs, alone, shapes):
            assert torch.equal(x, ref), (len(members), shape)
        batch.close()
    for m in meshes + [second]:
        m.close()
