"""The CG-fused operator over several tiles per block: meshes with more
elements than the fused grid holds at once (and a remainder), at every order,
in both precisions and G forms.  Three CG iterations are compared with
Algorithm 1 written out in FP64 from the plain operator, the gather-scatter
and the weighted dot, each of which has its own parity test."""
import pytest

from gpu_common import say, to_dev
from seminputs import box_mesh, random_global_rhs

pytestmark = pytest.mark.gpu

ITERS = 3


def _reference(gm, b, geom):
    import torch
    x = torch.zeros_like(b)
    r, p = b.clone(), torch.zeros_like(b)
    rho, beta = gm.dot(r, r), 0.0
    for _ in range(ITERS):
        p = r + beta * p
        w = gm.gs(gm.ax(p, geom=geom))
        alpha = rho / gm.dot(p, w)
        x += alpha * p
        r -= alpha * w
        new = gm.dot(r, r)
        beta, rho = new / rho, new
    return x


# elements per axis: more tiles than the 2048 (FP32) or 4096 (FP64) blocks of
# the fused grid at the order's elements per block, not a multiple of them
@pytest.mark.parametrize("N,n", [(1, (67, 63, 65)), (2, (50, 49, 48)), (3, (41, 42, 40)),
                                 (4, (28, 29, 27)), (5, (31, 32, 30)), (6, (28, 27, 29)),
                                 (7, (26, 25, 27)), (8, (19, 20, 18)), (9, (17, 16, 16)),
                                 (10, (17, 16, 16)), (11, (17, 16, 16))])
def test_fused_operator_many_tiles(N, n):
    import torch
    import paper_2108_12188_amd as sem
    say(f"fused operator N={N} {n}")
    mesh = box_mesh(*n, N, perturb=0.1, seed=500 + N)
    gm = sem.Mesh.from_box(mesh, g_fp32=True, g_fp64=True)
    bh = random_global_rhs(mesh, seed=90 + N)
    for geom in (0, 1):
        b = to_dev(bh, torch.float64)
        ref = _reference(gm, b, geom)
        norm = float(ref.norm())
        # rounding of three FP64 iterations; FP32: the operator's bound of
        # 1e-5 per application
        for dtype, tol in ((torch.float64, 1e-12), (torch.float32, ITERS * 1e-5)):
            x, res = gm.cg_solve(b.to(dtype), geom=geom, fixed_iters=ITERS)
            assert res["iters"] == ITERS
            assert float((x.double() - ref).norm()) <= tol * norm, (N, geom, dtype)
    gm.close()
