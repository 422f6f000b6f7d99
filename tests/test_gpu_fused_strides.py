"""The CG-fused operator over several tiles per block at N = 8, where the mesh of
test_gpu_ax_fused leaves one tile per block in FP64."""
import pytest

from gpu_common import say, to_dev
from seminputs import box_mesh, random_global_rhs
from test_gpu_ax_fused import ITERS, _reference

pytestmark = pytest.mark.gpu

GRID = {"fp32": 2048, "fp64": 4096}     # most blocks of the VALU operator


@pytest.mark.parametrize("N,n", [(8, (24, 23, 25))])
def test_more_tiles_than_blocks(N, n):
    import torch
    import paper_2108_12188_amd as sem
    say(f"fused operator N={N} {n}")
    mesh = box_mesh(*n, N, perturb=0.1, seed=500 + N)
    gm = sem.Mesh.from_box(mesh, g_fp32=True, g_fp64=True)
    bh = random_global_rhs(mesh, seed=90 + N)
    for geom in (0, 1):
        b = to_dev(bh, torch.float64)
        ref = _reference(gm, b, geom)
        # the tolerances of test_fused_operator_many_tiles
        for prec, name, dtype, tol in ((sem.FP64, "fp64", torch.float64, 1e-12),
                                       (sem.FP32, "fp32", torch.float32, ITERS * 1e-5)):
            epb = sem.ax_shape_get(N, prec, geom)["elems_per_block"]
            assert sem.ax_engine_get(N, prec, geom) == sem.ENGINE_VALU
            tiles = -(-mesh.E // epb)
            assert tiles > GRID[name] and tiles % GRID[name]
            x, res = gm.cg_solve(b.to(dtype), geom=geom, fixed_iters=ITERS)
            assert res["iters"] == ITERS
            assert float((x.double() - ref).norm()) <= tol * float(ref.norm()), (geom, name)
    gm.close()
