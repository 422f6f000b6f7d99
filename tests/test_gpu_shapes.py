"""The largest shapes of the VALU operator, whose padded tiles take more than
64 KiB of LDS: the same bits from the plain operator as the default shape, the
same iterates up to the order of the partial sums."""
import pytest

from gpu_common import say, to_dev
from seminputs import box_mesh, random_global_rhs, random_local

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,fp64,epb", [(7, True, 8), (9, True, 4), (9, False, 4)])
@pytest.mark.parametrize("geom", [0, 1])
def test_largest_shapes(N, fp64, epb, geom):
    import torch
    import paper_2108_12188_amd as sem
    say(f"N={N} fp64={fp64} {epb} elements per block, geom={geom}")
    prec, dtype = (sem.FP64, torch.float64) if fp64 else (sem.FP32, torch.float32)
    mesh = box_mesh(*((5, 4, 3) if epb == 8 else (7, 3, 3)), N, perturb=0.1, seed=N)
    assert mesh.E % epb                                      # a ragged last block
    gm = sem.Mesh.from_box(mesh, g_fp32=not fp64, g_fp64=fp64)
    u = to_dev(random_local(mesh.n_local, seed=3), dtype)
    b = to_dev(random_global_rhs(mesh, seed=4), dtype)

    def both():
        w = gm.ax(u, geom=geom)
        x, _ = gm.cg_solve(b, geom=geom, fixed_iters=5)
        torch.cuda.synchronize()
        return w, x

    sem.ax_engine_set(N, prec, geom, sem.ENGINE_VALU)
    try:
        w0, x0 = both()
        sem.ax_shape_set(N, prec, geom, epb)
        assert sem.ax_shape_get(N, prec, geom)["elems_per_block"] == epb
        w1, x1 = both()
    finally:
        sem.ax_shape_set(N, prec, geom, 0)
        sem.ax_engine_set(N, prec, geom, sem.ENGINE_DEFAULT)
    assert torch.equal(w0, w1)
    # five iterations whose scalars differ by the order of FP64 sums
    tol = 1e-12 if fp64 else 1e-5
    assert float((x0 - x1).double().norm()) <= tol * float(x0.double().norm())
    gm.close()


@pytest.mark.parametrize("N,fp64,geom", [(2, False, 1), (2, True, 1), (3, True, 0), (6, True, 0)])
def test_plain_default_shape(N, fp64, geom):
    """The plain operator's own default shape gives the bits of the CG-fused
    one's, on full and ragged blocks."""
    import torch
    import paper_2108_12188_amd as sem
    say(f"plain default shape N={N} fp64={fp64} geom={geom}")
    prec, dtype = (sem.FP64, torch.float64) if fp64 else (sem.FP32, torch.float32)
    for n in ((1, 1, 1), (7, 2, 2), (5, 4, 3), (29, 1, 1)):
        mesh = box_mesh(*n, N, perturb=0.1, seed=N)
        gm = sem.Mesh.from_box(mesh, g_fp32=not fp64, g_fp64=fp64)
        u = to_dev(random_local(mesh.n_local, seed=3), dtype)
        w0 = gm.ax(u, geom=geom)
        sem.ax_shape_set(N, prec, geom, sem.ax_shape_get(N, prec, geom)["elems_per_block"])
        try:
            w1 = gm.ax(u, geom=geom)
            torch.cuda.synchronize()
        finally:
            sem.ax_shape_set(N, prec, geom, 0)
        assert torch.equal(w0, w1), n
        gm.close()
