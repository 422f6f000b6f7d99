"""The set-up kernels (operator diagonal, coordinates) at every built order,
with element counts that leave the last block of a launch partly empty."""
import numpy as np
import pytest

import oracle
from gpu_common import say, to_host
from seminputs import box_mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 3, 1), (13, 5, 1)])
@pytest.mark.parametrize("N", range(1, 12))
def test_diag_and_coords_every_order(N, shape):
    """Blocks take 256 / P^2 elements (64 at N = 1, one at N = 11): 1, 15 and
    65 elements end inside a block for every order that packs several.

    Coordinates are convex combinations of corners in [0, 1.1]: 8 products of
    three rounded factors, below 1e-14.  A diagonal entry is a sum of 3 P
    terms of one sign and 3 smaller mixed ones; both sides round D (about
    N^2 eps each) and the factors, below 1e-12 relative."""
    import paper_2108_12188_amd as sem
    say(f"setup N={N} shape={shape}")
    mesh = box_mesh(*shape, N, perturb=0.1, seed=31 + N, permute=True, reorient=True)
    pr = oracle.Problem(mesh)
    gm = sem.Mesh.from_box(mesh)
    xyz = to_host(gm.coords())
    assert np.max(np.abs(xyz.reshape(3, -1) - pr.coords())) < 1e-14
    np.testing.assert_allclose(to_host(gm.diag()), pr.diag_A(), rtol=1e-12)
    gm.close()
