"""The FP64 right-hand side on both sides of the size where it goes from one
launch to two: bitwise that of the product summed in place."""
import ctypes as C

import pytest

from gpu_common import say
from seminputs import box_mesh, random_local

pytestmark = pytest.mark.gpu


# below and above 2^22 points (N = 1), 3 * 2^19 (2, 3, 4) and 2^21
@pytest.mark.parametrize("N,n", [(1, (80, 80, 81)), (1, (81, 81, 80)), (2, (38, 38, 40)),
                                 (2, (39, 39, 39)), (3, (29, 29, 29)), (3, (29, 29, 30)),
                                 (4, (23, 23, 23)), (4, (23, 23, 24)), (5, (21, 21, 22)),
                                 (5, (21, 22, 22)), (7, (16, 16, 16)), (7, (16, 16, 17)),
                                 (8, (14, 14, 14)), (8, (14, 14, 15)), (9, (12, 13, 13)),
                                 (9, (13, 13, 13)), (11, (3, 2, 2))])
def test_routes_agree(N, n):
    import torch
    import paper_2108_12188_amd as sem
    say(f"rhs N={N} {n}")
    mesh = box_mesh(*n, N, perturb=0.1, seed=N)
    gm = sem.Mesh.from_box(mesh)
    f = torch.as_tensor(random_local(mesh.n_local, seed=5), dtype=torch.float64, device="cuda")
    b = gm.rhs(f)
    b32 = gm.rhs(f, prec=sem.FP32)
    # over its own input: always the stored product
    g = f.clone()
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert sem.lib().sem_rhs(gm.handle, sem.FP64, C.c_void_p(g.data_ptr()),
                             C.c_void_p(g.data_ptr()), stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(b, g)
    assert torch.equal(b32, g.float())
    gm.close()
