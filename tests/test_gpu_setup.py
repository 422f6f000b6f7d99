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


def _odd_groups(N, seed, dirichlet):
    """A 4x3x2 box whose local points are joined at random into groups of 1,
    2, 3, 4, 5, 8 and 11 copies, one group in five on the Dirichlet boundary."""
    mesh = box_mesh(4, 3, 2, N, perturb=0.1, seed=seed)
    rng = np.random.default_rng(seed)
    order = rng.permutation(mesh.n_local)
    gid = np.empty(mesh.n_local, np.int64)
    at = g = 0
    while at < mesh.n_local:
        m = int(rng.choice([1, 2, 3, 4, 5, 8, 11]))
        gid[order[at:at + m]] = g
        at, g = at + m, g + 1
    d = (rng.random(g) < 0.2).astype(mesh.dirichlet.dtype)[gid] if dirichlet \
        else np.zeros(mesh.n_local, mesh.dirichlet.dtype)
    return mesh.vert, gid.reshape(mesh.glob_id.shape), d.reshape(mesh.dirichlet.shape), g


@pytest.mark.parametrize("dirichlet", [True, False])
@pytest.mark.parametrize("groups", ["box", "odd", "none"])
def test_mask_and_rhs_in_one_launch(groups, dirichlet):
    """mask(QQ^T w) and mask(QQ^T (B f)) over every group size, without
    groups and without Dirichlet points.  The sums keep the order of the
    oracle's, so FP64 is bitwise the oracle's; a mask clears infinities and
    NaN.  A right-hand side over its own input goes through memory and has to
    give the same bits."""
    import ctypes as C
    import torch
    import paper_2108_12188_amd as sem
    say(f"mask and rhs groups={groups} dirichlet={dirichlet}")
    N = 4
    if groups == "odd":
        vert, gid, d, ng = _odd_groups(N, 7, dirichlet)
    else:
        box = box_mesh(*((1, 1, 1) if groups == "none" else (4, 3, 5)), N, perturb=0.1, seed=7)
        vert, gid, ng = box.vert, box.glob_id, box.n_glob
        d = box.dirichlet if dirichlet else np.zeros_like(box.dirichlet)
    gm = sem.Mesh(vert, gid, d, N)
    rng = np.random.default_rng(3)
    w = rng.uniform(-1, 1, gm.n)
    off = d.ravel() != 0

    def mask_gs(v):
        out = np.asarray(oracle.gs(gid, ng, v)).ravel().copy()
        out[off] = 0.0
        return out

    bad = w.copy()
    bad[off] = np.where(rng.random(off.sum()) < 0.5, np.nan, np.inf)
    got = to_host(gm.gs(torch.as_tensor(bad, device="cuda"), mask=True))
    np.testing.assert_array_equal(got, mask_gs(w))
    g32 = gm.gs(torch.as_tensor(w, device="cuda").float(), mask=True)
    s32 = gm.gs(torch.as_tensor(w, device="cuda").float(), mask=False)
    s32[torch.as_tensor(off, device="cuda")] = 0
    assert torch.equal(g32, s32)

    f = torch.as_tensor(w, device="cuda")
    B = np.asarray(oracle.geom(vert, N)[1]).ravel()
    b64 = gm.rhs(f, prec=sem.FP64)
    # the oracle's mass may round differently: m <= 11 terms of 1e-14 each
    ref = mask_gs(B * w)
    bound = 2e-13 * np.max(np.abs(B))
    assert np.max(np.abs(to_host(b64) - ref)) <= bound
    assert torch.equal(gm.rhs(f, prec=sem.FP32), b64.float())
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    assert torch.equal(gm.rhs(f, prec=sem.FP32, stream=stream), b64.float())
    for prec, dt in ((sem.FP64, torch.float64), (sem.FP32, torch.float32)):
        buf = f.clone()
        s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert sem.lib().sem_rhs(gm.handle, prec, C.c_void_p(buf.data_ptr()),
                                 C.c_void_p(buf.data_ptr()), s) == 0
        assert torch.equal(buf.view(dt)[:gm.n], b64.to(dt))
    gm.close()
