"""The FP32 right-hand side on a stream of its own: it returns before the
launch has run, so neither its source nor its result may be touched early."""
import pytest

from gpu_common import say
from seminputs import box_mesh, random_local

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("own", [True, False])
def test_source_lives_until_it_is_read(own):
    """f belongs to another stream and is dropped right after the call, while
    the launch still waits; what is allocated there next must not be f."""
    import torch
    import paper_2108_12188_amd as sem
    say(f"rhs source on another stream, own={own}")
    mesh = box_mesh(6, 5, 4, 7, perturb=0.1, seed=3)
    gm = sem.Mesh.from_box(mesh)
    src = torch.as_tensor(random_local(mesh.n_local, seed=4), dtype=torch.float64, device="cuda")
    ref = gm.rhs(src, prec=sem.FP32)
    torch.cuda.synchronize()
    mine, run = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(mine):
        f = src.clone()
    torch.cuda.synchronize()
    with torch.cuda.stream(run):
        torch.cuda._sleep(200_000_000)
    if own:
        with torch.cuda.stream(run):
            b = gm.rhs(f, prec=sem.FP32)
    else:
        b = gm.rhs(f, prec=sem.FP32, stream=run)
    del f
    with torch.cuda.stream(mine):
        g = torch.full_like(src, float("nan"))
    if own:
        run.synchronize()
    assert torch.equal(b, ref)               # the current stream waits by itself
    torch.cuda.synchronize()
    assert bool(torch.isnan(g).all())
    gm.close()
