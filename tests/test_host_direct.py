"""Edge lists of the two-launch CG iteration on the CPU, point by point
against the copies of every global id (tests/host/direct_tables_check.cpp)."""
import os
import subprocess

import numpy as np
import pytest

from seminputs import box_mesh

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("host") / "direct_tables_check")
    cmd = [HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
           os.path.join(HERE, "host", "direct_tables_check.cpp"),
           os.path.join(ROOT, "paper_2108_12188_amd", "csrc", "sem_tables.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def tied_lines(mesh):
    """The scatter map with every interior line of element edges along z tied
    to the first one: edge groups of 4 q copies, corner groups of up to 8 q."""
    N, gx, gy = mesh.N, mesh.nx * mesh.N + 1, mesh.ny * mesh.N + 1
    g = mesh.glob_id
    x, y, z = g % gx, (g // gx) % gy, g // (gx * gy)
    line = ((x % N == 0) & (x > 0) & (x < gx - 1) & (y % N == 0) & (y > 0) & (y < gy - 1))
    return np.where(line, N + gx * (N + gy * z), g)


def _run(checker, tmp_path, mesh, gid):
    g, d = str(tmp_path / "gid.bin"), str(tmp_path / "dir.bin")
    np.ascontiguousarray(gid, dtype=np.int64).tofile(g)
    np.ascontiguousarray(mesh.dirichlet, dtype=np.uint8).tofile(d)
    r = subprocess.run([checker, str(mesh.E), str(mesh.N), g, d, "12188"], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return {k: int(v) for k, v in (kv.split("=") for kv in r.stdout.split())}


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7, 9, 11])
@pytest.mark.parametrize("tied", [False, True])
def test_edge_lists_sum_every_group(checker, tmp_path, N, tied):
    mesh = box_mesh(4, 3, 2, N, perturb=0.1, seed=70 + N, reorient=True, permute=True)
    out = _run(checker, tmp_path, mesh, tied_lines(mesh) if tied else mesh.glob_id)
    assert out["direct"] == 1
    assert out["checked"] > 0
    assert (out["generic"] > 0) == tied


def test_groups_off_the_edges_decline(checker, tmp_path):
    mesh = box_mesh(3, 2, 2, 4, perturb=0.1, seed=7)
    P = mesh.N + 1
    gid = mesh.glob_id.copy()
    gid[5, P * (2 + P * 2)] = gid[0, mesh.N + P * (2 + P * 2)]
    assert _run(checker, tmp_path, mesh, gid)["direct"] == 0
