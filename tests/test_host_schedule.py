"""Which launches a CG iteration takes, on the CPU
(tests/host/schedule_check.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("host") / "schedule_check")
    r = subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
                        os.path.join(HERE, "host", "schedule_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _rows(checker, N, fp64, sizes, pc=False):
    out = subprocess.run([checker, str(N), str(int(fp64)), str(int(pc)), *map(str, sizes)],
                         capture_output=True, text=True, check=True).stdout
    return [tuple(map(int, line.split(":"))) for line in out.split()]


@pytest.mark.parametrize("N", range(1, 12))
@pytest.mark.parametrize("fp64", [False, True])
def test_update_blocks_of_three_launches(checker, N, fp64):
    """No more partials than one round of loads of the operator's smallest
    block reads (1024 by the matrix-core blocks of 64 and 128 threads, 2048 by
    the others), and no block of more steps than the fewest that allows."""
    P3 = (N + 1) ** 3
    sizes = [e * P3 for e in range((1 << 20) // P3, (1 << 22) // P3 + 2, max(1, 4096 // P3))]
    most = 1024 if N in (7, 9) and not fp64 else 2048
    seen = 0
    for n, launches, blocks in _rows(checker, N, fp64, sizes):
        if launches != 3:
            continue
        seen += 1
        vec = -(-n // 1024)
        assert 0 < blocks <= most, n
        assert -(-vec // blocks) <= -(-vec // min(most, 1280)), n
    assert seen > 0 or N in (1, 3)


# last and first size of each schedule, as measured
@pytest.mark.parametrize("N,fp64,n,launches", [
    (1, False, 1 << 17, 2), (1, True, (1 << 17) + 8, 3), (2, False, 1 << 18, 2),
    (2, False, (1 << 18) + 27, 3), (3, True, 1 << 19, 2), (3, False, (1 << 19) + 64, 3),
    (4, False, 1 << 20, 2), (5, False, 1 << 20, 2), (5, False, (1 << 20) + 216, 3), (5, False, 3 << 20, 3),
    (5, False, (3 << 20) + 216, 4), (8, False, 3582 * 1000, 4), (6, False, 3177 * 1000, 4),
    (9, False, 1 << 22, 3), (9, False, (1 << 22) + 1000, 4), (7, False, (1 << 20) + 512, 4),
    (7, False, (1 << 21) - 512, 4), (7, False, 1 << 21, 3), (7, False, 1 << 22, 3),
    (7, True, 1 << 21, 3), (7, True, (1 << 21) + 512, 4), (1, True, 1 << 20, 3),
    (1, True, (1 << 20) + 8, 4), (1, False, (1 << 20) + 8, 3), (3, False, 1 << 20, 3),
    (3, False, (1 << 20) + 64, 4), (3, True, (1 << 20) + 64, 3)])
def test_limits(checker, N, fp64, n, launches):
    assert _rows(checker, N, fp64, [n])[0][1] == launches


@pytest.mark.parametrize("N,fp64,n,launches", [
    (7, False, 1 << 20, 2), (7, False, 1 << 21, 4), (7, False, 1 << 22, 4), (7, True, 1 << 21, 3),
    (5, False, 1 << 21, 3), (5, False, (1 << 21) + 216, 4), (9, False, 1 << 22, 3),
    (8, False, 3 << 20, 3)])
def test_limits_preconditioned(checker, N, fp64, n, launches):
    assert _rows(checker, N, fp64, [n], pc=True)[0][1] == launches
