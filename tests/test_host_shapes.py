"""Elements per block of the VALU operator that the library accepts, on the
CPU: every shape of up to 512 threads and 64 KiB of element values, whatever
padding its tiles have, and the shapes the tuner times are those."""
import pytest

import paper_2108_12188_amd as sem
from paper_2108_12188_amd import tune


@pytest.mark.parametrize("N", range(1, 12))
@pytest.mark.parametrize("prec", [sem.FP32, sem.FP64])
def test_accepted_shapes(N, prec):
    P2, P3 = (N + 1) ** 2, (N + 1) ** 3
    size = 8 if prec == sem.FP64 else 4
    staged = 8 * P3 + 96 if prec == sem.FP32 and P3 % 4 == 0 else 0
    most = 1
    while -(-(most + 1) * P2 // 64) * 64 <= 512 and \
            (most + 1) * (2 * size * P3 + staged) <= 65536:
        most += 1
    for geom in (sem.PRECOMPUTED, sem.ON_THE_FLY):
        engine = sem.ax_engine_get(N, prec, geom)
        sem.ax_engine_set(N, prec, geom, sem.ENGINE_VALU)
        try:
            for epb in range(1, most + 3):
                sem.ax_shape_set(N, prec, geom, epb)
                got = sem.ax_shape_get(N, prec, geom)
                assert got["elems_per_block"] == min(epb, most)
                assert got["threads"] == -(-min(epb, most) * P2 // 64) * 64
                # the padded tiles: what the CU has, with two blocks on it
                assert 2 * got["lds_bytes"] <= 160 * 1024
        finally:
            sem.ax_shape_set(N, prec, geom, 0)
            sem.ax_engine_set(N, prec, geom, sem.ENGINE_DEFAULT)
        assert sem.ax_engine_get(N, prec, geom) == engine
    assert tune.candidates(N, prec == sem.FP64) == list(range(1, most + 1))
