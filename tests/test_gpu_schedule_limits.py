"""CG on both sides of the limits that depend on the order: two launches at
N = 1, 2 and 3, three at N = 3, 6, 8 and, preconditioned, 5 and 7."""
import pytest

from test_gpu_schedules import test_schedules_agree_at_their_limits as _agree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n", [(1, (25, 25, 26)), (1, (26, 26, 25)), (2, (21, 21, 22)),
                                 (2, (22, 22, 21)), (3, (20, 20, 20)), (3, (20, 20, 21)),
                                 (1, (51, 51, 51)), (3, (26, 25, 26)), (5, (21, 21, 22)),
                                 (5, (21, 22, 22)), (6, (20, 21, 21)), (6, (20, 21, 22)),
                                 (8, (16, 16, 17)), (7, (16, 16, 17)), (9, (15, 15, 16))])
def test_schedules_agree(N, n):
    _agree(N, n)
