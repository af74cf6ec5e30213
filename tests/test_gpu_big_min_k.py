"""The large-tile threshold that a caller sets holds in the back-transform of complex
plans too."""
import ctypes

import pytest

from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce
from tests.test_gpu_gang import check_pencil, pencil, solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cplx", [False, True])
def test_threshold(cplx):
    """Four matrices of order 1100 complex or 2100 real: the reduction (inner dimension the
    order) and the back-transform (blocks of 128 or 256 reflectors) have the 1024 tiles
    that large ones start from, the tridiagonalisation has no products."""
    announce("large-tile threshold", cplx)
    count = ks.lib().ks_test_big_gemms
    count.restype = ctypes.c_int64
    n = 1100 if cplx else 2100
    H, S = pencil(n, cplx, 4, 3)
    plan = ks.Plan(n, batch=4, complex=cplx)
    base = plan.tuning_knobs()
    used = {}
    for block in (128, 256):
        for k in (64, 128, 129, 256, 257, 1000, ks.KS_TUNE_NEVER):
            plan.set_tuning(dict(base, gemm_big_min_k=k, backtr_block=block))
            before = count()
            eps, C = solve(plan, H, S)
            used[block, k] = count() - before
            check_pencil(H, S, eps, C)
    assert used[128, ks.KS_TUNE_NEVER] == used[256, ks.KS_TUNE_NEVER] == 0
    # blocks of 128 reflectors: from a threshold of 128 down, or with the default for complex data
    assert used[128, 64] >= used[128, 128] > used[128, 129] >= used[128, 257] >= used[128, 1000] > 0
    assert used[128, 256] == used[128, 128 if cplx else 257]
    # blocks of 256 reflectors: from a threshold of 256 down
    assert used[256, 129] >= used[256, 256] > used[256, 257] >= used[256, 1000] > 0
