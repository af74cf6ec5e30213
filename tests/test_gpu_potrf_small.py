"""Cholesky blocks of real matrices on both sides of the order from which panels take
over, alone and as the last block."""
import numpy as np
import pytest

from tests.gpu_helpers import announce
from tests.test_gpu_potrf_leaf import definite, factor
from tests.test_gpu_stages import L  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 27, 28, 29, 64 + 1, 64 + 28, 64 + 29])
def test_line(L, n):  # noqa: F811
    """L L^T = A to n units of rounding (of 2^-53, eightfold) of A, whose condition is
    below 10, L L^-1 = 1 alike; a bad last pivot is found."""
    announce("potrf line", n)
    A = definite(n, False)
    st, Lo, Li, info = factor(L, A)
    assert st == 0 and info == 0
    eps = 8 * (n + 8) * 2.0 ** -53
    assert np.abs(Lo @ Lo.T - A).max() <= eps * np.abs(A).max()
    assert np.abs(Lo @ Li - np.eye(n)).max() <= 10 * eps
    A[n - 1, n - 1] = -1e6
    assert factor(L, A)[3] == n
