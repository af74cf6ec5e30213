"""Cholesky factor and inverse of the blocks that one workgroup does: orders at the edges of
its 16-column panels and of the block, indefinite pivots in each panel."""
import ctypes

import numpy as np
import pytest
import torch

from tests.gpu_helpers import announce, dev, host, stream_handle
from tests.test_gpu_stages import L, P  # noqa: F401

pytestmark = pytest.mark.gpu


def factor(lib, A):
    n = A.shape[0]
    Ad, Li, info = dev(A), torch.full(A.shape, 7.0, dtype=dev(A).dtype, device="cuda"), ctypes.c_int32(0)
    st = lib.ks_test_potrf(int(np.iscomplexobj(A)), n, P(Ad), n, P(Li), ctypes.byref(info), stream_handle())
    return st, np.tril(host(Ad)), host(Li), info.value


def definite(n, cplx, scale=1.0):
    rng = np.random.default_rng(n)
    X = rng.normal(size=(n, n)) + (1j * rng.normal(size=(n, n)) if cplx else 0)
    return scale * (X @ X.conj().T + n * np.eye(n))


@pytest.mark.parametrize("scale", [1.0, 1e-300, 1e300])
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 128, 130])
def test_factor_and_inverse(L, n, cplx, scale):  # noqa: F811
    """L L^H = A to n units of rounding (of 2^-53, eightfold) of A, whose condition is
    below 10, L L^-1 = 1 alike, zeros above the diagonal of the inverse."""
    announce("potrf leaf", n, cplx, scale)
    A = definite(n, cplx, scale)
    st, Lo, Li, info = factor(L, A)
    assert st == 0 and info == 0
    eps = 8 * (n + 8) * 2.0 ** -53
    assert np.abs(Lo @ Lo.conj().T - A).max() <= eps * np.abs(A).max()
    assert np.abs(Lo @ Li - np.eye(n)).max() <= 10 * eps
    assert np.all(Li[np.triu_indices(n, 1)] == 0)


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n,j", [(1, 0), (16, 15), (33, 16), (64, 0), (64, 31), (64, 32), (64, 63), (130, 70)])
@pytest.mark.parametrize("bad", [-1e6, float("nan"), float("inf")])
def test_failing_column(L, n, j, cplx, bad):  # noqa: F811
    announce("potrf leaf", n, j, cplx, bad)
    A = definite(n, cplx)
    A[j, j] = bad
    assert factor(L, A)[3] == j + 1
