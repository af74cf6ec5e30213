"""Leaves and small merges of the divide and conquer (one workgroup each, in LDS):
orders at the edges of the leaf's halves, of a leaf and of the largest merge that
takes the LDS form, with ties, deflation and graded entries."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce, dev, host, stream_handle

pytestmark = pytest.mark.gpu


def run_stedc(d, e):
    lib = ks.lib()
    V, I32 = ctypes.c_void_p, ctypes.c_int32
    lib.ks_test_stedc.argtypes = [I32, V, V, V, V, ctypes.POINTER(I32), V]
    lib.ks_test_stedc.restype = I32
    n = len(d)
    dd, ee = dev(np.asarray(d, float)), dev(np.concatenate([np.asarray(e, float), [0.0]]))
    lam = torch.zeros(n, dtype=torch.float64, device="cuda")
    Z = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    info = I32(0)
    P = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    assert lib.ks_test_stedc(n, P(dd), P(ee), P(lam), P(Z), ctypes.byref(info), stream_handle()) == 0
    return host(lam), host(Z), info.value


def draw(kind, n):
    rng = np.random.default_rng(n)
    d, e = rng.normal(size=n), rng.normal(size=max(n - 1, 0))
    if kind == "ties":          # equal entries and decoupled pieces: whole merges deflate, some by rotations
        d, e = np.round(d), 1e-3 * e
        e[::5] = 0.0
    elif kind == "graded":      # twelve orders of magnitude, both ways
        d *= 10.0 ** (-12 * np.abs(np.linspace(-1, 1, n)))
        e *= 10.0 ** (-12 * np.abs(np.linspace(-1, 1, n)))[1:]
    elif kind == "constant":    # 2 on the diagonal, -1 beside it
        d, e = np.full(n, 2.0), np.full(max(n - 1, 0), -1.0)
    elif kind == "diagonal":
        e = np.zeros_like(e)
    elif kind == "tiny":        # squares below the range
        d, e = d * 1e-170, e * 1e-170
    return d, e


@pytest.mark.parametrize("kind", ["random", "ties", "graded", "constant", "diagonal", "tiny"])
@pytest.mark.parametrize("n", [1, 2, 3, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 192, 193])
def test_small_orders(kind, n):
    """Eigenvalues against the oracle's Jacobi and T Z = Z diag(lam) to 1e-11 of the
    largest entry, Z orthogonal to 1e-12: the bars of the larger orders."""
    announce("small divide and conquer", kind, n)
    d, e = draw(kind, n)
    lam, Z, info = run_stedc(d, e)
    assert info == 0
    T = np.diag(d) + np.diag(e, 1) + np.diag(e, -1) if n > 1 else np.diag(d)
    scale = np.abs(T).max() if kind == "tiny" else max(1.0, np.abs(T).max())
    unit = scale if kind == "tiny" else 1.0
    w, _, _ = O.jacobi(T / unit)
    assert np.all(np.diff(lam) >= 0)
    assert np.abs(lam / unit - w).max() < 1e-11 * (scale / unit)
    assert np.abs(Z.T @ Z - np.eye(n)).max() < 1e-12
    assert np.abs((T / unit) @ Z - Z * (lam / unit)).max() < 1e-11 * (scale / unit)
