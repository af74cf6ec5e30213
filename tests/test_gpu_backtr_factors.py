"""Triangular factors of the reflector blocks: orders at the edges of the 16- and
64-reflector blocks and of the compact-WY blocks, one matrix and batches on both
sides of the block count."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce, dev, host, stream_handle

pytestmark = pytest.mark.gpu


def hermitian(rng, n, cplx, batch=1):
    a = rng.normal(size=(batch, n, n))
    if cplx:
        a = a + 1j * rng.normal(size=(batch, n, n))
    return 0.5 * (a + a.conj().swapaxes(1, 2))


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n", [4, 16, 17, 18, 33, 34, 64, 65, 66, 81, 128, 129, 130, 192, 193, 194, 256, 257, 258, 385])
def test_similarity(n, cplx):
    """Q unitary and Q T Q^H = A, at the bars of the other orders (1e-12, times n
    and the largest entry for the product)."""
    announce("back-transform factors", n, cplx)
    lib = ks.lib()
    V, I32 = ctypes.c_void_p, ctypes.c_int32
    lib.ks_test_hetrd.argtypes = [I32, I32, V, V, V, V, I32, V, V]
    lib.ks_test_hetrd.restype = I32
    A = hermitian(np.random.default_rng(n), n, cplx)[0]
    Ad, X = dev(A), dev(np.eye(n))
    d = torch.zeros(n, dtype=torch.float64, device="cuda")
    e = torch.zeros(n, dtype=torch.float64, device="cuda")
    Y = torch.zeros((n, n), dtype=Ad.dtype, device="cuda")
    P = lambda t: V(t.data_ptr())  # noqa: E731
    assert lib.ks_test_hetrd(int(cplx), n, P(Ad), P(d), P(e), P(X), n, P(Y), stream_handle()) == 0
    Q, eh = host(Y), host(e)[:n - 1]
    T = np.diag(host(d)) + np.diag(eh, 1) + np.diag(eh, -1)
    assert np.abs(Q.conj().T @ Q - np.eye(n)).max() < 1e-12
    assert np.abs(Q @ T @ Q.conj().T - A).max() < 1e-12 * max(1.0, np.abs(A).max()) * n


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n,batch", [(65, 3), (130, 2), (200, 3), (300, 2), (300, 5), (520, 3)])
def test_batches(n, batch, cplx):
    """Each matrix of a batch against numpy: eigenvalues to 1e-10, H C = C diag(eps)
    and C^H C = 1 to 1e-11, as elsewhere."""
    announce("back-transform batch", n, batch, cplx)
    H = hermitian(np.random.default_rng(n + batch), n, cplx, batch)
    S = np.broadcast_to(np.eye(n, dtype=H.dtype), H.shape).copy()
    plan = ks.Plan(n, batch=batch, complex=cplx)
    out = plan.solve(dev(H), dev(S), float(n // 2), 0.05)
    eps, C = host(out["eps"]).reshape(batch, n), host(out["C"]).reshape(batch, n, n)
    plan.close()
    scale = np.abs(eps).max()
    for b in range(batch):
        assert np.abs(eps[b] - np.linalg.eigvalsh(H[b])).max() < 1e-10
        assert np.abs(C[b].conj().T @ C[b] - np.eye(n)).max() < 1e-11
        assert np.abs(H[b] @ C[b] - C[b] * eps[b]).max() < 1e-11 * scale
