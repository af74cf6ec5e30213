"""The last columns of the tridiagonalisation in registers: orders at the edges of
the shapes of its gangs, the kernels behind a gang that could not gather, whole
solves in batches, in the mixed form and on two streams at once."""
import ctypes
import threading

import numpy as np
import pytest
import torch

from paper_2606_09058_amd import inputs as I
from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce, dev, stream_handle

pytestmark = pytest.mark.gpu


@pytest.fixture()
def L():
    lib = ks.lib()
    V, I32 = ctypes.c_void_p, ctypes.c_int32
    lib.ks_test_hetrd.argtypes = [I32, I32, V, V, V, V, I32, V, V]
    lib.ks_test_hetrd.restype = I32
    lib.ks_test_set_gang_leave.argtypes = [I32]
    lib.ks_test_set_gang_leave.restype = I32
    yield lib
    assert lib.ks_test_set_gang_leave(0) == 0


def P(t):
    return ctypes.c_void_p(t.data_ptr())


def hetrd(L, A0, cplx):
    n = A0.shape[0]
    A, X = A0.clone(), torch.eye(n, dtype=torch.float64, device="cuda")
    d = torch.zeros(n, dtype=torch.float64, device="cuda")
    e = torch.zeros(n, dtype=torch.float64, device="cuda")
    Y = torch.zeros_like(A)
    st = L.ks_test_hetrd(int(cplx), n, P(A), P(d), P(e), P(X), n, P(Y), stream_handle())
    torch.cuda.synchronize()
    return st, d, e[:n - 1], Y


def check_similarity(L, n, cplx):
    """Q unitary to 1e-12 and Q T Q^H = A to 1e-12 max|A| n: n reflectors, each
    with a backward error of a few units in the last place of A's norm."""
    A0 = dev(I.random_hermitian(np.random.default_rng(n), n, cplx))
    st, d, e, Q = hetrd(L, A0, cplx)
    assert st == 0
    T = (torch.diag(d) + torch.diag(e, 1) + torch.diag(e, -1)).to(A0.dtype)
    Qh = Q.mH.contiguous()
    assert (Qh @ Q - torch.eye(n, dtype=A0.dtype, device="cuda")).abs().max().item() < 1e-12
    assert ((Q @ T) @ Qh - A0).abs().max().item() < 1e-12 * max(1.0, A0.abs().max().item()) * n


@pytest.mark.parametrize("cplx,n", [(False, n) for n in (64, 65, 128, 129, 200, 256, 257, 512, 513, 1024, 1025, 2048,
                                                         2049, 2560, 2561, 3072, 3105)] +
                         [(True, n) for n in (64, 65, 128, 129, 256, 257, 300, 512, 513, 1024, 1025, 1536, 1537, 1792, 1793,
                                              2048, 2081)])
def test_edges_of_the_shapes(L, cplx, n):
    announce("gang", cplx, n)
    check_similarity(L, n, cplx)


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("level,n", [(1, 1025), (1, 1700), (1, 2300), (2, 129), (2, 333), (2, 1030)])
def test_gangs_that_leave(L, cplx, level, n):
    """The form in memory (level 1) and the single workgroup (level 2) do the
    columns of gangs that left."""
    announce("gang leaves", cplx, level, n)
    assert L.ks_test_set_gang_leave(level) == 0
    check_similarity(L, n, cplx)


@pytest.mark.parametrize("n", [100, 300, 1100])
@pytest.mark.parametrize("bits", [0x7FF8000000000000, 0x7FF4A5A5DEADBEEF])
def test_nan_ends(L, n, bits):
    """A NaN spreads through the exchange and every wait ends, also for the bits
    that mark an empty entry."""
    announce("gang nan", n, hex(bits))
    A = I.random_hermitian(np.random.default_rng(1), n, False)
    A.view(np.uint64)[n - 3, 1] = bits
    st, d, e, _ = hetrd(L, dev(A), False)
    assert st in (0, 6)
    assert torch.isnan(d).any()


def solve(plan, H, S, il=1, iu=None):
    eps = torch.empty(plan._vshape(), dtype=torch.float64, device="cuda")
    C = torch.zeros_like(H)
    plan.gevd(H, S, eps, C, il=il, iu=iu)
    plan.check()
    return eps, C


def pencil(n, cplx, batch, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.complex128 if cplx else torch.float64
    H, S = (torch.randn(batch, n, n, generator=g, dtype=dt, device="cuda") for _ in range(2))
    S = (S + S.mH) * (0.1 / n ** 0.5) + torch.eye(n, dtype=dt, device="cuda")
    return ((H + H.mH) / n ** 0.5).contiguous(), S.contiguous()


def check_pencil(H, S, eps, C, bar=1e-12):
    """Frobenius residual and orthonormality, the bars of the whole-solve tests."""
    n = H.shape[-1]
    R = H @ C - (S @ C) * eps[:, None, :]
    assert (torch.linalg.norm(R) / (torch.linalg.norm(H) * torch.linalg.norm(C))).item() < bar
    G = C.mH.contiguous() @ (S @ C)
    assert (G - torch.eye(C.shape[-1], dtype=C.dtype, device="cuda")).abs().max().item() < 10 * bar * max(1, n // 1000)


@pytest.mark.parametrize("cplx,n,batch", [(False, 300, 20), (False, 1100, 3), (True, 140, 40), (True, 520, 9),
                                          (True, 1100, 2), (True, 1100, 6)])
def test_batches(cplx, n, batch):
    """Batches whose gangs follow each other, and those that take other shapes."""
    announce("gang batch", cplx, n, batch)
    H, S = pencil(n, cplx, batch, 5)
    eps, C = solve(ks.Plan(n, batch=batch, complex=cplx), H, S)
    check_pencil(H, S, eps, C)


@pytest.mark.parametrize("cplx,n", [(False, 700), (False, 2100), (True, 1100)])
def test_mixed(cplx, n):
    """FP32 storage of the trailing matrix; the residual bar of the mixed form."""
    announce("gang mixed", cplx, n)
    H, S = pencil(n, cplx, 1, 7)
    m = n // 3
    plan = ks.Plan(n, complex=cplx, precision=ks.KS_MIXED)
    eps, C = solve(plan, H[0].contiguous(), S[0].contiguous(), il=1, iu=m)
    check_pencil(H, S, eps[None, :m], C[None, :, :m].contiguous(), bar=1e-11)


def test_streams_and_threads():
    """Whole-GPU gangs of several streams at once: each solve equals its own
    result when alone to rounding."""
    announce("gang streams")
    shapes = [(False, 1500), (True, 1200), (False, 1500), (True, 400)]
    work = []
    for i, (cplx, n) in enumerate(shapes):
        H, S = pencil(n, cplx, 1, 20 + i)
        H, S = H[0].contiguous(), S[0].contiguous()
        eps, _ = solve(ks.Plan(n, complex=cplx), H, S)
        work.append((cplx, n, H, S, eps))
    torch.cuda.synchronize()
    errors = []

    def run(cplx, n, H, S, ref):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                plan = ks.Plan(n, complex=cplx, stream=s)
                for _ in range(3):
                    eps, C = solve(plan, H, S)
                    assert (eps - ref).abs().max().item() < 1e-11
                check_pencil(H[None], S[None], eps[None], C[None])
                s.synchronize()
        except Exception as x:  # noqa: BLE001 - told to the main thread
            errors.append(repr(x))

    threads = [threading.Thread(target=run, args=w) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
