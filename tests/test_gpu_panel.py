"""Panels of the tridiagonalisation in one launch (one matrix beyond the orders whose
trailing matrix fits the registers): orders at the edges of its block sizes, the
forms behind a panel whose workgroups could not gather, the mixed form, streams."""
import threading

import numpy as np
import pytest
import torch

from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce
from tests.test_gpu_gang import L, check_pencil, hetrd, pencil, solve  # noqa: F401

pytestmark = pytest.mark.gpu


def random_hermitian(n, cplx):
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn(n, n, generator=g, dtype=torch.complex128 if cplx else torch.float64, device="cuda")
    return (A + A.mH) / 2


def check_similarity(L, n, cplx):  # noqa: F811
    """Q unitary to 1e-12 and Q T Q^H = A to 1e-12 max|A| n, the bars of the other orders."""
    A0 = random_hermitian(n, cplx)
    st, d, e, Q = hetrd(L, A0, cplx)
    assert st == 0
    QT = Q * d
    QT[:, :-1] += Q[:, 1:] * e
    QT[:, 1:] += Q[:, :-1] * e
    Qh = Q.mH.contiguous()
    assert (Qh @ Q - torch.eye(n, dtype=A0.dtype, device="cuda")).abs().max().item() < 1e-12
    assert (QT @ Qh - A0).abs().max().item() < 1e-12 * max(1.0, A0.abs().max().item()) * n


@pytest.mark.parametrize("cplx,n", [(False, n) for n in (3073, 3104, 3137, 4114, 4115, 5566, 5567, 7019, 8229)] +
                         [(True, n) for n in (2049, 2080, 2113, 2662, 2663, 4114, 4115, 5567, 7019)])
def test_edges_of_the_blocks(L, cplx, n):  # noqa: F811
    announce("panel", cplx, n)
    check_similarity(L, n, cplx)


@pytest.mark.parametrize("cplx,n", [(False, 11132), (False, 11133), (True, 8229)])
def test_largest_orders(L, cplx, n):  # noqa: F811
    """The largest blocks, and an order whose first panel is beyond them."""
    announce("panel", cplx, n)
    check_similarity(L, n, cplx)


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("level", [1, 2])
def test_panels_that_leave(L, cplx, level):  # noqa: F811
    """The small form (level 1) and the single workgroup (level 2) do a panel's columns."""
    n = 2100 if cplx else 3100
    announce("panel leaves", cplx, level)
    assert L.ks_test_set_gang_leave(level) == 0
    check_similarity(L, n, cplx)


def test_small_form_of_larger_blocks(L):  # noqa: F811
    announce("panel leaves", 5600)
    assert L.ks_test_set_gang_leave(1) == 0
    check_similarity(L, 5600, False)


@pytest.mark.parametrize("bits", [0x7FF8000000000000, 0x7FF4A5A5DEADBEEF])
def test_nan_ends(L, bits):  # noqa: F811
    announce("panel nan", hex(bits))
    n = 3200
    A = random_hermitian(n, False).cpu().numpy()
    A.view(np.uint64)[n - 3, 1] = bits
    st, d, _, _ = hetrd(L, torch.from_numpy(A).cuda(), False)
    assert st in (0, 6)
    assert torch.isnan(d).any()


@pytest.mark.parametrize("cplx,n", [(False, 3300), (False, 4500), (False, 6000), (True, 2300), (True, 3000), (True, 4200),
                                    (True, 5600)])
def test_mixed(cplx, n):
    """FP32 storage of the trailing matrix; the residual bar of the mixed form."""
    announce("panel mixed", cplx, n)
    H, S = pencil(n, cplx, 1, 7)
    m = n // 8
    plan = ks.Plan(n, complex=cplx, precision=ks.KS_MIXED)
    eps, C = solve(plan, H[0].contiguous(), S[0].contiguous(), il=1, iu=m)
    plan.close()
    check_pencil(H, S, eps[None, :m], C[None, :, :m].contiguous(), bar=1e-11)


def test_streams_and_threads():
    """Panels of several streams at once, of which one has the chip: each solve equals
    its own result when alone to rounding."""
    announce("panel streams")
    work = []
    for i, (cplx, n) in enumerate([(False, 3200), (True, 2200), (False, 3400)]):
        H, S = pencil(n, cplx, 1, 40 + i)
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
                for _ in range(2):
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
