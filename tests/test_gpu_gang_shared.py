"""Tridiagonalisations that do not have the GPU to themselves: the forms in memory of
the whole-GPU gangs and panels form the same sums, so the bits do not depend on
what runs beside a solve."""
import threading

import pytest
import torch

from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce, stream_handle
from tests.test_gpu_gang import L, P, check_pencil, pencil, solve  # noqa: F401 - L is a fixture

pytestmark = pytest.mark.gpu


def reduce(lib, A0, cplx):
    """d, e of T and Q applied to sixteen columns."""
    n, m = A0.shape[0], 16
    A, X = A0.clone(), torch.eye(n, dtype=torch.float64, device="cuda")
    d, e = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
    Y = torch.zeros(n, m, dtype=A0.dtype, device="cuda")
    assert lib.ks_test_hetrd(int(cplx), n, P(A), P(d), P(e), P(X), m, P(Y), stream_handle()) == 0
    torch.cuda.synchronize()
    return d, e[:n - 1], Y


@pytest.mark.parametrize("cplx,n", [(False, n) for n in (1025, 2048, 2500, 3072, 3105, 3400, 4300, 5700, 7100, 8300)] +
                         [(True, n) for n in (1025, 1536, 1700, 2048, 2081, 2800, 4200, 5600, 7100, 8300)])
def test_forms_in_memory_give_the_same_bits(L, cplx, n):  # noqa: F811
    """On half the GPU (level 1) and a quarter (level 3), at every shape of the gangs
    and every row length of the panels."""
    announce("forms in memory", cplx, n)
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn(n, n, generator=g, dtype=torch.complex128 if cplx else torch.float64, device="cuda")
    A = ((A + A.mH) / n ** 0.5).contiguous()
    want = reduce(L, A, cplx)
    for level in (1, 3):
        assert L.ks_test_set_gang_leave(level) == 0
        got = reduce(L, A, cplx)
        assert all(torch.equal(a, b) for a, b in zip(want, got))


@pytest.mark.parametrize("cplx,n", [(False, 2300), (False, 3400), (True, 1300), (True, 2300)])
def test_beside_one_busy_workgroup(cplx, n):
    """A kernel of one workgroup on another stream keeps a compute unit for 0.3 s."""
    announce("busy workgroup", cplx, n)
    H, S = pencil(n, cplx, 1, 11)
    H, S = H[0].contiguous(), S[0].contiguous()
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(main):
        plan = ks.Plan(n, complex=cplx, stream=main)
        eps, C = solve(plan, H, S)
        with torch.cuda.stream(side):
            torch.cuda._sleep(700_000_000)
        for _ in range(2):
            again = solve(plan, H, S)
            assert torch.equal(again[0], eps) and torch.equal(again[1], C)
    torch.cuda.synchronize()
    check_pencil(H[None], S[None], eps[None], C[None])


def test_beside_each_other():
    """Solves of panels and whole-GPU gangs on three streams: each gives the bits that
    it gives alone."""
    announce("beside each other")
    work = []
    for i, (cplx, n) in enumerate([(False, 3400), (True, 2300), (False, 2100)]):
        H, S = pencil(n, cplx, 1, 30 + i)
        H, S = H[0].contiguous(), S[0].contiguous()
        work.append((cplx, n, H, S) + solve(ks.Plan(n, complex=cplx), H, S))
    torch.cuda.synchronize()
    errors = []

    def run(cplx, n, H, S, eps, C):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                plan = ks.Plan(n, complex=cplx, stream=s)
                for _ in range(4):
                    again = solve(plan, H, S)
                    assert torch.equal(again[0], eps) and torch.equal(again[1], C)
                s.synchronize()
        except Exception as x:  # noqa: BLE001 - told to the main thread
            errors.append(repr(x))

    threads = [threading.Thread(target=run, args=w) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
