"""Batches of two to four matrices whose gangs take the whole GPU: one matrix after
the other, so that repeated solves give the same bits."""
import pytest
import torch

from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce
from tests.test_gpu_gang import check_pencil, pencil, solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cplx,n,batch", [(False, 1100, 4), (False, 2100, 2), (False, 2600, 3), (True, 1600, 3),
                                          (True, 1800, 2)])
def test_repeated_solves_agree_bitwise(cplx, n, batch):
    announce("gang batch repeated", cplx, n, batch)
    H, S = pencil(n, cplx, batch, 3)
    plan = ks.Plan(n, batch=batch, complex=cplx)
    eps, C = solve(plan, H, S)
    check_pencil(H, S, eps, C)
    for _ in range(4):
        again = solve(plan, H, S)
        assert torch.equal(again[0], eps) and torch.equal(again[1], C)
