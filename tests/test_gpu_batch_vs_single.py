"""Batches whose kernels take other branches than a single matrix's (thin products,
shapes of the gangs, panels): equal to rounding, not bit for bit."""
import pytest
import torch

from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce
from tests.test_gpu_gang import check_pencil, pencil, solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cplx,n,batch", [(True, 520, 9), (False, 700, 6), (False, 1300, 3), (True, 1100, 5), (False, 3200, 2)])
def test_batch_equals_single_solves_to_rounding(cplx, n, batch):
    """Both are backward stable to a few hundred units of rounding of a pencil of
    norm 2 with S near the identity: eigenvalues within 1e-12."""
    announce("batch vs single", cplx, n, batch)
    H, S = pencil(n, cplx, batch, 9)
    eps, C = solve(ks.Plan(n, batch=batch, complex=cplx), H, S)
    check_pencil(H, S, eps, C)
    one = ks.Plan(n, complex=cplx)
    for b in range(batch):
        e1, _ = solve(one, H[b].contiguous(), S[b].contiguous())
        assert (eps[b] - e1).abs().max().item() < 1e-12
    torch.cuda.synchronize()
