"""KS_PLAN_GRAPH for batches whose tridiagonalisation runs as two groups: the captured
sequence is a chain, and its replays equal eager solves."""
import ctypes

import pytest
import torch

from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce
from tests.test_gpu_gang import pencil, solve

pytestmark = pytest.mark.gpu


def replays(cplx, n, batch, il, iu, reps):
    """Every replay, with new contents in the same buffers and eager work in between,
    has the bits of an eager plan; returns the forks of the captured sequence."""
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        gplan = ks.Plan(n, batch=batch, complex=cplx, stream=stream, flags=ks.KS_PLAN_GRAPH)
        eplan = ks.Plan(n, batch=batch, complex=cplx, stream=stream)
        H, S = pencil(n, cplx, batch, 0)
        eps, C = torch.empty(batch, n, dtype=torch.float64, device="cuda"), torch.zeros_like(H)
        for rep in range(reps):
            H2, S2 = pencil(n, cplx, batch, 100 + rep)
            H.copy_(H2)
            S.copy_(S2)
            gplan.gevd(H, S, eps, C, il=il, iu=iu)
            _ = (H.abs() * 2.0).sum().item()
            gplan.check("replay")
            want = solve(eplan, H, S, il=il, iu=iu)
            assert torch.equal(eps, want[0]) and torch.equal(C, want[1]), rep
        stream.synchronize()
        assert gplan.graph_stats() == (1, reps - 1)
        forks = ctypes.c_int32(-1)
        fn = ks.lib().ks_test_graph_forks
        fn.argtypes, fn.restype = [ctypes.c_void_p, ctypes.c_void_p], ctypes.c_int32
        assert fn(gplan._h, ctypes.byref(forks)) == 0
    return forks.value


@pytest.mark.parametrize("cplx,n,batch", [(False, 1100, 5), (True, 1100, 6)])
def test_two_groups_are_one_chain(cplx, n, batch):
    announce("graph chain", cplx, n, batch)
    assert replays(cplx, n, batch, 1, n // 4, 4) == 0


@pytest.mark.skip(reason="thousands of replays of a small k-point batch on several streams once ended the process (host "
                         "side, with a forked sequence); the cause was not found, so this case stays off")
def test_small_kpoint_batch():
    announce("graph small batch")
    assert replays(True, 208, 8, 1, 60, 4) == 0
