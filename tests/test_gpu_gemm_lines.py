"""Products on both sides of the lines between the thin kernel and the 64 x 64 tiles:
the inner dimension from which the number of tiles decides, and that number for full
and lower products."""
import numpy as np
import pytest

from tests.gpu_helpers import announce, dev, host, stream_handle
from tests.test_gpu_gemm_thin import op
from tests.test_gpu_stages import L, P  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lower,m", [(0, 704), (0, 705), (0, 736), (0, 800), (0, 832), (1, 832), (1, 863), (1, 928), (1, 960), (1, 993)])
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("opa,opb", [(0, 0), (0, 2), (2, 0)])
def test_lines(L, cplx, opa, opb, lower, m):  # noqa: F811
    """k terms of size up to max|A| max|B|: 1e-13 of their sum, as for the small shapes."""
    announce("gemm line", cplx, opa, opb, lower, m)
    rng = np.random.default_rng(m)
    for k in (256, 257, 300):
        def rnd(*s):
            x = rng.normal(size=s)
            return (x + 1j * rng.normal(size=s)) if cplx else x
        A, B = (rnd(m, k) if opa == 0 else rnd(k, m)), (rnd(k, m) if opb == 0 else rnd(m, k))
        C = dev(np.zeros((m, m), A.dtype))
        Ad, Bd = dev(A), dev(B)
        assert L.ks_test_gemm(int(cplx), opa, opb, m, m, k, 1.0, P(Ad), A.shape[1], P(Bd), B.shape[1], 0.0, P(C), m, lower,
                              stream_handle()) == 0
        ref = op(A, opa) @ op(B, opb)
        ref = np.tril(ref) if lower else ref
        assert np.abs(host(C) - ref).max() < 1e-13 * (np.abs(A).max() * np.abs(B).max() * k + 1), k
