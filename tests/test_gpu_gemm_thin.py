"""Products with few output tiles: a 32 x 32 tile per workgroup whose four wavefronts
share the inner dimension.  Edges of the tile and of a wavefront's share."""
import numpy as np
import pytest

from tests.gpu_helpers import announce, dev, host, stream_handle
from tests.test_gpu_stages import L, P  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (31, 33, 7), (32, 32, 8), (33, 31, 9), (64, 65, 31), (63, 64, 32), (95, 97, 33), (2, 200, 127),
          (200, 3, 128), (70, 70, 129), (40, 500, 257), (129, 66, 1000), (960, 1024, 5), (1000, 1100, 40)]


def op(X, o):
    return X if o == 0 else (X.T if o == 1 else X.conj().T)


@pytest.mark.parametrize("lower", [0, 1])
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("opa,opb", [(0, 0), (0, 1), (0, 2), (1, 0), (2, 0)])
def test_matches_numpy(L, cplx, opa, opb, lower):  # noqa: F811
    """Against numpy with strides beyond the rows: k terms of size up to max|A| max|B|
    (three products each for complex data), 1e-13 of their sum."""
    rng = np.random.default_rng(10 * opa + opb)
    for (m, n, k) in SHAPES:
        announce("thin gemm", cplx, opa, opb, lower, m, n, k)

        def rnd(*s):
            x = rng.normal(size=s)
            return (x + 1j * rng.normal(size=s)) if cplx else x
        A = rnd(m, k + 3) if opa == 0 else rnd(k, m + 3)
        B = rnd(k, n + 5) if opb == 0 else rnd(n, k + 5)
        C0 = rnd(m, n + 2)
        a = op(A[:, :k] if opa == 0 else A[:, :m], opa)
        b = op(B[:, :n] if opb == 0 else B[:, :k], opb)
        for beta in (0.0, 0.3):
            ref = C0.copy()
            ref[:, :n] = -0.7 * a @ b + beta * C0[:, :n]
            if lower:
                ref[:, :n] = np.where(np.tri(m, n, dtype=bool), ref[:, :n], C0[:, :n])
            Ad, Bd, Cd = dev(A), dev(B), dev(C0)
            assert L.ks_test_gemm(int(cplx), opa, opb, m, n, k, -0.7, P(Ad), A.shape[1], P(Bd), B.shape[1], beta,
                                  P(Cd), n + 2, lower, stream_handle()) == 0
            got = host(Cd)
            scale = np.abs(A).max() * np.abs(B).max() * k + 1
            assert np.abs(got - ref).max() < 1e-13 * scale, (m, n, k)
            assert np.array_equal(got[:, n:], C0[:, n:])
