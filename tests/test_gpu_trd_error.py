"""Eigenvalues of the standard problem (S = I) against references good to 1e-19: the
tridiagonalisation with the trailing matrix in registers and the divide and conquer
behind it are no further off than when every column was two launches and the
trailing matrix was updated 32 columns at a time."""
import numpy as np
import pytest
import torch

from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce, dev, host

pytestmark = pytest.mark.gpu

LD = np.longdouble


def overlap_like(n, seed):
    """Hermitian, decaying away from the diagonal, as the overlap whose small
    eigenvalues the Loewdin route needs."""
    r = np.random.default_rng(1000 + seed)
    i = np.arange(n)
    A = 0.4 * r.uniform(size=(n, n)) * np.exp(-np.abs(i[:, None] - i) / 9.0) * np.exp(2j * np.pi * r.uniform(size=(n, n)))
    A = np.tril(A, -1)
    return A + A.conj().T + 2.0 * np.eye(n)


def exact_product(A, X):
    """A X of real matrices: three slices of 19 bits each, whose products sum without
    rounding in 64 bits, added up in extended precision."""
    def slices(M):
        top, out = np.ceil(np.log2(np.abs(M).max())), []
        for q in range(1, 4):
            unit = 2.0 ** (top - 19 * q)
            out.append(np.rint(M / unit) * unit)
            M = M - out[-1]
        return out
    return sum((a @ x).astype(LD) for a in slices(A) for x in slices(X))


def rayleigh(A):
    """Rayleigh quotients of LAPACK's eigenvectors (error quadratic in theirs)."""
    X = np.linalg.eigh(A)[1]
    ar, ai, xr, xi = (np.ascontiguousarray(p) for p in (A.real, A.imag, X.real, X.imag))
    yr, yi = exact_product(ar, xr) - exact_product(ai, xi), exact_product(ar, xi) + exact_product(ai, xr)
    xr, xi = xr.astype(LD), xi.astype(LD)
    return np.sort((xr * yr + xi * yi).sum(0) / (xr * xr + xi * xi).sum(0))


@pytest.mark.parametrize("n,seeds,before", [(600, 4, 1.17), (1500, 2, 1.26)])
def test_eigenvalue_error(n, seeds, before):
    """before: root mean square error in units of 2^-53 of the largest eigenvalue
    with two launches per column."""
    announce("eigenvalue error", n)
    sq = []
    for seed in range(seeds):
        A = overlap_like(n, seed)
        H, S = dev(A), torch.eye(n, dtype=torch.complex128, device="cuda")
        eps, C = torch.empty(n, dtype=torch.float64, device="cuda"), torch.zeros_like(H)
        plan = ks.Plan(n, complex=True)
        plan.gevd(H, S, eps, C)
        plan.check("gevd")
        plan.close()
        ref = rayleigh(A)
        e = (host(eps).astype(LD) - ref).astype(np.float64) / float(np.abs(ref).max()) * 2.0 ** 53
        sq.append((e * e).mean())
    assert np.sqrt(np.mean(sq)) <= before
