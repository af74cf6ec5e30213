"""Fermi level far below the levels: electron counts so small that every state is a
tail of the distribution."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ne", [1e-12, 1e-17, 1e-19, 3e-21])
@pytest.mark.parametrize("n,batch", [(64, 1), (700, 2), (4097, 1), (1025, 64)])
def test_few_electrons(n, batch, ne):
    """The levels lie in [-1, 1] and mu up to 50 kT below them, so that every
    occupation is its tail: mu to the width of the last interval (1e-14) and the
    rounding of x / kT <= 60, occupations to these over kT, 1e-11 for both."""
    announce("fermi tail", n, batch, ne)
    rng = np.random.default_rng(n)
    kT = 0.02
    eps = np.sort(rng.uniform(-1, 1, size=(batch, n)), axis=1)
    plan = ks.Plan(n, batch=batch)
    sq, vec = ((batch, n, n), (batch, n)) if batch > 1 else ((n, n), (n,))
    one = lambda: torch.zeros(1, dtype=torch.float64, device="cuda")  # noqa: E731
    mu, eb, occ = one(), one(), torch.zeros(vec, dtype=torch.float64, device="cuda")
    C = torch.zeros(sq, dtype=torch.float64, device="cuda")
    plan.density(dev(eps.reshape(vec)), C, ne, kT, torch.empty_like(C), mu, eb, occ=occ)
    plan.check("density")
    plan.close()
    r = O.fermi(eps, ne, kT, 2.0)
    f = host(occ).reshape(batch, n)
    assert abs(float(host(mu)[0]) - r["mu"]) < 1e-11
    assert abs(f.sum() / r["occ"].sum() - 1.0) < 1e-11  # (the electrons asked for, unless the search ends 50 kT below the levels)
    big = r["occ"] > 1e-300
    assert np.abs(f[big] / r["occ"][big] - 1.0).max() < 1e-11
