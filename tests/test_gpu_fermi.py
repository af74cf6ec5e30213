"""Fermi level: orders and batches at the edges of the chunks of 64 eigenvalues, of
the number of chunks that every wavefront holds and of the number that the
workgroup holds."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2606_09058_amd import ks
from tests.gpu_helpers import announce, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kT", [1e-4, 0.02, 0.5])
@pytest.mark.parametrize("n,batch", [(1, 1), (2, 3), (63, 2), (64, 1), (65, 5), (64, 12), (65, 6), (64, 13), (64, 32), (128, 32), (129, 32), (4096, 1),
                                     (4097, 1), (1024, 63), (1024, 64)])
def test_levels(n, batch, kT):
    """The electron count to 1e-12 and the width of the last bisection interval
    (1e-14 over kT per state); where the levels are no more than 20 kT apart, mu to 1e-11
    and occupations and band energy to 1e-9 of the oracle's."""
    announce("fermi", n, batch, kT)
    rng = np.random.default_rng(n + batch)
    eps = np.sort(np.linspace(-1, 1, n) + rng.uniform(-0.4, 0.4, size=(batch, n)) / max(n, 2), axis=1)
    wk = rng.uniform(0.2, 1.0, size=batch)
    wk /= wk.sum()
    ne = 2.0 * (int(0.37 * n) + 0.4)
    plan = ks.Plan(n, batch=batch)
    sq = (batch, n, n) if batch > 1 else (n, n)
    vec = (batch, n) if batch > 1 else (n,)
    one = lambda: torch.zeros(1, dtype=torch.float64, device="cuda")  # noqa: E731
    mu, eb, occ = one(), one(), torch.zeros(vec, dtype=torch.float64, device="cuda")
    C = torch.zeros(sq, dtype=torch.float64, device="cuda")
    plan.density(dev(eps.reshape(vec)), C, ne, kT, torch.empty_like(C), mu, eb, occ=occ, kweights=wk)
    plan.check("density")
    plan.close()
    f, mu, eb = host(occ).reshape(batch, n), float(host(mu)[0]), float(host(eb)[0])
    assert abs(wk @ f.sum(axis=1) - ne) < 1e-12 * ne + 2.0 * n * 1e-14 / kT
    if 2.0 / max(n - 1, 1) <= 20 * kT:
        r = O.fermi(eps, ne, kT, 2.0, wk=wk)
        assert abs(mu - r["mu"]) < 1e-11
        assert np.abs(f - r["occ"]).max() < 1e-9
        assert abs(eb - r["eband"]) < 1e-9 * max(1.0, abs(r["eband"]))
