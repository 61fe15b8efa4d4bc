"""K-L field sampling with a mean much larger than the fluctuations."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import galerkin, geometry, kl

pytestmark = pytest.mark.gpu


def test_large_mean_is_added_once():
    # mu + fluctuation is one rounding: with the FP64 oracle's own at most one
    # unit in the last place of mu between the two (the fluctuations, of size
    # 10, differ by less than 1e-3 of that unit)
    args = (2, (5, 4, 4), "exponential", 0.6)
    o = galerkin.GalerkinIBQ(geometry.make_domain("quarter_annulus"), *args)
    p = K.Problem(K.make_desc(block=16, method="galerkin", domain="quarter_annulus", p=2, nel=(5, 4, 4),
                              kernel="exponential", ell=0.6))
    rng = np.random.default_rng(51)
    M, S, mu = 100, 70, 1.0e6
    V, xi, lam = rng.standard_normal((o.N, M)), rng.standard_normal((M, S)), rng.random(M) + 0.1
    grid = [np.sort(rng.random(n)) for n in (11, 7, 9)]
    F = torch.empty((S, 11 * 7 * 9), dtype=torch.float64, device="cuda")
    K.ka_kl_sample(p.h, lam, torch.tensor(V.T.copy(), device="cuda"), grid, torch.tensor(xi.T.copy(), device="cuda"), F,
                   mu=mu)
    p.close()
    ref = kl.sample(o, lam, V, grid, xi, mu=mu).T
    assert np.abs(F.cpu().numpy() - ref).max() <= np.spacing(mu)
