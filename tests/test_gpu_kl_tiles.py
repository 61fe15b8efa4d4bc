"""K-L field sampling where the tiling of the field product and the mode
products in front of it end: single points and samples, one past a tile of 128
points or 64 samples, draws that are not a multiple of four, more columns than
one pass of the mode products takes, several sample tiles walked by one
workgroup with an incomplete last group, and rows longer than the grid.

All FP64 against the FP64 oracle.  A field value is a sum of M products of
values that the oracle forms the same way up to rounding: (M + 3 * 7) roundings
of 2^-53 on terms bounded by max|field| times a few, far inside the bar of
1e-12 of max|field| that the sampling tests use."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import collocation, galerkin, geometry, kl

pytestmark = pytest.mark.gpu


def _make(method):
    cls = {"collocation": collocation.Collocation, "galerkin": galerkin.GalerkinIBQ}[method]
    args = (2, (5, 4, 4), "exponential", 0.6)
    o = cls(geometry.make_domain("quarter_annulus"), *args)
    p = K.Problem(K.make_desc(block=16, method=method, domain="quarter_annulus", p=2, nel=(5, 4, 4),
                              kernel="exponential", ell=0.6))
    assert p.N == o.N
    return o, p


@pytest.mark.parametrize("method", ["galerkin", "collocation"])
@pytest.mark.parametrize("npts,S,M", [
    ((1, 1, 1), 1, 1),
    ((129, 1, 1), 65, 5),
    ((1, 1, 128), 64, 4),
    ((3, 43, 2), 66, 7),
    ((2, 3, 65), 3, 130),      # a second pass of the mode products
    ((40, 41, 39), 1090, 6),   # 500 point tiles x 18 sample tiles: 4 per workgroup, 2 in the last group
])
def test_field_tiles_match_oracle(method, npts, S, M):
    o, prob = _make(method)
    rng = np.random.default_rng(17)
    V = rng.standard_normal((o.N, M))
    lam = rng.random(M) + 0.1
    grid = [np.sort(rng.random(n)) for n in npts]
    xi = rng.standard_normal((M, S))
    P = int(np.prod(npts))
    pad = 5
    F = torch.full((S + 1, P + pad), 7.0, dtype=torch.float64, device="cuda")
    K.ka_kl_sample(prob.h, lam, torch.tensor(V.T.copy(), device="cuda"), grid, torch.tensor(xi.T.copy(), device="cuda"),
                   F[:S], mu=0.5)
    torch.cuda.synchronize()
    prob.close()
    got = F.cpu().numpy()
    ref = kl.sample(o, lam, V, grid, xi, mu=0.5).T
    assert np.abs(got[:S, :P] - ref).max() < 1e-12 * np.abs(ref).max()
    assert (got[:S, P:] == 7.0).all() and (got[S] == 7.0).all()


def test_zero_norm_leaves_the_field():
    o, prob = _make("galerkin")
    V = torch.ones((3, prob.N), dtype=torch.float64, device="cuda")
    V[1] = 0
    F = torch.full((70, 8), 7.0, dtype=torch.float64, device="cuda")
    xi = torch.ones((70, 3), dtype=torch.float64, device="cuda")
    with pytest.raises(K.KAError) as e:
        K.ka_kl_sample(prob.h, np.ones(3), V, [np.array([0.2, 0.7])] * 3, xi, F)
    prob.close()
    assert e.value.code == K.KA_ERR_SINGULAR
    assert (F == 7.0).all()
