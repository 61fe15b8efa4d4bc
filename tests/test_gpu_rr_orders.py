"""Rayleigh-Ritz steps of rising order: the small dense stages (pivoted and
plain Cholesky, back-transformation with 8, 16, 32 or 64 elements per lane) at
orders on either side of 128, 256 and 512, with blocks of each width.

Bars as in the eigenvalue tests: floored relative error 1e-6 against the exact
product-of-1D spectra, Z-orthonormal eigenvectors to 1e-6; collocation pairs by
their residual, 1e-4 of the largest eigenvalue (FP32 operator: an absolute error
of a few 1e-7 lambda_1 per pair and the solver's own 1e-6)."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import collocation, errors, galerkin, product1d

pytestmark = pytest.mark.gpu


def _solve(method, nel, M, block):
    prob = K.Problem(K.make_desc(method, "cube", 2, nel, "exponential", 1.0, block=block, seed=3))
    V = torch.zeros((M, prob.N), dtype=torch.float64, device="cuda")
    rc, lam, _ = K.ka_eigs(prob.h, M, tol=1e-6, maxit=60, V=V)
    prob.close()
    assert rc == 0
    return lam, V.cpu().numpy().T


@pytest.mark.parametrize("M,block", [(3, 16), (90, 16), (110, 32), (230, 64), (400, 64)])
def test_galerkin_orders(M, block):
    nel = (8, 8, 8)
    lam, V = _solve("galerkin", nel, M, block)
    ref = product1d.galerkin_box_spectrum(2, nel, "exponential", 1.0, M=M)
    assert errors.floored_rel_errors(ref, lam).max() < 1e-6
    Z = galerkin.GalerkinIBQ("cube", 2, nel, "exponential", 1.0).Z_dense()
    assert np.abs(V.T @ Z @ V - np.eye(M)).max() < 1e-6


@pytest.mark.parametrize("M,block", [(3, 16), (90, 16), (110, 32), (230, 64)])
def test_collocation_orders(M, block):
    nel = (7, 8, 7)
    lam, V = _solve("collocation", nel, M, block)
    o = collocation.Collocation("cube", 2, nel, "exponential", 1.0)
    re, im = lam[0::2], lam[1::2]
    R = o.apply_Aprime(V)
    # a complex pair's columns are its real and imaginary parts
    W = V * re
    i = 0
    while i < M:
        if im[i] != 0.0 and i + 1 < M:
            a, b = V[:, i].copy(), V[:, i + 1].copy()
            W[:, i], W[:, i + 1] = re[i] * a - im[i] * b, im[i] * a + re[i] * b
            i += 2
        else:
            i += 1
    res = np.linalg.norm(R - W, axis=0) / np.linalg.norm(V, axis=0)
    if im[M - 1] != 0.0 and (M < 2 or im[M - 2] != -im[M - 1]):
        res = res[:-1]                       # half of a pair
    assert res.max() < 1e-4 * re[0]
