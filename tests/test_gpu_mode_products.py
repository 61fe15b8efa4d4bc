"""Kronecker mode products at the edges of their tiling: modes of 3, 15, 16, 17
(one row tile and one past it), 80 and 81 (one pass over the input and two),
140 (the matrix in several chunks), in each direction, with full and partial
blocks of vectors, through the solves (column-major throughout) and both ends
of the block application (column-major to point-major and back).

Bars as in the operator tests: the solves are FP64, 1e-12 of max|ref| (modes of
140: 3 x 140 roundings of 2^-53 against mass matrices of condition below 1e3);
the operators hold FP32 chains, 2e-5 of a column's max|ref|."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import collocation, galerkin, geometry
from workloads import normal_block

pytestmark = pytest.mark.gpu

MESHES = [(1, 1, 1), (13, 14, 15), (15, 3, 2), (78, 1, 2), (1, 79, 1), (138, 1, 1), (1, 138, 1), (1, 1, 138)]


def _pair(method, nel, block):
    cls = {"galerkin": galerkin.GalerkinIBQ, "collocation": collocation.Collocation}[method]
    o = cls(geometry.make_domain("cube"), 2, nel, "exponential", 1.0)
    p = K.Problem(K.make_desc(block=block, method=method, domain="cube", p=2, nel=nel, kernel="exponential", ell=1.0))
    assert p.N == o.N
    return o, p


@pytest.mark.parametrize("nvec,block", [(1, 16), (33, 32), (64, 64)])
@pytest.mark.parametrize("nel", MESHES, ids=str)
def test_solves(nel, nvec, block):
    o, prob = _pair("galerkin", nel, block)
    X = normal_block(5, o.N, nvec)
    for op, ref in ((K.KA_ZINV, o.solve_Z(X)), (K.KA_LINV, o._Lsolve(X, trans=0)), (K.KA_LTINV, o._Lsolve(X, trans=1))):
        Xd = torch.full((nvec + 1, o.N), 7.0, dtype=torch.float64, device="cuda")
        Xd[:nvec] = torch.tensor(X.T.copy(), device="cuda")
        K.ka_solve_Z(prob.h, op, Xd[:nvec])
        torch.cuda.synchronize()
        got = Xd.cpu().numpy()
        assert np.abs(got[:nvec].T - ref).max() < 1e-12 * np.abs(ref).max(), op
        assert (got[nvec] == 7.0).all()
    prob.close()


@pytest.mark.parametrize("method", ["galerkin", "collocation"])
@pytest.mark.parametrize("nel", [m for m in MESHES if m != (13, 14, 15)], ids=str)
def test_operators(nel, method):
    o, prob = _pair(method, nel, 16)
    X = normal_block(6, o.N, 19)
    for form, ref in ((K.KA_APRIME, o.apply_Aprime(X)), (K.KA_A, o.apply_A(X))):
        Xd = torch.tensor(X.T.copy(), device="cuda")
        Yd = torch.full((20, o.N), 7.0, dtype=torch.float64, device="cuda")
        K.ka_apply_A(prob.h, form, Xd, Yd[:19])
        torch.cuda.synchronize()
        got = Yd.cpu().numpy()
        assert (np.abs(got[:19].T - ref).max(axis=0) / np.abs(ref).max(axis=0)).max() < 2e-5, form
        assert (got[19] == 7.0).all()
    prob.close()


def test_non_finite_values_stay_in_their_vector():
    o, prob = _pair("galerkin", (15, 15, 1), 16)
    X = normal_block(7, o.N, 3)
    Xd = torch.tensor(X.T.copy(), device="cuda")
    Xd[1, o.N - 1] = float("inf")
    K.ka_solve_Z(prob.h, K.KA_LTINV, Xd)
    got = Xd.cpu().numpy().T
    prob.close()
    ref = o._Lsolve(X, trans=1)
    assert not np.isfinite(got[:, 1]).all()
    for j in (0, 2):
        assert np.abs(got[:, j] - ref[:, j]).max() < 1e-12 * np.abs(ref).max()
