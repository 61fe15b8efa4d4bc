"""Finite rows far from the data in a large kernel product, and points far from
the launch's middle row: no row may overflow, and the rows that are not far are
what they are without them.

Bars, |Z - Z_ref| <= tol (|Gamma| |Y|) elementwise: 1e-5 as for every kernel
product.  On the strip the points of a row block lie up to 128 correlation
lengths (154 scaled units) from its middle, so a scaled FP32 coordinate is 2^-17
off and a pair's difference 2^-16; an exponent d^2 with d <= 5 (Gamma >= 2^-25)
is 2 d 2^-16 off and Gamma ln 2 times that: 1.1e-4."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import kernels
from workloads import normal_block, tensor_grid_points, uniform_points

pytestmark = pytest.mark.gpu

NAMES = {K.KA_GAUSSIAN: "gaussian", K.KA_EXP_L1: "exponential"}


def _product(kernel, ell, X, C, Y, precision=K.KA_FP32):
    d = dict(dtype=torch.float32, device="cuda")
    xr, xc, y = torch.tensor(X, **d), torch.tensor(C, **d), torch.tensor(Y, **d)
    z = torch.full((len(X), Y.shape[1]), float("nan"), **d)
    nb = K.ka_gamma_workspace(len(X), len(C), Y.shape[1], precision)
    # the split-FP16 route
    least = 1.3e9 if kernel == K.KA_EXP_L1 and Y.shape[1] == 16 else 4e8
    assert len(X) * len(C) * Y.shape[1] > least and nb >= len(C) * (4 * Y.shape[1] + 64)
    K.ka_gamma_apply(kernel, 1.0, ell, xr, xc, y, z, precision, torch.empty(nb // 4, **d))
    return z.cpu().numpy().astype(np.float64)


def _errors(kernel, ell, X, C, Y, Z):
    """|Z - Z_ref| over |Gamma| |Y|, rows whose bar is below FP32's range left out."""
    X, C, Y = (np.asarray(a, dtype=np.float32).astype(np.float64) for a in (X, C, Y))
    G = kernels.kernel_matrix(NAMES[kernel], X, C, ell, 1.0)
    ref, scale = G @ Y, np.abs(G) @ np.abs(Y)
    return np.where(scale > 1e-30, np.abs(Z - ref) / np.maximum(scale, 1e-30), 0.0)


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
@pytest.mark.parametrize("b", [16, 64])
def test_far_middle_row(kernel, b):
    # the row that the launch's coordinates are relative to
    nr, rows = (1500, 128) if b == 64 else (7000 if kernel == K.KA_EXP_L1 else 3000, 256)
    C, Y = tensor_grid_points((23, 23, 23)), normal_block(23, 23 ** 3, b, dtype=np.float32)
    others = np.arange(nr) // rows != (nr // 2) // rows      # rows of other blocks
    for f, ell in ((1e5, 0.1), (1e6, 0.5), (1e7, 0.5), (1e8, 0.5), (1e8, 5.0)):
        X = uniform_points(21, nr)
        X[nr // 2] = f
        Z = _product(kernel, ell, X, C, Y)
        assert np.isfinite(Z).all() and (Z[nr // 2] == 0).all()
        err = _errors(kernel, ell, X[others], C, Y, Z[others])
        assert err.max() < 1e-5, (f, ell, err.max())


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
@pytest.mark.parametrize("b", [16, 64])
def test_strip_far_from_the_middle_row(kernel, b):
    # points one correlation length apart, about 1e6 .. 4e6 of them from the middle row
    n = 9100 if b == 16 else 3000
    for far in (1e6, 4e6):
        X = np.zeros((n, 3))
        X[:, 0] = far + np.arange(n)
        X[n // 2] = 0.0
        Y = normal_block(24, n, b, dtype=np.float32)
        Z = _product(kernel, 1.0, X, X, Y)
        assert np.isfinite(Z).all()
        rows = 128 if b == 64 else 256
        others = np.arange(n) // rows != (n // 2) // rows
        err = _errors(kernel, 1.0, X[others], X, Y, Z[others])
        assert err.max() < 1.1e-4, (far, err.max())


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
@pytest.mark.parametrize("b", [16, 64])
def test_far_row_leaves_its_block(kernel, b):
    # one row of a block far off, in turn the launch's middle row and another
    nr, ell = 1500 if b == 64 else (7000 if kernel == K.KA_EXP_L1 else 3000), 0.5
    C, Y = tensor_grid_points((23, 23, 23)), normal_block(23, 23 ** 3, b, dtype=np.float32)
    for row in (3, nr // 2):
        for f in (1e2, 1e3, 1e5, 1e7, 1e30):
            X = uniform_points(21, nr)
            X[row] = f
            Z = _product(kernel, ell, X, C, Y)
            assert (Z[row] == 0).all()
            err = _errors(kernel, ell, X, C, Y, Z)
            assert err.max() < 1e-5, (row, f, err.max())
