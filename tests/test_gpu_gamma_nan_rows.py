"""Large products of scattered points, most rows far from all columns, with values in
the block that are not finite: the vectors without them are as close as ever.

Bar: |Z - Z_ref| <= 1e-5 (|Gamma| |Y|) elementwise in these vectors; where |Gamma| |Y|
is below 1e-30 (FP32's underflow is near) results only have to be small."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import kernels
from workloads import normal_block, uniform_points

pytestmark = pytest.mark.gpu

NAMES = {K.KA_GAUSSIAN: "gaussian", K.KA_EXP_L1: "exponential"}


@pytest.mark.parametrize("kernel,ell", [(K.KA_GAUSSIAN, 0.05), (K.KA_EXP_L1, 0.02)])
@pytest.mark.parametrize("b,nr,nc", [(16, 60000, 1600), (32, 15000, 905), (64, 9421, 905), (64, 4000, 2500)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_other_vectors(kernel, ell, b, nr, nc, value):
    C = np.array(sorted(uniform_points(82, nc).tolist(), key=lambda p: p[2]))
    Y = normal_block(83, nc, b)
    Y[nc // 3, 5] = Y[nc - 7, 9] = value
    d = dict(dtype=torch.float32, device="cuda")
    xr, xc, y = torch.tensor(uniform_points(81, nr), **d), torch.tensor(C, **d), torch.tensor(Y, **d)
    z = torch.full((nr, b), float("nan"), **d)
    nb = K.ka_gamma_workspace(nr, nc, b, K.KA_FP32)
    assert nb >= nc * (4 * b + 64)   # the split-FP16 route
    K.ka_gamma_apply(kernel, 1.0, ell, xr, xc, y, z, K.KA_FP32, torch.zeros(nb // 4, **d))
    rows = np.r_[0:1000, nr - 1000:nr]
    Z = z.cpu().numpy()[rows].astype(np.float64)
    G = kernels.kernel_matrix(NAMES[kernel], xr.cpu().numpy()[rows].astype(np.float64),
                              xc.cpu().numpy().astype(np.float64), ell, 1.0)
    keep = np.isfinite(Y).all(0)
    assert not np.isfinite(Z[:, ~keep]).any() or value == np.inf
    Yd, Z = Y.astype(np.float32).astype(np.float64)[:, keep], Z[:, keep]
    ref, scale = G @ Yd, G @ np.abs(Yd)
    ok = scale > 1e-30
    assert np.isfinite(Z).all() and (np.abs(Z[~ok]) < 1e-29).all()
    assert (np.abs(Z - ref)[ok] <= 1e-5 * scale[ok]).all()
