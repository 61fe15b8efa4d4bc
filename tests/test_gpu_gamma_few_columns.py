"""Large products with groups of 512 columns of which about 64, the number up to which
columns in FP32 are listed, are not zero: unit vectors on 64 neighbouring columns, and
63 to 65 columns in one group between full ones.

Bar: |Z - Z_ref| <= 1e-5 (|Gamma| |Y|) elementwise."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import kernels
from workloads import normal_block, uniform_points

pytestmark = pytest.mark.gpu

NAMES = {K.KA_GAUSSIAN: "gaussian", K.KA_EXP_L1: "exponential"}


def _check(kernel, nr, Y):
    nc, b = Y.shape
    d = dict(dtype=torch.float32, device="cuda")
    xr, xc = torch.tensor(uniform_points(61, nr), **d), torch.tensor(uniform_points(62, nc), **d)
    y, z = torch.tensor(Y, **d), torch.full((nr, b), float("nan"), **d)
    nb = K.ka_gamma_workspace(nr, nc, b, K.KA_FP32)
    assert nr * nc * b >= (1.3e9 if b == 16 else 4e8) and nb >= nc * (4 * b + 64)   # the split-FP16 route
    K.ka_gamma_apply(kernel, 1.0, 0.4, xr, xc, y, z, K.KA_FP32, torch.zeros(nb // 4, **d))
    rows = np.r_[0:200, nr // 2:nr // 2 + 200, nr - 200:nr]
    Z = z.cpu().numpy()[rows].astype(np.float64)
    G = kernels.kernel_matrix(NAMES[kernel], xr.cpu().numpy()[rows].astype(np.float64),
                              xc.cpu().numpy().astype(np.float64), 0.4, 1.0)
    Yd = Y.astype(np.float32).astype(np.float64)
    assert (np.abs(Z - G @ Yd) <= 1e-5 * (np.abs(G) @ np.abs(Yd))).all()


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
@pytest.mark.parametrize("b,nr", [(16, 21000), (32, 5000), (64, 2501)])
@pytest.mark.parametrize("count", [63, 64, 65])
def test_columns_in_a_group(kernel, b, nr, count):
    Y = normal_block(63, 4225, b)
    at = 1024 + np.random.default_rng(64).permutation(512)[count:]
    Y[at] = 0.0
    _check(kernel, nr, Y)


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
@pytest.mark.parametrize("tail", [63, 64, 65])
def test_columns_in_the_last_group(kernel, tail):
    Y = normal_block(65, 4096 + 140, 64)
    Y[4096 + tail:] = 0.0
    _check(kernel, 2501, Y)


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
@pytest.mark.parametrize("first", [0, 1100, 4161])
def test_unit_vectors(kernel, first):
    Y = np.zeros((4225, 64))
    Y[first:first + 64] = np.eye(64)
    _check(kernel, 2501, Y)
