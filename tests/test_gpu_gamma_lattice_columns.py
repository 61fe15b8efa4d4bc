"""Large Gaussian products on the lattice's whole range, many columns: each column's
operands (the parts of its coordinates and of their products) are formed once, and a
last place lost in one of them shows in the rows next to that column only.

Bar: |Z - Z_ref| <= 1e-5 (|Gamma| |Y|) elementwise; rows are the columns themselves, so
that each result is mostly its own column's."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from workloads import normal_block, uniform_points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,n", [(16, 20000), (32, 20000), (64, 20000)])
@pytest.mark.parametrize("ell", [0.04, 0.047, 0.06])
def test_every_column(b, n, ell):
    d = dict(dtype=torch.float32, device="cuda")
    x = torch.tensor(uniform_points(71, n) - 0.5, **d)
    x[n // 2] = 0.0   # the launch's centre: all points within 16 units each way
    y, z = torch.tensor(normal_block(72, n, b), **d), torch.full((n, b), float("nan"), **d)
    nb = K.ka_gamma_workspace(n, n, b, K.KA_FP32)
    assert nb >= n * (4 * b + 64)   # the split-FP16 route
    K.ka_gamma_apply(K.KA_GAUSSIAN, 1.0, ell, x, x, y, z, K.KA_FP32, torch.zeros(nb // 4, **d))
    xd, yd, worst = x.double().cpu().numpy(), y.double().cpu().numpy(), 0.0
    Z = z.double().cpu().numpy()
    for i in range(0, n, 500):
        # exponents in FP64 from differences of the FP32 points
        e = sum((xd[i:i + 500, None, k] - xd[None, :, k]) ** 2 for k in range(3))
        G = np.exp(-e / ell ** 2)
        worst = max(worst, (np.abs(Z[i:i + 500] - G @ yd) / (G @ np.abs(yd))).max())
    assert worst <= 1e-5, worst
