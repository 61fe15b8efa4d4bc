"""Kernel products at the line between the FP32 and the split-FP16 route, which
lies higher for the exponential kernel at b = 16 and with few columns: sizes on
both sides of it, with block and group edges.

Bar: |Z - Z_ref| <= 1e-5 (|Gamma| |Y|) elementwise on either route."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import kernels
from workloads import normal_block, tensor_grid_points, uniform_points

pytestmark = pytest.mark.gpu

KNAME = {K.KA_GAUSSIAN: "gaussian", K.KA_EXP_L1: "exponential"}


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
@pytest.mark.parametrize("b,nr,nc", [(16, 5000, 16200), (16, 5000, 16300), (16, 257, 320001), (16, 62500, 1301),
                                     (32, 100000, 128), (32, 100000, 129), (64, 97000, 65)])
def test_both_sides(kernel, b, nr, nc):
    X = tensor_grid_points((10, 10, -(-nr // 100)))[:nr]
    C, Y = uniform_points(nc, nc), normal_block(b, nc, b, dtype=np.float32)
    d = dict(dtype=torch.float32, device="cuda")
    xr, xc, y = torch.tensor(X, **d), torch.tensor(C, **d), torch.tensor(Y, **d)
    z = torch.full((nr, b), float("nan"), **d)
    work = torch.full((K.ka_gamma_workspace(nr, nc, b, K.KA_FP32) // 4,), float("nan"), **d)
    K.ka_gamma_apply(kernel, 1.0, 0.4, xr, xc, y, z, K.KA_FP32, work)
    got, Yd = z.cpu().numpy().astype(np.float64), Y.astype(np.float64)
    Xd, Cd = xr.cpu().numpy().astype(np.float64), xc.cpu().numpy().astype(np.float64)
    step = max(1, int(2e7) // nc)
    for i in range(0, nr, step):
        G = kernels.kernel_matrix(KNAME[kernel], Xd[i:i + step], Cd, 0.4, 1.0)
        bar = 1e-5 * (np.abs(G) @ np.abs(Yd))
        assert (np.abs(got[i:i + step] - G @ Yd) <= bar).all()
