"""Large products at KA_BF16X3: the Gaussian kernel takes the split-FP16 route
where the scratch holds its operands, the exponential kernel and less scratch
split BF16.  Bars as for the kernel products: |Z - Z_ref| <= tol (|Gamma| |Y|)
elementwise, 1e-5 for split FP16 and 6e-5 for split BF16."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import kernels
from workloads import normal_block, tensor_grid_points, uniform_points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,name", [(K.KA_GAUSSIAN, "gaussian"), (K.KA_EXP_L1, "exponential")])
@pytest.mark.parametrize("b,nr,nc", [(16, 1320, 20000), (32, 257, 50000), (64, 6200, 1025)])
def test_routes(kernel, name, b, nr, nc):
    X = tensor_grid_points((10, 10, -(-nr // 100)))[:nr]
    C, Y = uniform_points(nc, nc), normal_block(b, nc, b, dtype=np.float32)
    d = dict(dtype=torch.float32, device="cuda")
    xr, xc, y = torch.tensor(X, **d), torch.tensor(C, **d), torch.tensor(Y, **d)
    stated = K.ka_gamma_workspace(nr, nc, b, K.KA_BF16X3)
    G = kernels.kernel_matrix(name, xr.cpu().numpy().astype(np.float64), xc.cpu().numpy().astype(np.float64), 0.4, 1.0)
    ref, scale = G @ Y.astype(np.float64), np.abs(G) @ np.abs(Y).astype(np.float64)
    # without the split-FP16 operands (Y and the points), but with split BF16's
    for nbytes, tol in ((stated, 1e-5 if kernel == K.KA_GAUSSIAN else 6e-5), (stated - nc * (4 * b + 60), 6e-5)):
        z = torch.full((nr, b), float("nan"), **d)
        work = torch.full((nbytes // 4,), float("nan"), **d)
        K.ka_gamma_apply(kernel, 1.0, 0.4, xr, xc, y, z, K.KA_BF16X3, work)
        err = np.abs(z.cpu().numpy().astype(np.float64) - ref) / scale
        assert np.isfinite(err).all() and err.max() < tol, (nbytes, err.max())
