"""Small kernel products, whose columns go in splits of 64 or a multiple of 128
where the scratch holds their partial sums: one row, column counts around one
and two tiles, ragged last splits, more splits than rows, each block width and
precision, with the scratch that ka_gamma_workspace states and with the least
that is accepted (which selects splits of 512 columns or none).

Bar: |Z - Z_ref| <= tol (|Gamma| |Y|) elementwise with the kernel products'
tolerances, 1e-5 in FP32 and 6e-5 for split BF16; more splits only shorten the
sums that the tolerances allow for."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import kernels
from workloads import normal_block, uniform_points

pytestmark = pytest.mark.gpu

KNAME = {K.KA_GAUSSIAN: "gaussian", K.KA_EXP_L1: "exponential"}


def _apply(kernel, xr, xc, y, precision, nbytes):
    z = torch.full((xr.shape[0], y.shape[1]), float("nan"), dtype=torch.float32, device="cuda")
    work = torch.full((max(nbytes // 4, 4),), float("nan"), dtype=torch.float32, device="cuda")[:nbytes // 4]
    K.ka_gamma_apply(kernel, 1.0, 0.5, xr, xc, y, z, precision, work if nbytes else None)
    torch.cuda.synchronize()
    return z.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
@pytest.mark.parametrize("precision,tol", [(K.KA_FP32, 1e-5), (K.KA_BF16X3, 6e-5)])
@pytest.mark.parametrize("b", [16, 32, 64])
@pytest.mark.parametrize("nr,nc", [(1, 65), (255, 64), (257, 63), (300, 129), (1, 9000), (1030, 1000), (2047, 1025),
                                   (3000, 700)])
def test_edges_of_fine_splits(kernel, precision, tol, b, nr, nc):
    X, C = uniform_points(nr, nr), uniform_points(nc, nc)
    Y = normal_block(b + nc, nc, b, dtype=np.float32)
    d = dict(dtype=torch.float32, device="cuda")
    xr, xc, y = torch.tensor(X, **d), torch.tensor(C, **d), torch.tensor(Y, **d)
    Xr, Xc = xr.cpu().numpy().astype(np.float64), xc.cpu().numpy().astype(np.float64)
    G = kernels.kernel_matrix(KNAME[kernel], Xr, Xc, 0.5, 1.0)
    Yd = Y.astype(np.float64)
    bar = tol * (np.abs(G) @ np.abs(Yd))
    stated = K.ka_gamma_workspace(nr, nc, b, precision)
    sizes = [stated]
    # the least that is accepted: partial sums of 512-column splits, then the split Y
    rows = 128 if b == 64 else 256
    ns = max(1, min(-(-2048 // -(-nr // rows)), nc // 512, 64))
    least = (-(-ns * nr * b * 4 // 256) * 256 if ns > 1 else 0)
    least += -(-nc // 64) * 64 * b * 4 if precision == K.KA_BF16X3 else 0
    if ns < 8 and least < stated:
        sizes.append(least)
    for nbytes in sizes:
        Z = _apply(kernel, xr, xc, y, precision, nbytes)
        assert np.isfinite(Z).all()
        assert (np.abs(Z - G @ Yd) <= bar).all(), (nbytes, (np.abs(Z - G @ Yd) / bar).max())
