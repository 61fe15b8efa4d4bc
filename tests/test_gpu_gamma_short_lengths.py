"""Large products whose columns are split and whose correlation length is short:
most partial sums are of columns far from the row and far below what their boxes
could give.

Bars: |Z - Z_ref| <= 1e-5 (|Gamma| |Y|) elementwise, also where the near columns are
zero or tiny, so that far ones decide (results below 1e-30 (max |Y| is about 4) but
for their being small: FP32 underflow).  Time: at most half as much again as with a
long correlation length, where no such sums are; work on them done twice takes more."""
import statistics

import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import kernels
from workloads import normal_block, tensor_grid_points, uniform_points

pytestmark = pytest.mark.gpu

NAMES = {K.KA_GAUSSIAN: "gaussian", K.KA_EXP_L1: "exponential"}


def _product(kernel, ell, xr, xc, y):
    z = torch.full((len(xr), y.shape[1]), float("nan"), dtype=torch.float32, device="cuda")
    nb = K.ka_gamma_workspace(len(xr), len(xc), y.shape[1], K.KA_FP32)
    assert nb >= len(xc) * (4 * y.shape[1] + 64)   # the split-FP16 route
    work = torch.zeros(nb // 4, dtype=torch.float32, device="cuda")
    return z, lambda: K.ka_gamma_apply(kernel, 1.0, ell, xr, xc, y, z, K.KA_FP32, work)


@pytest.mark.parametrize("kernel,ell", [(K.KA_GAUSSIAN, 0.2), (K.KA_GAUSSIAN, 0.05), (K.KA_EXP_L1, 0.06)])
@pytest.mark.parametrize("b", [16, 32, 64])
@pytest.mark.parametrize("same", [True, False])
def test_far_columns_decide(kernel, ell, b, same):
    X = tensor_grid_points((24, 22, 18) if b == 16 else (19, 18, 13))
    n = len(X)
    C = X if same else np.array(sorted(uniform_points(41, n).tolist(), key=lambda p: p[2]))
    Y = normal_block(43, n, b)
    Y[: n // 2, 1] = 0.0          # rows below see the columns above
    Y[n // 3:, 2] = 1e-25
    Y[600:, 3] = 0.0
    Y[::2, 4] *= 1e-7
    Y[:, 5] *= 1e-9
    d = dict(dtype=torch.float32, device="cuda")
    xr, xc, y = torch.tensor(X, **d), torch.tensor(C, **d), torch.tensor(Y, **d)
    z, run = _product(kernel, ell, xr, xc, y)
    run()
    Z = z.cpu().numpy().astype(np.float64)
    G = kernels.kernel_matrix(NAMES[kernel], xr.cpu().numpy().astype(np.float64), xc.cpu().numpy().astype(np.float64),
                              ell, 1.0)
    Yd = y.cpu().numpy().astype(np.float64)
    ref, scale = G @ Yd, np.abs(G) @ np.abs(Yd)
    ok = scale > 1e-30
    assert np.isfinite(Z).all() and (np.abs(Z[~ok]) < 1e-29).all()
    assert (np.abs(Z - ref)[ok] <= 1e-5 * scale[ok]).all()


def _half_ring(counts, r0, r1, height, angle):
    t, r, z = np.meshgrid(*(np.linspace(0, 1, n) for n in counts), indexing="ij")
    t, r, z = (a.transpose(2, 1, 0).ravel() for a in (angle * t, r0 + (r1 - r0) * r, height * z))
    return np.stack([r * np.cos(t), r * np.sin(t), z], 1)


@pytest.mark.parametrize("b,X,short,far", [
    (16, _half_ring((16, 15, 22), 8.0, 10.0, 15.0, np.pi), 0.97, 20.0),
    (32, _half_ring((14, 22, 14), 1.0, 2.0, 1.0, np.pi / 2), 0.119, 2.0),
])
def test_time(b, X, short, far):
    d = dict(dtype=torch.float32, device="cuda")
    x, y = torch.tensor(X, **d), torch.tensor(normal_block(47, len(X), b), **d)
    took = {}
    for ell in (short, far):
        _, run = _product(K.KA_GAUSSIAN, ell, x, x, y)
        for _ in range(5):
            run()
        times = []
        for _ in range(7):
            a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                run()
            e.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(e) / 20)
        took[ell] = statistics.median(times)
    assert took[short] <= 1.5 * took[far], took
