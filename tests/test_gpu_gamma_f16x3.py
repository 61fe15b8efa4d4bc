"""The split-FP16 route of the FP32 kernel product (large products through
ka_gamma_apply) against the FP64 oracle: sizes at the edges of its row blocks
and column groups, its two exponent forms, the scales that keep FP16 in range,
values that are not finite, and the FP32 route that less scratch selects.

Bar: |Z - Z_ref| <= tol (|Gamma| |Y|) elementwise, tol = 1e-5 as for the FP32
matrix cores.  The parts of a value are 2^-23 off at most, the dropped lo lo
2^-22, the exponent a few 2^-24 of its size (|e| <= 20 where Gamma counts) and
exp2 2^-23; sums of at most 16 MFMAs of 4 roundings each add 64 2^-24 at most:
together below 6e-6.  FP16's last place adds 2^-40 of the largest |Y| per pair
where a group's box says nothing about the row (scattered columns).
"""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from oracle import kernels
from workloads import normal_block, tensor_grid_points, uniform_points

pytestmark = pytest.mark.gpu

TOL = 1e-5
KNAME = {K.KA_GAUSSIAN: "gaussian", K.KA_EXP_L1: "exponential"}


def _run(kernel, ell, Xr, Xc, Y, full=True):
    xr = torch.tensor(Xr, dtype=torch.float32, device="cuda")
    xc = torch.tensor(Xc, dtype=torch.float32, device="cuda")
    y = torch.tensor(Y, dtype=torch.float32, device="cuda")
    z = torch.full((len(Xr), Y.shape[1]), float("nan"), dtype=torch.float32, device="cuda")
    nb = K.ka_gamma_workspace(len(Xr), len(Xc), Y.shape[1], K.KA_FP32)
    # the route under test needs its scratch: Y and the points in FP16 parts
    assert nb >= len(Xc) * (4 * Y.shape[1] + 64)
    if not full:
        nb -= len(Xc) * 4 * Y.shape[1]
    work = torch.full((nb // 4,), float("nan"), dtype=torch.float32, device="cuda")
    K.ka_gamma_apply(kernel, 1.0, ell, xr, xc, y, z, K.KA_FP32, work)
    torch.cuda.synchronize()
    return z.cpu().numpy().astype(np.float64)


def _reference(kernel, ell, Xr, Xc, Y):
    Xr, Xc, Y = (np.asarray(a, dtype=np.float32).astype(np.float64) for a in (Xr, Xc, Y))
    G = kernels.kernel_matrix(KNAME[kernel], Xr, Xc, ell, 1.0)
    return G @ Y, np.abs(G) @ np.abs(Y)


def _check(kernel, ell, Xr, Xc, Y, tol=TOL, **kw):
    Z = _run(kernel, ell, Xr, Xc, Y, **kw)
    ref, scale = _reference(kernel, ell, Xr, Xc, Y)
    assert np.isfinite(Z).all()
    bar = tol * scale + 2.0 ** -40 * np.abs(Y).sum(axis=0)
    assert (np.abs(Z - ref) <= bar).all(), (np.abs(Z - ref) / bar).max()


@pytest.mark.parametrize("kernel,ell", [(K.KA_GAUSSIAN, 0.4), (K.KA_EXP_L1, 0.6)])
@pytest.mark.parametrize("b,nr,nc", [(16, 255, 100353), (16, 257, 99999), (16, 8000, 3201), (32, 256, 49217),
                                     (32, 4097, 3136), (32, 65, 200001), (64, 127, 49215), (64, 129, 48704),
                                     (64, 6200, 1025), (64, 12500, 511)])
def test_edges_of_blocks_and_groups(kernel, ell, b, nr, nc):
    Xr = uniform_points(nr + 1, nr) if nr < 1000 else tensor_grid_points((10, 10, -(-nr // 100)))[:nr]
    _check(kernel, ell, Xr, uniform_points(nc, nc), normal_block(b + nr, nc, b, dtype=np.float32))


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
@pytest.mark.parametrize("b", [16, 64])
def test_scales_keep_small_kernels_and_odd_blocks(kernel, b):
    # rows near their columns, rows at a distance where Gamma is about 1e-12 from
    # a face and from a corner of the columns' box; vectors of very different
    # size, one of zeros, and one whose size jumps from column group to group
    ell = 0.25
    Xc = np.concatenate([tensor_grid_points((40, 40, 12)), uniform_points(3, 800)])
    far = 5.3 * ell if kernel == K.KA_GAUSSIAN else 9.0 * ell
    Xr = np.concatenate([uniform_points(1, 700), uniform_points(2, 600) * [0.05, 1, 1] + [1.0 + far, 0, 0],
                         uniform_points(4, 300) * 0.1 - far / np.sqrt(3.0)])
    Y = normal_block(5, len(Xc), b)
    Y[:, 1] *= 1e-30
    Y[:, 2] *= 1e30
    Y[:, 3] = 0.0
    Y[:, 4] *= 10.0 ** (np.arange(len(Xc)) // 512 % 30 - 15)
    Z = _run(kernel, ell, Xr, Xc, Y)
    ref, scale = _reference(kernel, ell, Xr, Xc, Y)
    ok = scale > 1e-36
    assert np.isfinite(Z).all() and (Z[:, 3] == 0).all() and ok[:, [0, 2, 4]].all()
    assert (np.abs(Z - ref)[ok] / scale[ok]).max() < TOL


def test_points_off_the_lattice_take_differences():
    # some columns and some rows further than the Gram form's range from the
    # launch's centre (ell = 0.02: 31 scaled units are 0.52), the rest inside.
    # Differences of FP32 coordinates of up to 45 units (half of 1.5 / 0.02
    # sqrt(log2 e)) are 2 * 45 * 2^-24 off, an exponent d^2 with d <= 6 (Gamma >=
    # 2^-36) 12 times that, Gamma ln 2 times that: 4.5e-5, with the rest 5.5e-5.
    ell = 0.02
    Xr = np.concatenate([tensor_grid_points((20, 20, 4)) * 0.2, uniform_points(7, 900) * 1.5])
    Xc = np.concatenate([tensor_grid_points((25, 25, 20)) * 0.2, uniform_points(8, 12000) * 1.5])
    _check(K.KA_GAUSSIAN, ell, Xr, Xc, normal_block(9, len(Xc), 16), tol=5.5e-5)
    # large offsets: coordinates relative to the launch's centre
    _check(K.KA_GAUSSIAN, 8.0, Xr[:1000] * 100 + 3000.0, Xc * 100 + 3000.0, normal_block(9, len(Xc), 32))


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
def test_values_that_are_not_finite(kernel):
    # +inf, -inf and NaN in three vectors of one column, NaN in a row's and inf
    # in a column's coordinates: the vectors, the row and nothing else show it
    b, ell = 16, 0.5
    Xr, Xc = uniform_points(11, 1500), uniform_points(12, 20000)
    Y = normal_block(13, len(Xc), b)
    Y[777, 1], Y[777, 2], Y[777, 3] = np.inf, -np.inf, np.nan
    Xr[40] = np.nan
    Z = _run(kernel, ell, Xr, Xc, Y)
    rows = np.arange(len(Xr)) != 40
    assert np.isnan(Z[40]).all() and np.isnan(Z[:, 3]).all()
    assert (Z[rows, 1] == np.inf).all() and (Z[rows, 2] == -np.inf).all()
    clean = [j for j in range(b) if j not in (1, 2, 3)]
    ref, scale = _reference(kernel, ell, Xr[rows], Xc, Y[:, clean])
    assert (np.abs(Z[rows][:, clean] - ref) / scale).max() < TOL
    # a point at infinity contributes exp2(-inf) = 0
    Xc2 = Xc.copy()
    Xc2[9000, 0] = np.inf
    Y2 = normal_block(14, len(Xc), b)
    Y3 = Y2.copy()
    Y3[9000] = 0.0
    Z2 = _run(kernel, ell, Xr[rows], Xc2, Y2)
    ref, scale = _reference(kernel, ell, Xr[rows], Xc, Y3)
    assert (np.abs(Z2 - ref) / scale).max() < TOL


@pytest.mark.parametrize("kernel", [K.KA_GAUSSIAN, K.KA_EXP_L1])
def test_less_scratch_takes_the_fp32_matrix_cores(kernel):
    Xr, Xc = tensor_grid_points((12, 11, 10)), uniform_points(15, 25000)
    _check(kernel, 0.4, Xr, Xc, normal_block(16, len(Xc), 32), full=False)
