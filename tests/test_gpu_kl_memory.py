"""Device memory of a K-L sampling call whose grid is fine in two directions only."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K

pytestmark = pytest.mark.gpu


def test_memory_of_a_plane_grid():
    # the intermediate blocks (300 x 300 x 42 values a vector, two of them) go 32
    # vectors at a time where they are large: 1.94 GB, and 0.1 GB for the rest
    p = K.Problem(K.make_desc("galerkin", "cube", 2, (8, 8, 40), "gaussian", 0.5))
    rng = np.random.default_rng(52)
    M = 64
    V = torch.tensor(rng.standard_normal((M, p.N)), device="cuda")
    xi = torch.tensor(rng.standard_normal((4, M)), device="cuda")
    grid = [np.linspace(0, 1, 300), np.linspace(0, 1, 300), np.array([0.5])]
    F = torch.empty((4, 90000), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    K.ka_kl_sample(p.h, np.ones(M), V, grid, xi, F)
    used = before - torch.cuda.mem_get_info()[0]
    p.close()
    assert used < 2.2e9, used
