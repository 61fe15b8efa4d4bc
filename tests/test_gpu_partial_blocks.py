"""An operator application of fewer vectors than the block width after a wider
one: its result does not depend on what the wider one left behind."""
import numpy as np
import pytest
import torch

import paper_2101_00629_amd as K
from workloads import normal_block

pytestmark = pytest.mark.gpu


def _problem(precision):
    return K.Problem(K.make_desc("galerkin", "cube", 2, (18, 17, 16), "gaussian", 0.5, block=32, precision=precision))


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("bad", [np.nan, np.inf, 1e300])
def test_narrow_block_after_a_wide_one(precision, bad):
    fresh, used = _problem(precision), _problem(precision)
    X = torch.tensor(normal_block(41, 32, fresh.N), device="cuda")
    want, got = (torch.full((5, fresh.N), 7.0, dtype=torch.float64, device="cuda") for _ in range(2))
    K.ka_apply_A(fresh.h, K.KA_APRIME, X[:5], want)
    X[31, 1234] = bad
    wide = torch.empty_like(X)
    K.ka_apply_A(used.h, K.KA_APRIME, X, wide)
    K.ka_apply_A(used.h, K.KA_APRIME, X[:5], got)
    torch.cuda.synchronize()
    fresh.close()
    used.close()
    assert torch.isfinite(want).all() and torch.equal(want, got)
