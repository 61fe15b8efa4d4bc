"""Scratch that the kernel product states (no GPU): columns go in finer splits,
with partial sums, only where these cost less than the shorter chains save."""
import pytest

import paper_2101_00629_amd as K


@pytest.mark.parametrize("b", [16, 32, 64])
@pytest.mark.parametrize("precision", [K.KA_FP32, K.KA_BF16X3])
def test_many_rows_and_few_columns_take_no_partial_sums(b, precision):
    sizes = [(20000, 65), (33000, 65), (33000, 130), (66000, 65), (66000, 130), (130000, 65), (500000, 65)]
    for nr, nc in sizes:
        if nr * nc * b >= 4e8:   # split FP16
            continue
        ysplit = -(-nc // 64) * 64 * b * 4 if precision == K.KA_BF16X3 else 0
        assert K.ka_gamma_workspace(nr, nc, b, precision) == ysplit, (nr, nc)


@pytest.mark.parametrize("b", [16, 32, 64])
def test_small_products_keep_their_fine_splits(b):
    for nr, nc in [(300, 1000), (1000, 1000), (3000, 600), (3000, 1000)]:
        # more partial sums than splits of 512 columns have
        assert K.ka_gamma_workspace(nr, nc, b, K.KA_FP32) > max(1, nc // 512) * nr * b * 4, (nr, nc)


def test_exponential_products_that_split_fp16_does_not_pay_for():
    # the scratch is for either kernel, that of the routes in FP32 included
    for nr, nc, b in [(20000, 1300, 16), (5832, 5832, 16), (130000, 65, 64), (300000, 65, 32)]:
        f16 = -(-nc // 512) * 512 * (4 * b + 64)
        assert K.ka_gamma_workspace(nr, nc, b, K.KA_FP32) >= f16, (nr, nc, b)


def _held(method, p, nel, kernel, nq=None):
    """What a request holds beyond the setup of its problem alone, and the scratch
    that its product would take on its own beyond that of a batched launch."""
    d = K.make_desc(method, "cube", p, nel, kernel, 0.5, nq=nq)
    N, Nt, Nq = K.ka_desc_size(d)
    nr, nc = (N, Nq) if method == "collocation" else (Nt, Nt)
    stated, blocks = K.ka_gamma_workspace(nr, nc, 16, K.KA_FP32), -(-nr // 256)
    ns = max(1, min(-(-2048 // blocks), nc // 512, 64))      # splits of 512 columns and up
    ns = -(-ns // 8) * 8 if ns >= 8 else ns
    ns = -(-nc // (-(-(-(-nc // ns)) // 128) * 128))
    extra = max(stated, 256) - (max(-(-ns * nr * 64 // 256), 1) * 256 if ns > 1 else 256)
    return K.ka_request_bytes(d, 30) - K.ka_footprint(d), extra if blocks * ns < 2048 else 0


@pytest.mark.parametrize("a,b", [
    (("collocation", 2, (16, 14, 12), "gaussian"), ("collocation", 2, (16, 14, 12), "gaussian", 2)),
    (("galerkin", 3, (12, 12, 12), "gaussian"), ("galerkin", 3, (12, 12, 12), "exponential"))])
def test_a_served_request_holds_the_scratch_that_its_product_takes(a, b):
    # The solver's workspace depends on the unknowns, which a and b have in common.
    # Products that run in batched launches take the splits of 512 columns; the
    # exponential problem's product is large enough to run on its own.
    (held_a, extra_a), (held_b, extra_b) = _held(*a), _held(*b)
    assert extra_a > 0 and (extra_b == 0) == (b[3] == "exponential")
    assert held_a + extra_a == held_b + extra_b
