"""flexco_gemm_k_ranges (host arithmetic, no GPU): the ranges of the plan's 256-column tiles, which fit the scratch and hold whole stages,
and are taken where the 256 x 256 tiles of the larger models' products would leave CUs idle."""
import numpy as np
import pytest

import paper_2402_18789_amd.binding as B

pytestmark = pytest.mark.skipif(B.HOST_ONLY, reason="needs the whole library, this is a host-only build")


def test_ranges_are_well_formed():
    g = np.random.default_rng(11)
    taken = 0
    for n in range(3000):
        M, N, K = int(g.integers(1, 5000 if n % 10 else 70)), 8 * int(g.integers(1, 8000)), 64 * int(g.integers(1, 900))
        pe = int(g.choice([0, M * 32768, 1 << 20]))
        trans = int(g.integers(0, 2))
        r = B.flexco_gemm_k_ranges(M, N, K, trans, pe)
        assert 0 <= r <= 16 and not (M <= 64 and r > 0 and not trans)      # (forward, few rows: the plan's 64-row tiles)
        plan = B.flexco_gemm_plan(M, N, K, trans, pe)
        large = len(plan) == 1 and plan[0][0] > 128 and plan[0][1] == 256
        assert r == (plan[0][3] if large and (trans or plan[0][3] > 1) else 0)
        if r > 1:
            taken += 1
            assert r * M * N <= pe and K // 64 >= 4 * r
    assert taken > 50


def test_ranges_of_the_models_products():
    # (forward: without scratch, or with the tiles filling the chip, the plan stands)
    assert B.flexco_gemm_k_ranges(1024, 4096, 14336, 0, 0) == 0
    assert B.flexco_gemm_k_ranges(2048, 24576, 5120, 0, 2048 * 13824) == 0
    assert B.flexco_gemm_k_ranges(2048, 4096, 14336, 0, 2048 * 14336) == 2
    assert B.flexco_gemm_k_ranges(1405, 5120, 27648, 0, 1405 * 27648) == 2
    # the loss head's input gradient, 2004 stages of K in eight ranges of 250 and 251
    assert B.flexco_gemm_k_ranges(512, 4096, 128256, 1, 16 * 512 * 4096) == 8
    assert B.flexco_gemm_k_ranges(1024, 5120, 7168, 1, 1024 * 32768) == 3


def test_ranges_reject_what_the_plan_rejects():
    for args in ((0, 64, 64, 0, 0), (64, 64, 64, 0, -1), (64, 64, 72, 0, 0), (64, 12, 64, 1, 0)):
        with pytest.raises(B.FlexcoError):
            B.flexco_gemm_k_ranges(*args)
