"""The projection kernels' launches (flexco_gemm_plan: host arithmetic, no GPU, the function the launchers plan with): those of the
configurations' own products are what the measurements chose, and any plan is well formed - its launches cover the output
columns exactly once with tile shapes the kernels are built for, and ranges of K are whole 64-wide stages and fit the scratch."""
import time

import numpy as np
import pytest

import paper_2402_18789_amd.binding as B
from workload import CONFIGS

pytestmark = pytest.mark.skipif(B.HOST_ONLY, reason="needs the whole library, this is a host-only build")

SPLITK_COLS = 32768          # floats of split-K scratch per row that the layer calls bring (windows of at most 256 rows: twice)


def proj_shapes(cfg):
    qkv = cfg.q_dim + 2 * cfg.kv_dim
    return {"qkv": (qkv, cfg.hidden), "o": (cfg.hidden, cfg.q_dim), "gate_up": (2 * cfg.ffn, cfg.hidden),
            "down": (cfg.hidden, cfg.ffn)}


def test_forward_plans_of_the_benchmark_step():
    cfg = CONFIGS["c2_llama8b_layer"]
    sh = proj_shapes(cfg)
    T = 1024
    plan = {k: B.flexco_gemm_plan(T, n, kk, 0, 0) for k, (n, kk) in sh.items()}
    assert plan["qkv"] == [(128, 192, 6144, 1, 4)]                                    # 256 tiles: one round
    assert plan["o"] == [(128, 128, 4096, 1, 4)] and plan["down"] == [(128, 128, 4096, 1, 4)]
    # one round of 256 x 256 tiles and one of 256 x 192 tiles side by side
    assert plan["gate_up"] == [(256, 256, 16384, 1, 2), (256, 192, 12288, 1, 2)]


def test_input_gradient_plans_by_window_length():
    c2, c4 = CONFIGS["c2_llama8b_layer"], CONFIGS["c4_qwen14b_full"]
    # a 256-row window: two row tiles of 128 on the kernel of eight wavefronts (ring of four), K whole or in four ranges; gate/up on one
    # row tile of 256, sixteen ranges
    pe = 256 * 2 * SPLITK_COLS
    for (n, kk), ranges in (((c2.ffn, c2.hidden), 1), ((c2.q_dim, c2.hidden), 4), ((c2.hidden, c2.q_dim + 2 * c2.kv_dim), 4)):
        assert B.flexco_gemm_plan(256, n, kk, 1, pe) == [(128, 128, n, ranges, 4)]
    assert B.flexco_gemm_plan(256, c2.hidden, 2 * c2.ffn, 1, pe) == [(256, 256, c2.hidden, 16, 2)]
    # 16 rows: 128 x 128 by eight wavefronts where ranges of K fill the chip, else by four, two blocks to a CU (ring of two)
    assert B.flexco_gemm_plan(16, c2.hidden, c2.hidden, 1, 16 * 2 * SPLITK_COLS) == [(128, 128, c2.hidden, 8, 4)]
    assert B.flexco_gemm_plan(16, c2.ffn, c2.hidden, 1, 0) == [(128, 128, c2.ffn, 1, 2)]
    # 1024 rows at the 14B shape: 256 x 256 tiles (down: 216; the others: 80 in three ranges)
    pe = 1024 * SPLITK_COLS
    assert B.flexco_gemm_plan(1024, c4.ffn, c4.hidden, 1, pe) == [(256, 256, c4.ffn, 1, 2)]
    for n, kk in ((c4.hidden, 2 * c4.ffn), (c4.q_dim, c4.hidden), (c4.hidden, c4.q_dim + 2 * c4.kv_dim)):
        assert B.flexco_gemm_plan(1024, n, kk, 1, pe) == [(256, 256, n, 3, 2)]
    # without scratch K stays whole
    assert B.flexco_gemm_plan(1024, c4.hidden, 2 * c4.ffn, 1, 0)[0][3] == 1
    assert B.flexco_gemm_plan(256, c2.hidden, 2 * c2.ffn, 1, 0) == [(128, 128, c2.hidden, 1, 2)]


def test_forward_products_on_256_by_128_tiles():
    for M, N, K, rows in ((1200, 6144, 4096, 256), (2048, 4096, 4096, 256), (1024, 7168, 5120, 256), (1405, 5120, 5120, 256), (256, 28672, 4096, 256),
                          (200, 28672, 4096, 224), (180, 28672, 4096, 192)):
        assert B.flexco_gemm_plan(M, N, K, 0, 0) == [(rows, 128, N, 1, 2)]
    assert B.flexco_gemm_plan(1024, 5120, 5120, 0, 0)[0][:2] == (128, 192)        # 160 blocks would have to win by a tenth


# rows of the large tiles: M cut into the fewest row tiles or into one more, whole 32s of it
def test_large_tiles_have_the_rows_there_are():
    for M, N, rows in ((300, 28672, 160), (600, 28672, 160), (800, 28672, 224), (1024, 28672, 256)):
        assert B.flexco_gemm_plan(M, N, 4096, 0, 0)[0][:2] == (rows, 256)


def test_decode_only_batches_cut_k():
    c2 = CONFIGS["c2_llama8b_layer"]
    # up to 64 rows: the 64-row tile; up to 256: the 128-row tile
    for M, tile in ((16, (64, 128)), (64, (64, 128)), (65, (128, 128)), (256, (128, 128))):
        (bm, bn, cols, splits, stages), = B.flexco_gemm_plan(M, c2.q_dim + 2 * c2.kv_dim, c2.hidden, 0, M * SPLITK_COLS)
        assert (bm, bn, cols) == tile + (6144,) and splits > 1
    assert B.flexco_gemm_plan(16, 6144, c2.hidden, 0, 0) == [(64, 128, 6144, 1, 6)]    # no scratch, no cut
    assert B.flexco_gemm_plan(100, 6144, c2.hidden, 0, 0) == [(128, 128, 6144, 1, 4)]


def test_any_plan_is_well_formed():
    g = np.random.default_rng(7)
    shapes = {(64, 128), (128, 128), (128, 192), (160, 256)} | {(rows, bn) for rows in (192, 224, 256) for bn in (128, 192, 256)}
    for n in range(3000):
        M = int(g.integers(1, 5000 if n % 10 else 70))
        N = 8 * int(g.integers(1, 8000))
        K = 64 * int(g.integers(1, 900))
        trans = int(g.integers(0, 2))
        pe = int(g.choice([0, M * SPLITK_COLS, 1 << 20]))
        plan = B.flexco_gemm_plan(M, N, K, trans, pe)
        assert 1 <= len(plan) <= 2, (M, N, K, trans, pe, plan)
        assert sum(p[2] for p in plan) == N
        for i, (bm, bn, cols, splits, stages) in enumerate(plan):
            assert (bm, bn) in shapes and cols > 0 and stages in ((6,) if bm == 64 else (2, 4))
            assert (bm == 64) == (M <= 64 and not trans)
            if trans:
                assert ((bm, bn) == (128, 128) or (bm > 128 and bn == 256)) and len(plan) == 1
            if bm > 128:
                assert stages == 2 and (M + bm - 1) // bm <= (M + 255) // 256 + 1
            if bn == 128 and bm > 128:
                assert len(plan) == 1 and splits == 1
            if i + 1 < len(plan):
                assert cols % bn == 0                       # the next launch starts at a tile boundary
            # (equal cuts of the four-wavefront 128 x 128 tiles)
            assert splits >= 1 and (bm != 128 or (trans and stages == 4) or K % (64 * splits) == 0)
            if splits > 1:
                assert splits * M * N <= pe and len(plan) == 1
                assert K // 64 // splits >= 4


# Planning is host time of every call: the search over the columns does not cost by their number (a loss head's 152064 columns
# against 1024; every one of 594 column splits priced: 10 to 20 times as long)
def test_planning_of_many_columns_is_quick():
    def us(M, N, K):
        best = 1e9
        for _ in range(20):
            t0 = time.perf_counter()
            for _ in range(50):
                B.flexco_gemm_plan(M, N, K, 0, 0)
            best = min(best, time.perf_counter() - t0)
        return best / 50 * 1e6
    few, many = us(300, 1024, 5120), us(300, 152064, 5120)
    assert many < 3 * few, (few, many)


def test_rejects_shapes_the_matrix_core_path_does_not_take():
    for args in ((0, 64, 64, 0, 0), (64, 64, 64, 0, -1)):
        with pytest.raises(B.FlexcoError):
            B.flexco_gemm_plan(*args)
    for args in ((64, 64, 72, 0, 0), (64, 12, 64, 1, 0)):
        with pytest.raises(B.FlexcoError):
            B.flexco_gemm_plan(*args)
