"""Layers on few tokens, where a projection leaves its partial sums to the kernel that reads it next (the rotation, the
second norm), and the merge of many key splits (run with -m gpu on an MI355X)."""
import numpy as np
import pytest
import torch

import bench
from workload import gen, CONFIGS

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2402_18789_amd.binding as B
    from paper_2402_18789_amd import host as HH
    from gpu_common import Case, TOL, assert_close
    from test_gpu_parity import attention_case, run_layer_case

# K of 32 stages: three ranges of it per projection at up to 64 tokens
WIDE = CONFIGS["c2_llama8b_layer"].with_(name="wide_bf16", hidden=2048, n_q_heads=16, n_kv_heads=4, head_dim=128, ffn=2816,
                                         qkv_bias=True, lora_targets=("q", "v", "o", "gate", "down"))


# 30 tokens a pass (64-row tiles), then 130 (128-row tiles)
@pytest.mark.parametrize("chunk,window", [(12, 14), (60, 66)])
def test_layer_partial_sums_left_to_the_next_kernel(chunk, window):
    print(f"layer of few tokens: prefill chunk {chunk}, window {window}", flush=True)
    b = gen.batch_scaled(17, 4, 3, 90, [(0, chunk, 2 * chunk)], [(0, window, 2 * window)])
    assert b.n_tokens <= 256
    run_layer_case(WIDE, b, ft_window=window, prefill_chunk=chunk, bwd_windows=[window, window], seed=17)


# ... of a run's v rows, added by the blocks that store its positions side by side: pages of 16 (whole runs and pieces of them), of 24 and of
# 12 (no 16-byte pieces), runs of 2 to 15 tokens, and v rows of more pieces than a block has threads (40 kv heads)
@pytest.mark.parametrize("kv,page,chunk,window", [(4, 16, 33, 20), (4, 24, 30, 25), (4, 12, 29, 17), (4, 16, 2, 15), (40, 16, 30, 19)])
def test_layer_partial_sums_of_runs_of_tokens(kv, page, chunk, window):
    cfg = WIDE.with_(name="runs", n_kv_heads=kv, n_q_heads=max(16, kv), page_size=page, lora_targets=("q", "v"))
    b = gen.mixed_batch(page, 23, decode_ctx=(1, 5, 40), prefill=[(3, chunk, 3 + chunk)], finetune=[(0, window, 2 * window + 1)])
    print(f"layer of {b.n_tokens} tokens, {kv} kv heads, pages of {page}", flush=True)
    assert B.flexco_gemm_plan(b.n_tokens, cfg.q_dim + 2 * cfg.kv_dim, cfg.hidden, 0, b.n_tokens * 32768)[0][3] > 1
    run_layer_case(cfg, b, ft_window=window, prefill_chunk=chunk, bwd_windows=[window, window + 1], seed=23)


# ... in about the time that as many single tokens take (one thread per piece and run: three to four times as long)
def test_rotation_of_a_chunks_partial_sums_takes_no_longer_than_of_single_tokens():
    kid, us = B.KERNEL_IDS["elemwise"], {}
    cfg = WIDE.with_(name="rope_time", n_kv_heads=8, lora_targets=())
    dev = HH.DeviceLayer(cfg, gen.layer_weights(cfg, 29, 0))
    for name, b in (("single", gen.mixed_batch(16, 1, decode_ctx=(20,) * 128)), ("chunk", gen.mixed_batch(16, 1, prefill=[(0, 128, 128)]))):
        db, pool = HH.DeviceBatch(cfg, b.requests, b.seq_pages, b.num_pages), HH.DevicePool(cfg, b.num_pages)
        ws = HH.Workspace(dev.c, 128, db.host_maps.n_parts)
        x = torch.randn(128, cfg.hidden, device="cuda").bfloat16()
        y = torch.empty_like(x)
        B.flexco_layer_forward(dev.c, dev.w, None, db.maps, x, y, pool.c, None, ws.ptr, ws.bytes)
        B.flexco_kernel_timer_sample(kid, 1)
        B.flexco_kernel_timer_start(kid, 64)
        for _ in range(8):
            B.flexco_layer_forward(dev.c, dev.w, None, db.maps, x, y, pool.c, None, ws.ptr, ws.bytes)
        torch.cuda.synchronize()
        each = B.flexco_kernel_timer_read(kid)
        B.flexco_kernel_timer_stop(kid)
        us[name] = 1e3 * min(each[1::len(each) // 8])           # the rotation, between the two norms
    print(f"rotation: {us}", flush=True)
    assert B.flexco_gemm_plan(128, cfg.q_dim + 2 * cfg.kv_dim, cfg.hidden, 0, 128 * 32768)[0][3] > 1
    assert us["chunk"] <= 1.6 * us["single"]


# Rows of every weight a multiple of 4 KB apart, at most 128 tokens: the column tiles of the products start at stages of their own - the 64-row
# form cut over K in unequal ranges, the 128 x 128 form in equal ones, the gated form of either
@pytest.mark.parametrize("chunk,window", [(12, 14), (30, 30), (31, 30), (47, 46), (62, 62)])
@pytest.mark.parametrize("hidden,ffn", [(2048, 4096), (2048, 6144)])
def test_layer_products_from_their_own_stage(hidden, ffn, chunk, window):
    cfg = WIDE.with_(name="spread", hidden=hidden, ffn=ffn)
    b = gen.batch_scaled(17, 4, 3, 90, [(0, chunk, 2 * chunk)], [(0, window, 2 * window)])
    T, bm = b.n_tokens, 64 if b.n_tokens <= 64 else 128
    print(f"layer of {T} tokens, hidden {hidden}, ffn {ffn}", flush=True)
    assert T == 4 + chunk + window <= 128
    unequal = 0
    for N, K in ((cfg.q_dim + 2 * cfg.kv_dim, hidden), (hidden, cfg.q_dim), (hidden, ffn)):
        (rows, cols, _, splits, _), = B.flexco_gemm_plan(T, N, K, 0, T * 32768)
        assert (rows, cols) == (bm, 128) and splits > 1 and K % 2048 == 0 and B.flexco_gemm_k_ranges(T, N, K, 0, T * 32768) == 0
        unequal += K // 64 % splits != 0
    assert unequal == (3 if bm == 64 else 0)
    assert B.flexco_gemm_plan(T, 2 * ffn, hidden, 0) == [(bm, 128, 2 * ffn, 1, 6 if bm == 64 else 4)]
    run_layer_case(cfg, b, ft_window=window, prefill_chunk=chunk, bwd_windows=[window, window], seed=17)


# A gated product that covers the chip in one round of 128-column tiles (up to 256 tokens) or 256-column ones, of 192, 256, 160, 192
# and 224 rows; adapter and finetune rows, a last column tile of eight activations
@pytest.mark.parametrize("chunk,window,tile", [(60, 66, (192, 128)), (141, 96, (256, 128)), (150, 110, (160, 256)), (200, 130, (192, 256)),
                                               (220, 196, (224, 256))])
def test_layer_gated_product_on_tiles_of_its_rows(chunk, window, tile):
    cfg = WIDE.with_(name="gated_rows", ffn=13832)
    b = gen.batch_scaled(17, 4, 3, 90, [(0, chunk, 2 * chunk)], [(0, window, 2 * window)])
    print(f"layer of {b.n_tokens} tokens, ffn {cfg.ffn}", flush=True)
    assert B.flexco_gemm_plan(b.n_tokens, 2 * cfg.ffn, cfg.hidden, 0) == [(*tile, 2 * cfg.ffn, 1, 2)]
    run_layer_case(cfg, b, ft_window=window, prefill_chunk=chunk, bwd_windows=[window, window], seed=17)


# K that is no multiple of 64 runs on the type-generic kernel, uncut, whatever the planner of the matrix-core path would
# do with it: the qkv and down products (hidden, ffn), then o (q_dim = 27 x 48); few tokens, no adapter rows, a bias
@pytest.mark.parametrize("hidden,heads,kv,d", [(2056, 16, 4, 128), (2048, 27, 9, 48), (1352, 11, 11, 128)])
def test_layer_of_a_width_the_matrix_cores_do_not_take(hidden, heads, kv, d):
    cfg = WIDE.with_(name=f"odd_{hidden}_{heads * d}", hidden=hidden, n_q_heads=heads, n_kv_heads=kv, head_dim=d, ffn=1400, lora_targets=())
    for n_decode, chunk in ((8, 0), (40, 8), (64, 36), (64, 236)):
        print(f"{cfg.name}: {n_decode} decode tokens, a chunk of {chunk}", flush=True)
        b = gen.mixed_batch(cfg.page_size, 23, decode_ctx=tuple(range(3, 3 + n_decode)), prefill=[(5, chunk, 5 + chunk)] if chunk else [])
        case = Case(cfg, b, seed=23)
        got, ref, _ = case.forward(b, gen.layer_input(cfg, 23, b.n_tokens))
        assert_close("y", got, ref, TOL["bf16"])


# More than 256 tokens: the [T, 2 ffn] buffer of gate and up is lent to the other projections, whose sums of unequal ranges
# of K lie in it until the norm (o) or the rotation (qkv) has read them; with the finetune window's adapter rows folded
# in, and without adapters
O_CUT = CONFIGS["c2_llama8b_layer"].with_(name="o_cut", hidden=512, n_q_heads=64, n_kv_heads=8, head_dim=128, ffn=2816, qkv_bias=True,
                                          lora_targets=("q", "v", "o", "gate", "down"))
QKV_CUT = O_CUT.with_(name="qkv_cut", hidden=4096, n_q_heads=4, n_kv_heads=1)


@pytest.mark.parametrize("adapter", [True, False])
@pytest.mark.parametrize("cfg", [O_CUT, QKV_CUT])
def test_layer_partial_sums_in_the_lent_buffer(cfg, adapter):
    b = gen.batch_scaled(29, 5, 3, 90, [(0, 131, 262)], [(0, 141, 282)])
    T = b.n_tokens
    assert T == 277
    cuts = {"qkv": B.flexco_gemm_k_ranges(T, cfg.q_dim + 2 * cfg.kv_dim, cfg.hidden, 0, T * cfg.ffn),
            "o": B.flexco_gemm_k_ranges(T, cfg.hidden, cfg.q_dim, 0, T * cfg.ffn)}
    print(f"layer of {T} tokens, {cfg.name}, cuts {cuts}, adapter {adapter}", flush=True)
    r, K = (cuts["o"], cfg.q_dim) if cfg is O_CUT else (cuts["qkv"], cfg.hidden)
    assert r > 1 and (K // 64) % r != 0
    if not adapter:
        cfg = cfg.with_(name=cfg.name + "_base", lora_targets=())
    run_layer_case(cfg, b, ft_window=141, prefill_chunk=131, bwd_windows=[141, 141], seed=29)


# the down product's partial sums take h, qkv and attn in front of that buffer as well
@pytest.mark.parametrize("adapter", [True, False])
@pytest.mark.parametrize("ffn", [5632, 6016])
def test_layer_down_partial_sums_past_the_lent_buffer(ffn, adapter):
    cfg = WIDE.with_(name="down_cut", ffn=ffn, lora_targets=("q", "v", "o", "gate", "down") if adapter else ())
    b = gen.batch_scaled(29, 5, 3, 90, [(0, 131, 262)], [(0, 141, 282)])
    T = b.n_tokens
    ranges = [B.flexco_gemm_k_ranges(T, cfg.hidden, ffn, 0, T * w) for w in (ffn, ffn + cfg.hidden // 2 + cfg.q_dim + cfg.kv_dim)]
    print(f"layer of {T} tokens, ffn {ffn}, ranges of the down product {ranges}, adapter {adapter}", flush=True)
    assert T == 277 and ranges[1] > max(1, ranges[0])
    run_layer_case(cfg, b, ft_window=141, prefill_chunk=131, bwd_windows=[141, 141], seed=29)


# the benchmark's account of the projections' launches against those that the layer makes
@pytest.mark.parametrize("ffn", [2816, 5632])
def test_launches_of_the_projections_are_those_the_benchmark_counts(ffn):
    cfg = WIDE.with_(name="down_cut", ffn=ffn, lora_targets=())
    b = gen.batch_scaled(29, 5, 3, 90, [(0, 131, 262)], [(0, 141, 282)])
    db = HH.DeviceBatch(cfg, b.requests, b.seq_pages, b.num_pages)
    T, dev = db.host_maps.T, HH.DeviceLayer(cfg, gen.layer_weights(cfg, 29, 0))
    counted = sum(n for _, _, n in bench.forward_launches(B, cfg, T))
    print(f"layer of {T} tokens, ffn {ffn}: {counted} launches counted", flush=True)
    pool, ft = HH.DevicePool(cfg, b.num_pages), HH.DeviceFtState(cfg, 282)
    ws = HH.Workspace(dev.c, T, db.host_maps.n_parts, 141, 282)
    x = torch.randn(T, cfg.hidden, device="cuda").bfloat16()
    y = torch.empty_like(x)
    kid = B.KERNEL_IDS["gemm_fwd"]
    B.flexco_kernel_timer_sample(kid, 1)
    B.flexco_kernel_timer_start(kid, 64)
    B.flexco_layer_forward(dev.c, dev.w, dev.lora, db.maps, x, y, pool.c, ft.c, ws.ptr, ws.bytes)
    torch.cuda.synchronize()
    each = B.flexco_kernel_timer_read(kid)
    B.flexco_kernel_timer_stop(kid)
    assert T == 277 and len(each) == counted


# (split: pages of 16 keys) contexts of one split, then of up to six, then of 1, 2, 8, 9 and 12
@pytest.mark.parametrize("split", [24, 4, 2])
def test_attention_merge_of_many_splits(split):
    print(f"attention, key splits of {split} pages", flush=True)
    cfg = WIDE
    batch = gen.mixed_batch(cfg.page_size, 4, decode_ctx=(1, 17, 256, 270, 384), prefill=[(0, 33, 33), (270, 18, 288)], finetune=[(50, 21, 71)])
    out, a_o, lse, lse_o = attention_case(cfg, batch, split)
    assert_close("attention out", out, a_o, TOL[cfg.dtype])
    assert float(np.max(np.abs(lse - lse_o))) <= 2e-2


# the type-generic LoRA kernels: up to 256 rows of narrow products of a low rank (at these widths: every target at ranks of
# up to 16, q, v and o at ranks of up to 32) in one launch with the products' sums kept in LDS, others in two
@pytest.mark.parametrize("window", [256, 257])
@pytest.mark.parametrize("rank", [5, 16, 24, 40])
def test_generic_lora_rows(window, rank):
    print(f"type-generic LoRA of rank {rank}, windows of {window}", flush=True)
    cfg = CONFIGS["c1_tiny_f32"].with_(name="tiny_r%d" % rank, lora_rank=rank, lora_targets=("q", "v", "o", "gate", "up", "down"))
    b = gen.mixed_batch(cfg.page_size, 19, decode_ctx=(1, 40), finetune=[(0, window, 2 * window)])
    run_layer_case(cfg, b, ft_window=window, prefill_chunk=32, bwd_windows=[window, window], seed=19)


# the matrix-core shrink products x A^T and dy B: blocks of 8 and 16 rows with a remainder, one to four tiles of
# ranks, fewer groups of 128 columns than wavefronts, and contractions of over 16384 columns cut
# over blocks in unequal ranges; rows of other adapters and of none beside them
@pytest.mark.parametrize("rank,ffn,window", [(16, 16512, 23), (16, 1408, 9), (32, 16512, 140), (48, 1408, 23), (64, 1408, 140), (16, 1408, 1100)])
def test_shrink_products(rank, ffn, window):
    print(f"LoRA rank {rank}, ffn {ffn}, windows of {window}", flush=True)
    cfg = WIDE.with_(name="shrink_r%d" % rank, hidden=640, n_q_heads=5, n_kv_heads=1, ffn=ffn, lora_rank=rank,
                     lora_targets=("q", "k", "v", "o", "gate", "up", "down"))
    b = gen.mixed_batch(cfg.page_size, 31, decode_ctx=(1, 40, 3), prefill=[(0, 37, 37)], finetune=[(0, window, 2 * window)])
    run_layer_case(cfg, b, ft_window=window, prefill_chunk=37, bwd_windows=[window, window], seed=31)


# fp32 gate/up product of few tiles and many columns: with the norm within, the gate not - about what the plain product of its size takes
# (1.5 to 1.7 times that with half the blocks and half the steps in flight)
def test_fp32_gate_up_product_of_few_tiles_takes_about_the_plain_products_time():
    kid, T = B.KERNEL_IDS["generic"], 16
    cfg = CONFIGS["c1_tiny_f32"].with_(name="long_f32", hidden=8192, ffn=512, lora_targets=())
    dev = HH.DeviceLayer(cfg, gen.layer_weights(cfg, 31, 0))
    b = gen.mixed_batch(16, 1, decode_ctx=(20,) * T)
    db, pool = HH.DeviceBatch(cfg, b.requests, b.seq_pages, b.num_pages), HH.DevicePool(cfg, b.num_pages)
    ws = HH.Workspace(dev.c, T, db.host_maps.n_parts)
    x = torch.randn(T, cfg.hidden, device="cuda")
    y, gu = torch.empty_like(x), torch.empty(T, 2 * cfg.ffn, device="cuda")

    def timed(fn):
        fn()
        B.flexco_kernel_timer_sample(kid, 1)
        B.flexco_kernel_timer_start(kid, 256)
        for _ in range(10):
            fn()
        torch.cuda.synchronize()
        each = B.flexco_kernel_timer_read(kid)
        B.flexco_kernel_timer_stop(kid)
        n = len(each) // 10
        return [1e3 * min(each[i::n]) for i in range(n)]
    layer = timed(lambda: B.flexco_layer_forward(dev.c, dev.w, None, db.maps, x, y, pool.c, None, ws.ptr, ws.bytes))
    (plain,) = timed(lambda: B.flexco_gemm(x, dev.t["wgu"], gu, None, None, T, 2 * cfg.ffn, cfg.hidden, 0, B.FLEXCO_F32))
    print(f"type-generic launches of the layer {layer}, the plain product {plain:.1f} us", flush=True)
    assert layer[-2] <= 1.35 * plain             # qkv, (attention,) o, gate/up, down
