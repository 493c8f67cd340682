"""The bf16 projections' tile kernels at the sizes where they can go wrong: each tile shape with ragged last rows and
columns, one, two and three 64-wide stages of K, K in unequal ranges, weights past 4 GiB (run with -m gpu on an MI355X)."""
from types import SimpleNamespace

import pytest
import torch

from workload import CONFIGS

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2402_18789_amd.binding as B
    from paper_2402_18789_amd import host as HH
    from gpu_common import TOL, assert_close, to_np
    from test_gpu_train import run_loss


def run_gemm(M, N, K, trans, bias=True, res=True, tile=None, stages=None):
    """tile, stages: the (rows, columns) and LDS ring the product is meant to run on, in one launch over all of K"""
    if tile:
        (rows, cols, width, ranges, ring), = B.flexco_gemm_plan(M, N, K, trans, 0)
        assert (rows, cols) == tile and (width, ranges) == (N, 1) and ring == (stages or ring), (rows, cols, width, ranges, ring)
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N * 3 + K + trans)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    A, W = rnd(M, K), rnd(*((K, N) if trans else (N, K)))
    b, r = rnd(N) if bias else None, rnd(M, N) if res else None
    guard = torch.full((M + 2, N), 7.0, device="cuda", dtype=torch.bfloat16)
    B.flexco_gemm(A, W, guard[:M], b, r, M, N, K, trans, B.FLEXCO_BF16)
    torch.cuda.synchronize()
    Wt = (W if trans else W.t()).double()
    ref, mag = A.double() @ Wt, A.double().abs() @ Wt.abs()
    for t in (b, r):
        if t is not None:
            ref, mag = ref + t.double(), mag + t.double().abs()
    # K + 2 terms added in fp32 in any order, one rounding to bf16
    bound = (K + 2) * 2.0 ** -24 * mag + 2.0 ** -8 * ref.abs() * 1.01 + 1e-30
    assert bool(((guard[:M].double() - ref).abs() <= bound).all())
    assert bool((guard[M:] == 7.0).all())               # nothing past the last row


@pytest.mark.parametrize("tile,M,N,K", [((160, 256), 257, 32776, 4160), ((256, 256), 1000, 28672, 448), ((256, 256), 1000, 28672, 512),
                                        ((256, 192), 511, 24392, 448), ((256, 192), 511, 24392, 512), ((128, 192), 129, 24392, 448)]
                         + [((128, 128), M, N, K) for M, N in ((100, 136), (129, 40), (257, 12296)) for K in (64, 128, 192)])
def test_forward_tiles(tile, M, N, K):
    print(f"forward tile {tile} M={M} N={N} K={K}", flush=True)
    assert tile in [s[:2] for s in B.flexco_gemm_plan(M, N, K, 0, 0)]
    run_gemm(M, N, K, 0)


# 256 x 128 tiles (one launch where the plan has two rounds or leaves CUs idle): odd and even numbers of stages, bias and residual
# or neither, ragged last rows and columns
@pytest.mark.parametrize("bias,res", [(True, True), (False, False)])
@pytest.mark.parametrize("M,N,K,rows", [(1000, 7160, 64 * 25, 256), (1000, 7160, 64 * 20, 256), (1200, 6152, 64 * 25, 256), (769, 8192, 64 * 20, 224)])
def test_forward_tiles_256_by_128(M, N, K, rows, bias, res):
    print(f"forward M={M} N={N} K={K} bias {bias} residual {res}", flush=True)
    run_gemm(M, N, K, 0, bias=bias, res=res, tile=(rows, 128))


# the 256-row kernel's rows are M's own, 160 to 256 in steps of 32: each of them at each width, even and odd numbers of stages
ROWS_THERE_ARE = {(160, 256): [(257, 24592, 512), (257, 24616, 448)], (192, 256): [(321, 24880, 512), (324, 24736, 448)],
                  (224, 256): [(387, 24648, 512), (578, 16360, 448)], (256, 256): [(673, 16368, 512), (449, 24656, 448)],
                  (192, 192): [(131, 32824, 512), (132, 33208, 448)], (224, 192): [(386, 16544, 512), (194, 32864, 448)],
                  (256, 192): [(899, 8216, 512), (681, 10888, 448)], (192, 128): [(129, 29552, 512), (258, 11240, 576)],
                  (224, 128): [(193, 29520, 512), (387, 14752, 448)], (256, 128): [(674, 9840, 512), (900, 7336, 448)]}


@pytest.mark.parametrize("tile,M,N,K", [(tile, *p) for tile, products in ROWS_THERE_ARE.items() for p in products])
def test_forward_tiles_of_the_rows_there_are(tile, M, N, K):
    print(f"forward tile {tile} M={M} N={N} K={K}", flush=True)
    run_gemm(M, N, K, 0, tile=tile)


@pytest.mark.parametrize("rows,M,N,K", [(160, 129, 33352, 512), (160, 130, 32832, 448), (192, 161, 32928, 512), (192, 163, 32848, 448),
                                        (224, 193, 32968, 512), (224, 389, 16400, 448), (256, 674, 10984, 512), (256, 675, 10952, 448)])
def test_input_gradient_tiles_of_the_rows_there_are(rows, M, N, K):
    print(f"input gradient of {rows} rows, M={M} N={N} K={K}", flush=True)
    run_gemm(M, N, K, 1, bias=False, res=False, tile=(rows, 256))


# at most 64 rows: 64 x 128 tiles with a ring of six stages
@pytest.mark.parametrize("K", [64, 192, 384, 448, 704])
@pytest.mark.parametrize("M,N", [(1, 8), (63, 136), (64, 1000)])
def test_forward_tiles_of_few_rows(M, N, K):
    print(f"forward M={M} N={N} K={K}", flush=True)
    run_gemm(M, N, K, 0, tile=(64, 128))


# rows of W a multiple of 4 KB apart: the column tiles of the 64-row form start at stages of their own (its cut form, the cut 128 x 128 one and the
# gated ones: test_layer_products_from_their_own_stage)
@pytest.mark.parametrize("K", [2048, 6144])
@pytest.mark.parametrize("M,N", [(1, 136), (30, 1000), (63, 136), (64, 6152)])
def test_forward_tiles_of_few_rows_from_their_own_stage(M, N, K):
    print(f"forward, spread stages, M={M} N={N} K={K}", flush=True)
    (bm, bn, _, splits, _), = B.flexco_gemm_plan(M, N, K, 0)
    assert (bm, bn, splits) == (64, 128, 1) and N > bn        # a second column tile: only it starts elsewhere
    run_gemm(M, N, K, 0)


# ... and the forms that walk them in order at such a pitch too: one column tile, whole 128 x 128 tiles
@pytest.mark.parametrize("K", [2048, 6144])
@pytest.mark.parametrize("M,N", [(1, 8), (63, 128), (64, 8), (65, 136), (128, 6152)])
def test_forward_tiles_of_few_rows_at_a_pitch_of_4_kb(M, N, K):
    print(f"forward, M={M} N={N} K={K}", flush=True)
    run_gemm(M, N, K, 0)


# (four wavefronts, a ring of two: windows of many rows, and of few where the tiles leave CUs idle)
@pytest.mark.parametrize("K", [64, 128, 192, 448])
@pytest.mark.parametrize("M,N", [(1030, 13832), (258, 136), (64, 40), (33, 264), (1, 8)])
def test_input_gradient_tiles_128(M, N, K):
    print(f"input gradient M={M} N={N} K={K}", flush=True)
    run_gemm(M, N, K, 1, bias=False, res=False, tile=(128, 128), stages=2)


# 128 x 128 tiles by eight wavefronts, two halves of every stage of K: one stage to two rounds of the ring of four, ragged last
# rows and columns (with a rank-r extension: the windows of test_gpu_small_batches and test_gpu_model_iter)
@pytest.mark.parametrize("K", [64 * n for n in (1, 2, 3, 4, 5, 7, 8, 9)])
@pytest.mark.parametrize("M,N", [(1, 32008), (33, 32648), (80, 32136), (127, 128), (129, 4104), (130, 136), (256, 1000)])
def test_input_gradient_tiles_by_eight_wavefronts(M, N, K):
    print(f"input gradient M={M} N={N} K={K}", flush=True)
    run_gemm(M, N, K, 1, bias=False, res=False, tile=(128, 128), stages=4)


# ... in ranges that differ by a stage (131 stages in 4, 67 in 7 and more), which the loss head's scratch is for
@pytest.mark.parametrize("n,H,V", [(200, 4096, 64 * 131), (100, 520, 64 * 67), (1, 4096, 64 * 67), (8, 4104, 64 * 67), (33, 264, 64 * 67)])
def test_input_gradient_by_eight_wavefronts_in_ranges(n, H, V):
    (rows, cols, _, ranges, ring), = B.flexco_gemm_plan(n, H, V, 1, 16 * n * H)
    print(f"loss head n={n} H={H} V={V}: {ranges} ranges", flush=True)
    assert (rows, cols, ring) == (128, 128, 4) and (V // 64) % ranges != 0
    run_loss("bf16", n, H, V, seed=5)


@pytest.mark.parametrize("M,N,K", [(1023, 13832, 5120), (1000, 13816, 5184)])
def test_input_gradient_tiles_256(M, N, K):
    print(f"input gradient M={M} N={N} K={K}", flush=True)
    assert B.flexco_gemm_plan(M, N, K, 1, 0) == [(256, 256, N, 1, 2)]
    run_gemm(M, N, K, 1, bias=False, res=False)


# the loss head brings split-K scratch of 16 n H floats: its input gradient contracts over V in V / 64 stages
@pytest.mark.parametrize("n,H,V", [(385, 4104, 64 * 43), (257, 4096, 64 * 131)])
def test_input_gradient_in_unequal_ranges(n, H, V):
    (rows, cols, _, r, _), = B.flexco_gemm_plan(n, H, V, 1, 16 * n * H)
    print(f"loss head n={n} H={H} V={V}: {r} ranges", flush=True)
    assert rows > 128 and cols == 256 and r > 1 and (V // 64) % r != 0
    run_loss("bf16", n, H, V, seed=3)


# rows of logits that a block holds in registers: 4 and 8, 9 and 16, 17 and 19 pieces of 8192 (the last ragged or whole),
# and the first lengths and the first number of rows past them
@pytest.mark.parametrize("n,V", [(5, V) for V in (16392, 24576, 24584, 65536, 65544, 131072, 131080, 155648, 155656)]
                         + [(256, 24584), (257, 24584), (257, 65544)])
def test_loss_rows(n, V):
    print(f"loss head n={n} V={V}", flush=True)
    run_loss("bf16", n, 256, V, seed=4, ignore=(1, 4))


# gate and up rows of one weight matrix of more than 4 GiB, on the 64-, 128- and 256-row tiles.  One-token sequences: the
# attention output of a token is its value row.
def test_gated_projection_of_weights_past_4_gib():
    H, F, nq, nkv, d = 1024, 64 * 16448, 8, 2, 128
    assert 2 * F * H * 2 > 1 << 32
    cfg = CONFIGS["c2_llama8b_layer"].with_(name="wide_ffn", hidden=H, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=F, lora_targets=())
    g = torch.Generator(device="cuda").manual_seed(31)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    wqkv, wo, wgu, wd = (rnd(*s).mul_(0.02) for s in ((cfg.q_dim + 2 * cfg.kv_dim, H), (H, cfg.q_dim), (2 * F, H), (H, F)))
    g1, g2 = (1 + 0.02 * rnd(H).float()).bfloat16(), (1 + 0.02 * rnd(H).float()).bfloat16()
    w = B.BaseWeights(*[t.data_ptr() if t is not None else None for t in (wqkv, None, wo, wgu, wd, g1, g2)])
    c = HH.c_cfg(cfg)
    norm = lambda x, gain: x * torch.rsqrt(x.square().mean(-1, keepdim=True) + cfg.rms_eps) * gain.double()  # noqa: E731
    for T in (8, 130, 520):
        print(f"gated projection, {wgu.numel() * 2 / 2 ** 30:.2f} GiB of weights, {T} tokens, {B.flexco_gemm_plan(T, 2 * F, H, 0, 0)}", flush=True)
        reqs = [SimpleNamespace(kind=B.FLEXCO_DECODE, seq_id=i, start_pos=0, n_new=1, adapter=-1) for i in range(T)]
        pool = HH.DevicePool(cfg, T + 1)
        db = HH.DeviceBatch(cfg, reqs, [[i] for i in range(T)], T + 1)
        ws = HH.Workspace(c, T, db.host_maps.n_parts)
        x, y = rnd(T, H), torch.empty(T, H, device="cuda", dtype=torch.bfloat16)
        B.flexco_layer_forward(c, w, None, db.maps, x, y, pool.c, None, ws.ptr, ws.bytes)
        torch.cuda.synchronize()
        v = (norm(x.double(), g1) @ wqkv[cfg.q_dim + cfg.kv_dim:].double().t()).view(T, nkv, 1, d).expand(T, nkv, nq // nkv, d).reshape(T, -1)
        ref = x.double() + v @ wo.double().t()
        h = norm(ref, g2)
        for f0 in range(0, F, 1 << 16):
            f1 = min(F, f0 + (1 << 16))
            gate, up = h @ wgu[f0:f1].double().t(), h @ wgu[F + f0:F + f1].double().t()
            ref = ref + (gate * torch.sigmoid(gate) * up) @ wd[:, f0:f1].double().t()
        assert_close(f"y of {T} tokens", to_np(y), to_np(ref), TOL["bf16"])
        del ws
