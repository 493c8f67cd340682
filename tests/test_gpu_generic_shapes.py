"""The fp32 matrix-core projection and the type-generic attention kernels at the sizes where their tiles, remainders and
vector accesses can go wrong (run with -m gpu on an MI355X)."""
import numpy as np
import pytest
import torch

from workload import gen, CONFIGS

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2402_18789_amd.binding as B
    from paper_2402_18789_amd import host as HH
    from oracle import ops as OO
    from gpu_common import Case, to_np, TOL, assert_close
    from test_gpu_parity import attention_case

C1 = CONFIGS["c1_tiny_f32"]
ODD_F32 = C1.with_(name="odd_f32", n_q_heads=6, n_kv_heads=2, head_dim=20, page_size=5)          # V page rows: no whole 16 bytes
WIDE_BF16 = C1.with_(name="wide_bf16", dtype="bf16", n_q_heads=4, n_kv_heads=2, head_dim=72, page_size=24)
D256_BF16 = C1.with_(name="d256_bf16", dtype="bf16", n_q_heads=4, n_kv_heads=2, head_dim=256)


# one tile; ragged tiles; K not a multiple of a step of 16; more steps than wavefronts x loads in flight; more than 1024 tiles of
# 16 x 16 (32 x 32 tiles), ragged; K without groups of four (the element-wise kernel)
@pytest.mark.parametrize("M,N,K", [(1, 1, 4), (16, 16, 16), (17, 33, 20), (68, 256, 688), (15, 40, 1000), (300, 260, 36),
                                   (530, 1036, 164), (33, 20, 30)])
@pytest.mark.parametrize("trans", [0, 1])
def test_gemm_f32(M, N, K, trans):
    print(f"gemm f32 M={M} N={N} K={K} trans={trans}", flush=True)
    g = gen.rng(9, "gemm_f32", M, N, K, trans)
    A, bias, res = (g.standard_normal(s, dtype=np.float32) for s in ((M, K), (N,), (M, N)))
    W = g.standard_normal((K, N) if trans else (N, K), dtype=np.float32)
    W64 = W.astype(np.float64) if trans else W.T.astype(np.float64)
    ref = A.astype(np.float64) @ W64 + bias + res
    # a sum of K + 2 products and terms in fp32, in any order: at most (K + 2) roundings of the terms' absolute sum
    bound = (K + 2) * 2.0 ** -24 * (np.abs(A).astype(np.float64) @ np.abs(W64) + np.abs(bias) + np.abs(res))
    dev = [torch.from_numpy(a).cuda() for a in (A, W, bias, res)]
    guard = torch.full((M + 2, N), 7.0, device="cuda")
    B.flexco_gemm(dev[0], dev[1], guard[:M], dev[2], dev[3], M, N, K, trans, B.FLEXCO_F32)
    torch.cuda.synchronize()
    got = to_np(guard)
    assert np.all(np.abs(got[:M] - ref) <= bound)
    assert np.all(got[M:] == 7.0)               # nothing past the last row


@pytest.mark.parametrize("cfg,split", [(ODD_F32, 0), (ODD_F32, 2), (WIDE_BF16, 0), (WIDE_BF16, 2), (D256_BF16, 4),
                                       (C1, 64)])           # 1024 keys per split: four wavefronts per block
def test_generic_attention_forward(cfg, split):
    print(f"attention forward {cfg.name} split={split}", flush=True)
    batch = gen.mixed_batch(cfg.page_size, 4, decode_ctx=(1, 7, 1100, 64), prefill=[(0, 33, 33), (21, 18, 39)], finetune=[(50, 21, 71)])
    out, a_o, lse, lse_o = attention_case(cfg, batch, split)
    assert_close("attention out", out, a_o, TOL[cfg.dtype])
    assert float(np.max(np.abs(lse - lse_o))) <= (1e-4 if cfg.dtype == "f32" else 2e-2)


@pytest.mark.parametrize("cfg,win_start,win_len", [(ODD_F32, 0, 1), (ODD_F32, 61, 68), (WIDE_BF16, 40, 37), (C1, 130, 21),
                                                   (D256_BF16, 70, 33)])
def test_generic_attention_backward(cfg, win_start, win_len):
    print(f"attention backward {cfg.name} [{win_start}, +{win_len})", flush=True)
    l = win_start + win_len
    n_pages = -(-l // cfg.page_size)
    g = gen.rng(12, "generic_bwd", cfg.name, win_start, win_len)
    pages = (g.permutation(n_pages + 3)[:n_pages] + 1).astype(np.int32)
    rnd = lambda *s: gen.storage_round(cfg, g.standard_normal(s, dtype=np.float32))  # noqa: E731
    K, V, q, do = rnd(l, cfg.kv_dim), rnd(l, cfg.kv_dim), rnd(win_len, cfg.q_dim), rnd(win_len, cfg.q_dim)
    pos = np.arange(win_start, l)
    f64 = lambda a: a.astype(np.float64)  # noqa: E731
    o, lse = OO.attention(f64(q), pos, f64(K), f64(V), cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim)
    dq_o, dk_o, dv_o = OO.attention_bwd(f64(q), pos, f64(K), f64(V), cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, f64(do))
    pool = HH.DevicePool(cfg, n_pages + 4)
    pool.write_rows(pages, K, V)
    dt = HH.TORCH_DTYPE[cfg.dtype]
    dev = lambda a, t=dt: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", t)  # noqa: E731
    q_d, o_d, do_d, lse_d = dev(q), dev(o), dev(do), dev(lse, torch.float32)
    dq, dk, dv = torch.empty_like(q_d), torch.ones(l, cfg.kv_dim, device="cuda"), torch.ones(l, cfg.kv_dim, device="cuda")
    ws = torch.empty(win_len * cfg.n_q_heads * 4 + 64, dtype=torch.uint8, device="cuda")
    B.flexco_attention_window_bwd(HH.c_cfg(cfg), pool.c, dev(pages, torch.int32), n_pages, win_start, win_len, q_d, o_d, lse_d, do_d,
                                  dq, dk, dv, ws, ws.numel())
    torch.cuda.synchronize()
    assert_close("dq", to_np(dq), dq_o, TOL[cfg.dtype])
    assert_close("dk", to_np(dk) - 1.0, dk_o, TOL[cfg.dtype])
    assert_close("dv", to_np(dv) - 1.0, dv_o, TOL[cfg.dtype])


# the forms of the backward kernels: one, two and four channels per lane; accumulator rows x kv heads up to 1024 and above it; Q and dO
# off their 16-byte alignment (element by element).  Forward: contexts around the 64 keys that are fetched ahead.
D64_F32, D128_F32, D256_F32 = (C1.with_(name="d%d_f32" % d, n_q_heads=4, n_kv_heads=2, head_dim=d) for d in (64, 128, 256))


@pytest.mark.parametrize("cfg,win_start,win_len,shift", [(D64_F32, 0, 64, 0), (D64_F32, 0, 65, 1), (D64_F32, 500, 30, 0), (D128_F32, 3, 50, 0),
                                                         (D128_F32, 505, 40, 0), (D256_F32, 20, 44, 1), (D256_F32, 490, 40, 0),
                                                         (D64_F32, 511, 1, 0), (D128_F32, 473, 40, 0), (D256_F32, 0, 1, 0),
                                                         (D256_F32, 20, 45, 0), (D256_F32, 472, 40, 0)])
def test_generic_attention_backward_forms(cfg, win_start, win_len, shift):
    print(f"attention backward forms {cfg.name} [{win_start}, +{win_len}) shift={shift}", flush=True)
    l = win_start + win_len
    n_pages = -(-l // cfg.page_size)
    g = gen.rng(13, "generic_bwd_forms", cfg.name, win_start, win_len)
    pages = (g.permutation(n_pages + 3)[:n_pages] + 1).astype(np.int32)
    rnd = lambda *s: g.standard_normal(s, dtype=np.float32)  # noqa: E731
    K, V, q, do = rnd(l, cfg.kv_dim), rnd(l, cfg.kv_dim), rnd(win_len, cfg.q_dim), rnd(win_len, cfg.q_dim)
    pos = np.arange(win_start, l)
    f64 = lambda a: a.astype(np.float64)  # noqa: E731
    o, lse = OO.attention(f64(q), pos, f64(K), f64(V), cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim)
    dq_o, dk_o, dv_o = OO.attention_bwd(f64(q), pos, f64(K), f64(V), cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, f64(do))
    pool = HH.DevicePool(cfg, n_pages + 4)
    pool.write_rows(pages, K, V)

    def dev(a, off=0):                       # off elements past an aligned address
        t = torch.zeros(a.size + off, device="cuda")
        t[off:] = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).flatten().cuda()
        return t[off:].view(a.shape)
    q_d, o_d, do_d, lse_d = dev(q, shift), dev(o), dev(do, shift), dev(lse)
    dq, dk, dv = torch.empty_like(q_d), torch.ones(l, cfg.kv_dim, device="cuda"), torch.ones(l, cfg.kv_dim, device="cuda")
    ws = torch.empty(win_len * cfg.n_q_heads * 4 + 64, dtype=torch.uint8, device="cuda")
    B.flexco_attention_window_bwd(HH.c_cfg(cfg), pool.c, torch.from_numpy(pages).cuda(), n_pages, win_start, win_len, q_d, o_d, lse_d, do_d,
                                  dq, dk, dv, ws, ws.numel())
    torch.cuda.synchronize()
    for name, got, ref in (("dq", to_np(dq), dq_o), ("dk", to_np(dk) - 1.0, dk_o), ("dv", to_np(dv) - 1.0, dv_o)):
        assert_close(name, got, ref, TOL["f32"])


def test_generic_attention_backward_over_the_output_rows():
    """dQ written over the rows of out (each block reads its own row before): as into a buffer of its own."""
    print("attention backward over the output rows", flush=True)
    cfg, win_start, win_len = D64_F32, 32, 32
    l = win_start + win_len
    n_pages = -(-l // cfg.page_size)
    g = gen.rng(14, "generic_bwd_over_out")
    dev = lambda *s: torch.from_numpy(g.standard_normal(s, dtype=np.float32)).cuda()  # noqa: E731
    pool = HH.DevicePool(cfg, n_pages + 1)
    pool.write_rows(np.arange(n_pages, dtype=np.int32), to_np(dev(l, cfg.kv_dim)), to_np(dev(l, cfg.kv_dim)))
    q, do, o, lse = dev(win_len, cfg.q_dim), dev(win_len, cfg.q_dim), dev(win_len, cfg.q_dim), 5.0 + dev(win_len, cfg.n_q_heads)
    got = []
    for over in (False, True):
        out = o.clone()
        dq = out if over else torch.empty_like(q)
        dk, dv = torch.zeros(l, cfg.kv_dim, device="cuda"), torch.zeros(l, cfg.kv_dim, device="cuda")
        ws = torch.empty(win_len * cfg.n_q_heads * 4 + 64, dtype=torch.uint8, device="cuda")
        B.flexco_attention_window_bwd(HH.c_cfg(cfg), pool.c, torch.arange(n_pages, dtype=torch.int32, device="cuda"), n_pages, win_start,
                                      win_len, q, out, lse, do, dq, dk, dv, ws, ws.numel())
        torch.cuda.synchronize()
        got.append((to_np(dq), to_np(dk), to_np(dv)))
    for a, b in zip(*got):
        assert np.max(np.abs(a - b)) <= 1e-5 * np.max(np.abs(a))          # (delta's sum in another order: a few roundings of its terms)


# One launch for dQ, dK and dV reads the rows of out once more per key: not where that costs more than a second launch does, which is
# what dQ over out takes.  (fp32, long windows behind long prefixes, many heads to a kv head: 1.34 and 1.27 with one launch.)
@pytest.mark.parametrize("d,heads,win_start,win_len", [(256, 16, 512, 256), (128, 32, 512, 256)])
def test_generic_attention_backward_in_one_launch_is_no_slower_than_in_two(d, heads, win_start, win_len):
    cfg = C1.with_(name="wide_group", n_q_heads=heads, n_kv_heads=1, head_dim=d)
    l = win_start + win_len
    n_pages = -(-l // cfg.page_size)
    pool = HH.DevicePool(cfg, n_pages + 1)
    pool.fill_random(1)
    q, do, o = (torch.randn(win_len, cfg.q_dim, device="cuda") for _ in range(3))
    lse, dk, dv = torch.full((win_len, heads), 30.0, device="cuda"), torch.zeros(l, d, device="cuda"), torch.zeros(l, d, device="cuda")
    pages, ws = torch.arange(n_pages, dtype=torch.int32, device="cuda"), torch.empty(win_len * heads * 4 + 64, dtype=torch.uint8, device="cuda")
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]

    def ms(dq):
        ev[0].record()
        for _ in range(4):
            B.flexco_attention_window_bwd(HH.c_cfg(cfg), pool.c, pages, n_pages, win_start, win_len, q, o, lse, do, dq, dk, dv, ws, ws.numel())
        ev[1].record()
        torch.cuda.synchronize()
        return ev[0].elapsed_time(ev[1]) / 4
    own = torch.empty_like(q)
    ms(own), ms(o)
    both = [(ms(own), ms(o)) for _ in range(5)]
    one, two = min(b[0] for b in both), min(b[1] for b in both)
    print(f"attention backward, {heads} heads of {d}, [{win_start}, +{win_len}): {one:.3f} ms, over out {two:.3f}", flush=True)
    assert one <= 1.12 * two


# Rows of one kept activation off their 16-byte alignment: the norm that is computed again from them goes element by element, the
# others as ever - gate's gradient reads the second norm's rows only and keeps its bits, q's the first norm's.
def test_rematerialised_rows_of_different_alignment():
    print("layer backward, saved_x off its alignment", flush=True)
    cfg = C1.with_(name="remat_f32", hidden=1024, lora_targets=("q", "gate", "down"))
    case = Case(cfg, gen.mixed_batch(cfg.page_size, 3, finetune=[(0, 40, 40)]), seed=3)
    (r,) = case.batch.requests
    case.forward(case.batch, gen.layer_input(cfg, 3, 40), oracle=False)
    st, pages = case.d_ft[r.seq_id], torch.from_numpy(case.dpages(case.batch.seq_pages[r.seq_id])).cuda()
    dY = torch.from_numpy(gen.layer_input(cfg, 4, 40, tag="dy")).cuda()
    ws = HH.Workspace(case.dev.c, 0, 0, 40, 40)
    off = torch.zeros(st.x.numel() + 1, device="cuda")[1:].copy_(st.x.flatten())
    assert st.x.data_ptr() % 16 == 0 and off.data_ptr() % 16 == 4
    got = []
    for rows in (st.x, off):
        st.c.saved_x = rows.data_ptr()
        case.dev.zero_grads()
        st.zero_accum()
        B.flexco_lora_bwd(case.dev.c, case.dev.w, case.dev.lora, case.d_pool.c, pages, len(pages), st.c, 0, 40, dY, None, ws.ptr, ws.bytes)
        torch.cuda.synchronize()
        got.append({t: case.dev.dA[t].clone() for t in cfg.lora_targets})
    assert torch.equal(got[0]["gate"], got[1]["gate"]) and torch.equal(got[0]["down"], got[1]["down"])
    assert_close("dA q", to_np(got[1]["q"]), to_np(got[0]["q"]), 1e-5)           # (the row's squares in another order)


@pytest.mark.parametrize("cfg", [D64_F32, D128_F32, ODD_F32, WIDE_BF16])
def test_generic_attention_forward_short_runs(cfg):
    print(f"attention forward short runs {cfg.name}", flush=True)
    batch = gen.mixed_batch(cfg.page_size, 6, decode_ctx=(1, 2, 3, 15, 16, 17, 47, 48, 62, 63, 64, 65), prefill=[(0, 64, 64), (30, 35, 65)], finetune=[(1, 63, 64)])
    for split in (0, 2):
        out, a_o, lse, lse_o = attention_case(cfg, batch, split)
        assert_close("attention out", out, a_o, TOL[cfg.dtype])
        assert float(np.max(np.abs(lse - lse_o))) <= (1e-4 if cfg.dtype == "f32" else 2e-2)


# the rows that the backward kernels fetch together: the last group of them full, of one and of all but one; one, two and four channels per lane, the
# last of them partly past head_dim
@pytest.mark.parametrize("win_start,win_len", [(0, 1), (0, 8), (7, 9), (40, 25), (63, 2), (260, 33)])
@pytest.mark.parametrize("head_dim,dtype", [(40, "f32"), (100, "f32"), (136, "f32"), (200, "bf16"), (256, "bf16")])
def test_generic_attention_backward_groups(head_dim, dtype, win_start, win_len):
    test_generic_attention_backward(C1.with_(name="d%d_%s" % (head_dim, dtype), dtype=dtype, n_q_heads=6, n_kv_heads=2, head_dim=head_dim),
                                    win_start, win_len)


# the forms of the forward kernel: every context of at most 64 keys and 64 channels (V fetched beside K), in one and in several ranges of
# keys; nothing but single tokens (one tile per item, as many blocks as a group of heads needs)
GROUP6_F32 = C1.with_(name="g6_f32", n_q_heads=12, n_kv_heads=2, head_dim=64)


@pytest.mark.parametrize("split", [0, 2])
@pytest.mark.parametrize("cfg", [C1, D64_F32, GROUP6_F32, ODD_F32, D128_F32])
@pytest.mark.parametrize("kind", ["short", "singles", "short singles"])
def test_generic_attention_forward_forms(cfg, split, kind):
    print(f"attention forward forms {cfg.name} {kind} split={split}", flush=True)
    ctx = (1, 2, 15, 16, 17, 31, 33, 48, 62, 63, 64) if "short" in kind else (1, 5, 63, 64, 65, 66, 127, 128, 129, 500)
    chunks = {} if "singles" in kind else dict(prefill=[(0, 17, 17), (20, 44, 64)], finetune=[(1, 63, 64)])
    out, a_o, lse, lse_o = attention_case(cfg, gen.mixed_batch(cfg.page_size, 8, decode_ctx=ctx, **chunks), split)
    assert_close("attention out", out, a_o, TOL[cfg.dtype])
    assert float(np.max(np.abs(lse - lse_o))) <= 1e-4
