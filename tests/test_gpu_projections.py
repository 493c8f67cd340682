"""The bf16 projections' tile kernels at the sizes where they can go wrong: each tile shape with ragged last rows and
columns, one, two and three 64-wide stages of K, K in unequal ranges (run with -m gpu on an MI355X)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2402_18789_amd.binding as B
    from test_gpu_train import run_loss


def run_gemm(M, N, K, trans, bias=True, res=True):
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


@pytest.mark.parametrize("tile,M,N,K", [((256, 256), 257, 32776, 4160), ((256, 256), 1000, 28672, 448), ((256, 256), 1000, 28672, 512),
                                        ((256, 192), 511, 24392, 448), ((256, 192), 511, 24392, 512), ((128, 192), 129, 24392, 448)]
                         + [((128, 128), M, N, K) for M, N in ((100, 136), (129, 40), (257, 12296)) for K in (64, 128, 192)])
def test_forward_tiles(tile, M, N, K):
    print(f"forward tile {tile} M={M} N={N} K={K}", flush=True)
    assert tile in [s[:2] for s in B.flexco_gemm_plan(M, N, K, 0, 0)]
    run_gemm(M, N, K, 0)


# at most 64 rows: 64 x 128 tiles with a ring of six stages
@pytest.mark.parametrize("K", [64, 192, 384, 448, 704])
@pytest.mark.parametrize("M,N", [(1, 8), (63, 136), (64, 1000)])
def test_forward_tiles_of_few_rows(M, N, K):
    print(f"forward M={M} N={N} K={K}", flush=True)
    run_gemm(M, N, K, 0)


@pytest.mark.parametrize("K", [64, 128, 192, 448])
@pytest.mark.parametrize("M,N", [(1030, 13832), (130, 136), (64, 40)])
def test_input_gradient_tiles_128(M, N, K):
    print(f"input gradient M={M} N={N} K={K}", flush=True)
    run_gemm(M, N, K, 1, bias=False, res=False)


@pytest.mark.parametrize("M,N,K", [(1023, 13832, 5120), (1000, 13816, 5184)])
def test_input_gradient_tiles_256(M, N, K):
    print(f"input gradient M={M} N={N} K={K}", flush=True)
    assert B.flexco_gemm_k_ranges(M, N, K, 1, 0) == 1 or B.flexco_gemm_plan(M, N, K, 1, 0)[0][0] == 256
    run_gemm(M, N, K, 1, bias=False, res=False)


# the loss head brings split-K scratch of 16 n H floats: its input gradient contracts over V in V / 64 stages
@pytest.mark.parametrize("n,H,V", [(300, 520, 64 * 67), (257, 4096, 64 * 131)])
def test_input_gradient_in_unequal_ranges(n, H, V):
    r = B.flexco_gemm_k_ranges(n, H, V, 1, 16 * n * H)
    print(f"loss head n={n} H={H} V={V}: {r} ranges", flush=True)
    assert r > 1 and (V // 64) % r != 0
    run_loss("bf16", n, H, V, seed=3)


# rows of logits that a block holds in registers: 4 and 8, 9 and 16, 17 and 19 pieces of 8192 (the last ragged or whole),
# and the first lengths and the first number of rows past them
@pytest.mark.parametrize("n,V", [(5, V) for V in (16392, 24576, 24584, 65536, 65544, 131072, 131080, 155648, 155656)]
                         + [(256, 24584), (257, 24584), (257, 65544)])
def test_loss_rows(n, V):
    print(f"loss head n={n} V={V}", flush=True)
    run_loss("bf16", n, 256, V, seed=4, ignore=(1, 4))
