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
    from gpu_common import to_np, TOL, assert_close
    from test_gpu_parity import attention_case

C1 = CONFIGS["c1_tiny_f32"]
ODD_F32 = C1.with_(name="odd_f32", n_q_heads=6, n_kv_heads=2, head_dim=20, page_size=5)          # V page rows: no whole 16 bytes
WIDE_BF16 = C1.with_(name="wide_bf16", dtype="bf16", n_q_heads=4, n_kv_heads=2, head_dim=72, page_size=24)


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
