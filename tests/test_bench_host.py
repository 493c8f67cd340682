"""bench.py's account of the forward projections' launches (host arithmetic, no GPU): a second launch only where a product
is cut over K with the scratch the layer has and nothing else adds its sums."""
import pytest

import bench
import paper_2402_18789_amd.binding as B
from workload import CONFIGS

pytestmark = pytest.mark.skipif(B.HOST_ONLY, reason="needs the whole library, this is a host-only build")

C2, C4, C5 = (CONFIGS[n] for n in ("c2_llama8b_layer", "c4_qwen14b_full", "c5_qwen32b_full"))


def launches(cfg, T, **kw):
    return [n for _, _, n in bench.forward_launches(B, cfg, T, **kw)]


def test_launches_of_the_benchmark_step():
    assert launches(C2, 1024) == [1, 1, 2, 2]         # gate/up in two tile shapes, down in ranges and their sum


def test_sums_left_to_the_next_kernel_are_no_launch():
    assert B.flexco_gemm_k_ranges(280, C2.hidden, C2.q_dim, 0, 280 * C2.ffn) > 1
    assert launches(C2, 280)[1] == 1                  # o: the norm adds them
    qkv = (C5.q_dim + 2 * C5.kv_dim, C5.hidden)
    assert B.flexco_gemm_k_ranges(600, *qkv, 0, 600 * C5.ffn) > 1
    assert launches(C5, 600)[0] == 1 and launches(C5, 600, use_ia3=True)[0] == 2      # the rotation, unless (IA)^3 comes between
    assert launches(C2, 16)[:2] == [1, 1] and launches(C2, 16)[3] == 2


def down_scratch(cfg, T):
    """floats: the gate/up buffer and, in front of it, the bf16 rows of h, qkv and the attention output"""
    return T * cfg.ffn + T * (cfg.hidden + cfg.q_dim + 2 * cfg.kv_dim + cfg.q_dim) // 2


def test_cuts_are_asked_for_with_the_layers_own_scratch():
    # tokens at which more scratch than the layer's would cut a product that the layer leaves whole
    more = [T for T in range(257, 2049) if B.flexco_gemm_k_ranges(T, C4.hidden, C4.hidden, 0, 1 << 30) > 1
            and B.flexco_gemm_k_ranges(T, C4.hidden, C4.hidden, 0, T * C4.ffn) <= 1]
    assert all(launches(C4, T)[1] == len(B.flexco_gemm_plan(T, C4.hidden, C4.q_dim, 0, T * C4.ffn)) for T in more)
    # tokens at which the gate/up buffer alone would leave the down product whole, and the layer cuts it
    cut = [T for T in range(257, 2049) if B.flexco_gemm_k_ranges(T, C4.hidden, C4.ffn, 0, down_scratch(C4, T)) > 1
           and B.flexco_gemm_k_ranges(T, C4.hidden, C4.ffn, 0, T * C4.ffn) <= 1]
    assert cut and all(launches(C4, T)[3] == 2 for T in cut)
    # ... and at which more than all of it would
    more = [T for T in range(257, 4097) for cfg in (C2, C4, C5) if B.flexco_gemm_k_ranges(T, cfg.hidden, cfg.ffn, 0, 1 << 40) > 1
            and B.flexco_gemm_k_ranges(T, cfg.hidden, cfg.ffn, 0, down_scratch(cfg, T)) <= 1
            and launches(cfg, T)[3] != len(B.flexco_gemm_plan(T, cfg.hidden, cfg.ffn, 0, down_scratch(cfg, T)))]
    assert not more


# the counted HBM bytes of a kernel are printed under that kernel's name only
def test_traffic_is_of_the_kernel_it_is_printed_for(monkeypatch):
    for name in ("attn_fwd", "gemm_fwd"):
        assert bench.measured_traffic(name) > 1e6
        assert bench.roofline_entry(name, 1.0, 1, {})["traffic"] == bench.measured_traffic(name)
        monkeypatch.setitem(bench.KERNEL_NAMES, name, "another_kernel")
        assert bench.measured_traffic(name) is None
