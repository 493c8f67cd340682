"""What the built gfx950 code of the LDS-staged kernels does, on every path of it (no GPU): a buffer is handed to new loads
only when its readers have their data, and the operands of a matrix product are there when it reads them."""
import os
import re

import pytest

import gfx_code
import paper_2402_18789_amd.binding as B

pytestmark = [pytest.mark.skipif(B.HOST_ONLY, reason="needs the whole library, this is a host-only build"),
              pytest.mark.skipif(not os.path.exists(gfx_code.OBJDUMP), reason="needs llvm-objdump")]


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    return gfx_code.kernels(B.LIB_PATH, str(tmp_path_factory.mktemp("code")))


def barriers_of(code, name):
    """{kernel's template arguments: reads on their way at each of its barriers}"""
    out = {}
    for mangled, ins in code.items():
        m = re.search(r"\d%sI((?:L[ib]\d+E)+)E" % name, mangled)
        if m and not mangled.endswith(".kd"):
            out[tuple(int(v) for v in re.findall(r"L[ib](\d+)E", m.group(1)))] = gfx_code.lds_reads_at_barriers(ins)
    assert out, name
    return out


# Rings of two stages (the input-gradient form, and the forward form built with two): the buffer freed at a stage's barrier
# is the stage's own, so no wavefront may have a read on its way there.  Rings of four and six free the stage before:
# reads issued since the last barrier may be on their way, older ones may not.
# (template arguments: rows and columns of the tile, transposed, gated, stages, stages walked round from one of the tile's own)
def test_projection_rings_are_not_overwritten_under_a_read(code):
    two, rotated = 0, set()
    for args, reads in barriers_of(code, "gemm_bf16_kernel").items():
        bm, _, trans, glu, stages, spread, *_ = args
        assert len(reads) > 2
        assert all(old == 0 for _, old in reads), (args, reads)
        if trans or stages == 2:
            two += 1
            assert all(young == 0 for young, _ in reads), (args, reads)
        if spread:
            rotated.add((bm, glu))
    assert two == 3
    assert rotated == {(64, 0), (64, 1), (128, 0), (128, 1)}
    for args, reads in barriers_of(code, "gemm_bf16_quad_kernel").items():
        assert all(r == (0, 0) for r in reads), (args, reads)


# The input-gradient kernel of eight wavefronts frees a stage's own buffer at its barrier, too.
def test_ring_of_the_eight_wavefront_kernel_is_not_overwritten_under_a_read(code):
    (ins,) = [i for n, i in code.items() if "gemm_bf16_pair_kernel" in n and not n.endswith(".kd")]
    reads = gfx_code.lds_reads_at_barriers(ins)
    assert len(reads) > 7 and all(r == (0, 0) for r in reads), reads


# Attention: the buffer freed at a step's barrier is the one the step before has read (backward: two buffer sets; chunk
# items: rings of three and four, whose V is read in the step that ends at the barrier).
@pytest.mark.parametrize("name", ["attn_bwd_dq_mfma_kernel", "attn_bwd_dkv_mfma_kernel", "attn_fwd_chunk_kernel"])
def test_attention_buffers_are_not_overwritten_under_a_read(code, name):
    for args, reads in barriers_of(code, name).items():
        assert len(reads) > 2
        assert all(r == (0, 0) for r in reads), (args, reads)


# The projections' products are inline assembly, whose operands the compiler's hazard handling does not cover: none may be
# written by a vector instruction in the two wait states before.
def test_operands_of_the_products_are_not_written_just_before(code):
    products = 0
    for name, ins in code.items():
        products += sum(op.startswith("v_mfma") for _, op, _ in ins)
        assert gfx_code.operands_written_too_late(ins, 2) == [], name
    assert products > 1000


# The type-generic attention backward: the loops that add a run of keys' (pairs') rows hold several of them, the lane reads of all
# up front - a loop with lane reads and a remainder is one the compiler leaves as it is, one row's round trip after the other.
# dQ: 8 keys of three lane reads; dK / dV: 4, 8 or 16 pairs of four.
@pytest.mark.parametrize("name,at_least", [("attn_bwd_dq_generic_kernel", 8 * 3), ("attn_bwd_dkv_generic_kernel", 4 * 4),
                                           ("attn_bwd_few_generic_kernel", 8 * 3 + 4 * 4)])
def test_rows_of_the_generic_attention_backward_are_fetched_together(code, name, at_least):
    forms = {n: sum(op.startswith("v_readlane") for _, op, _ in ins) for n, ins in code.items() if name in n and not n.endswith(".kd")}
    assert len(forms) >= 6 and all(k >= at_least for k in forms.values()), forms


# ... and dK / dV of few key blocks has its form with 16 / 8 / 4 pairs at a time whether or not dQ is in the same launch
@pytest.mark.parametrize("du,pairs", [(1, 16), (2, 8), (4, 4)])
def test_key_value_gradients_of_few_blocks_fetch_more_rows_at_a_time(code, du, pairs):
    forms = [sum(op.startswith("v_readlane") for _, op, _ in ins) for n, ins in code.items()
             if "attn_bwd_dkv_generic_kernel" in n and "Li%dELb1ELb1E" % du in n and not n.endswith(".kd")]
    assert len(forms) == 2 and all(k >= pairs * 4 for k in forms), forms


# The attention's steps over pages that every row sees whole, lists of chunks alone: what a step does for its scores is what bounds it
# so no select or compare beside those of the running maximum
def test_attention_steps_of_chunks_alone_select_once(code):
    (ins,) = [i for n, i in code.items() if "attn_fwd_chunk_kernelILi3E" in n and not n.endswith(".kd")]
    at = {i[0]: k for k, i in enumerate(ins)}
    loops = []
    for k, (addr, op, args) in enumerate(ins):
        if op.startswith("s_cbranch") or op == "s_branch":
            off = int(args[0], 0) & 0xffff
            to = at[addr + 4 + 4 * (off - 0x10000 if off & 0x8000 else off)]
            body = [o for _, o, _ in ins[to:k + 1]]
            if to < k and sum(o.startswith("v_mfma") for o in body) == 6 * 16:
                loops.append((len(body), sum(o.startswith("v_cndmask") for o in body), sum(o.startswith("v_cmp") for o in body)))
    assert loops and min(loops)[1:] == (6, 6), loops
