"""The choices of the attention's work list (no GPU): which kernel takes it, how many key splits as one, and in which order its
items run then."""
import collections
import math

import numpy as np
import pytest

import paper_2402_18789_amd.binding as B
from attn_plan import attention_plan, lib
from workload.configs import KIND_DECODE, KIND_PREFILL

N_HEADS = 32


def build_maps(nkv, requests, split=0):
    """requests: [(kind, first position, new tokens)]"""
    pages = [-(-(start + n) // 16) for _, start, n in requests]
    first = np.concatenate(([0], np.cumsum(pages)))
    desc, keep = B.make_batch_desc([k for k, _, _ in requests], [s for _, s, _ in requests], [n for _, _, n in requests], [-1] * len(requests),
                                   [np.arange(a, b, dtype=np.int32) for a, b in zip(first, first[1:])])
    maps, blob = B.flexco_build_maps(desc, 16, int(first[-1]), N_HEADS, nkv, split)
    return maps, blob, keep


def decode(n, lo, hi, median=0):
    """n decode requests, contexts at the quantiles of lo..hi, or of a log-normal law clipped to it"""
    from statistics import NormalDist
    us = [(i + 0.5) / n for i in range(n)]
    lens = [int(median * math.exp(0.8 * NormalDist().inv_cdf(u))) if median else int(lo + u * (hi + 1 - lo)) for u in us]
    return [(KIND_DECODE, max(lo, min(hi, v)) - 1, 1) for v in lens]


@pytest.mark.parametrize("fold", [2, 4, 8, 64])
@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 1000, 4097])
def test_every_item_has_one_turn(n, fold):
    turns = lib().turns_of(n, fold)
    items = [lib().item_of_turn(t, n, fold) for t in range(turns)]
    assert n <= turns < n + fold and sorted(i for i in items if i < n) == list(range(n))
    assert all(0 <= i for i in items)


# The list's own order stays what it is but for a few neighbours: it begins with the longest items.
@pytest.mark.parametrize("fold", [2, 4, 16])
def test_turns_keep_the_order_of_the_list(fold):
    items = [lib().item_of_turn(t, 5000, fold) for t in range(lib().turns_of(5000, fold))]
    assert max(abs(i - t) for t, i in enumerate(items)) < 32 * fold


# Requests of an even number of splits: the items that are left with work (the first of every fold) fall to all parts of the chip that the
# turns are dealt to - 4, 8 or 32 of them - alike.
@pytest.mark.parametrize("parts", [4, 8, 32])
@pytest.mark.parametrize("requests,splits,fold", [(24, 8, 8), (24, 8, 4), (8, 24, 4), (48, 16, 2), (100, 32, 8), (16, 20, 4), (40, 7, 2)])
def test_items_with_work_are_dealt_to_all_parts(requests, splits, fold, parts):
    n = requests * splits
    turns = [t for t in range(lib().turns_of(n, fold)) if lib().item_of_turn(t, n, fold) < n and lib().item_of_turn(t, n, fold) % splits % fold == 0]
    per = collections.Counter(t % parts for t in turns)
    most = -(-len(turns) // parts)
    assert len(turns) == requests * -(-splits // fold) and max(per.values()) <= 1.2 * most + 1


# Lists on which a choice of splits taken together, or of none, was seen to cost 5 - 25 %, and others between them: kv heads, requests, chunks;
# measured us of the attention by the one-wavefront kernel (0) and by the other with 1, 2, .. splits as one.
MEASURED = [
    (2, decode(48, 2000, 8000), (), {0: 68.6, 1: 73.2, 2: 67.5, 4: 65.1, 8: 63.5, 16: 94.1}),
    (2, decode(96, 100, 600), (), {0: 18.2, 1: 21.7, 2: 18.2, 4: 20.6, 8: 17.6, 16: 17.9, 32: 17.7}),
    (4, decode(80, 2000, 8000), (), {0: 161.8, 1: 159.6, 2: 161.2, 4: 179.8}),
    (4, decode(112, 500, 4000), (), {0: 106.3, 1: 105.4, 2: 112.8, 4: 111.7}),
    (8, decode(24, 500, 4000), (), {0: 54.8, 1: 58.6, 2: 51.5, 4: 52.6, 8: 60.0, 16: 79.4}),
    (8, decode(40, 2000, 8000), (), {0: 157.9, 1: 155.8, 2: 155.0, 4: 178.1}),
    (8, decode(256, 16, 100), (), {0: 24.7, 1: 31.6}),
    (8, decode(4, 3072, 3072), (), {0: 24.3, 1: 28.3, 2: 21.0, 4: 19.3, 8: 25.2, 16: 38.2, 32: 47.9}),
    (8, decode(512, 16, 8192, 1024), (), {0: 503.4, 1: 507.2}),
    (8, decode(64, 500, 4000), ((1500, 300),), {0: 140.3, 1: 129.9, 2: 135.7, 4: 151.8}),
    (4, decode(128, 500, 4000), ((1500, 300),), {0: 142.4, 1: 133.1, 2: 139.9, 4: 152.7}),
    (8, decode(512, 16, 600), ((2967, 33),), {0: 231.9, 1: 134.8}),
    (8, decode(24, 500, 4000), ((0, 20),), {0: 55.7, 1: 58.6, 2: 51.7, 4: 52.7, 8: 60.4, 16: 77.4}),
]


@pytest.mark.parametrize("nkv,requests,chunks,us", MEASURED)
def test_choice_of_attention_kernel(nkv, requests, chunks, us):
    maps, blob, keep = build_maps(nkv, requests + [(KIND_PREFILL, s, n) for s, n in chunks])
    fold, _ = attention_plan(maps, nkv)
    assert us[fold] <= 1.03 * us[0] and us[fold] <= 1.1 * min(us.values())


@pytest.mark.parametrize("split", [0, 2, 4, 6, 12, 34, 64, 128, 200, 256])
@pytest.mark.parametrize("nkv", [1, 8, 32])
def test_limits_of_the_choice(nkv, split):
    for n, hi in ((1, 5), (1, 9000), (7, 300), (40, 5000), (300, 700)):
        for chunks in ((), ((0, 37),), ((4000, 1),), ((700, 300), (0, 17))):
            maps, blob, keep = build_maps(nkv, decode(n, 1, hi) + [(KIND_PREFILL, s, c) for s, c in chunks], split)
            fold, _ = attention_plan(maps, nkv)
            assert fold == 0 or (fold & (fold - 1) == 0 and (fold == 1 or fold * maps.kv_split_pages <= 256))
            maps.req_tok_off = None      # (which request has one token cannot be asked)
            assert attention_plan(maps, nkv)[0] == 0
    maps, blob, keep = build_maps(nkv, [(KIND_PREFILL, 0, 64), (KIND_PREFILL, 3000, 320)], split)
    assert maps.n_single == 0 and attention_plan(maps, nkv) == (1, True)
