"""The choices of the attention's work list (no GPU): in which order its items run where key splits are taken together."""
import collections

import pytest

from attn_plan import lib


@pytest.mark.parametrize("fold", [2, 4, 8, 64])
@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 1000, 4097])
def test_every_item_has_one_turn(n, fold):
    turns = lib().turns_of(n, fold)
    items = [lib().item_of_turn(t, n, fold) for t in range(turns)]
    assert n <= turns < n + fold and sorted(i for i in items if i < n) == list(range(n))
    assert all(0 <= i for i in items)


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
