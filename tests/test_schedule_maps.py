"""The index maps of the workgroup schedule, restated in Python: every (head, block)
is taken exactly once, whatever the number of heads and blocks.  direct_item is the
forward's order without tables; the slot map is how parts of a head find their
blocks (acp_schedule.h)."""
import random

import pytest


def direct_item(i, BH, nb):
    blk = i // BH
    bh = i - blk * BH + blk % BH
    bh -= BH if bh >= BH else 0
    return bh, nb - 1 - blk


def log_parts(BH, nb):
    if nb < 32:
        return 0
    s = 0
    while s < 3 and (BH <= 16 or ((BH << s) & 7) or (BH << (s + 1)) <= 64):
        s += 1
    return s if (BH << s) <= 64 else 3 if BH <= 32 else 0


@pytest.mark.parametrize("nb", [1, 2, 3, 8, 31, 32, 33, 63, 64, 100, 1024])
def test_direct_items_are_a_permutation(nb):
    for BH in (1, 2, 3, 7, 8, 12, 16, 33, 64, 100):
        items = [direct_item(i, BH, nb) for i in range(BH * nb)]
        assert sorted(items) == [(h, b) for h in range(BH) for b in range(nb)]
        # longest blocks first
        assert all(a[1] >= b[1] for a, b in zip(items, items[1:]))


@pytest.mark.parametrize("nb", [32, 33, 39, 63, 64, 127, 1000])
def test_parts_cover_every_block_once(nb):
    rng = random.Random(nb)
    for BH in list(range(1, 41)) + [48, 56, 64, 65]:
        lp = log_parts(BH, nb)
        parts, NP = 1 << lp, BH << lp
        deal = lp == 3 and BH <= 32
        greedy = not deal and NP % 8 == 0 and NP <= 64
        assert NP <= 256
        if lp == 0 or not (deal or greedy):
            assert lp == 0            # whole heads, or head order
            continue
        assert NP % 8 == 0
        if deal:
            rank = list(range(BH))
            rng.shuffle(rank)
            place = [None] * NP
            for t in range(NP):
                place[BH * (t & 7) + rank[t >> 3]] = t
        else:
            place = list(range(NP))
            rng.shuffle(place)
        first = [t * (nb >> lp) + sum((place[i] & (parts - 1)) < (nb & (parts - 1)) for i in range(t))
                 for t in range(NP)]
        seen = set()
        for lid in range(BH * nb):
            slot, step = 0, 128
            while step:
                if slot + step < NP and first[slot + step] <= lid:
                    slot += step
                step //= 2
            idx = (place[slot] & (parts - 1)) + ((lid - first[slot]) << lp)
            assert 0 <= idx < nb
            seen.add((place[slot] >> lp, idx))
        assert len(seen) == BH * nb
