"""The launch rules and index maps of the attention kernels' workgroup schedule
(csrc/acp_rules.h, which the kernels include), compiled for the host: every (head,
block) is taken exactly once, whatever the number of heads and blocks, and the rules
agree with one another."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_2504_06949_amd import build

WRAPPER = r"""
#include "acp_rules.h"
using namespace acp;
extern "C" {
int w_direct_item(int i, int BH, int nb) { return direct_item(i, BH, nb); }
int w_log_parts(int BH, int nb) { return schedule_log_parts(BH, nb); }
int w_placing(int BH, int lp) { return (int)schedule_placing(BH, lp); }
int w_deal_slot(int part, int rank, int BH) { return deal_slot(part, rank, BH); }
int w_part_blocks(int p, int lp, int nb) { return part_blocks(p, lp, nb); }
int w_slot_of(const int* first, int NP, int lid) { return slot_of(first, NP, lid); }
int w_part_index(int placed, int lp, int nth) { return part_index(placed, lp, nth); }
void w_range(int n, int x, int* lo, int* hi) { schedule_range(n, x, *lo, *hi); }
int w_forward_direct(int d, int n, int nb) { return forward_direct(d, n, nb); }
void w_fwd_groups(int d, int n, int nb, int direct, int* out) {
    const Groups g = fwd_groups(d, n, nb, direct != 0);
    out[0] = g.groups; out[1] = g.by_plan;
}
void w_bwd_groups(int d, int n, int nb, int* out) {
    const Groups g = bwd_groups(d, n, nb);
    out[0] = g.groups; out[1] = g.by_plan;
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.cpp", d / "librules.so"
    src.write_text(WRAPPER)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I", build.CSRC, "-o", str(lib), str(src)], check=True)
    return ctypes.CDLL(str(lib))


@pytest.mark.parametrize("nb", [1, 2, 3, 8, 31, 32, 33, 63, 64, 100, 1024])
def test_direct_items_are_a_permutation(rules, nb):
    for BH in (1, 2, 3, 7, 8, 12, 16, 33, 64, 100):
        items = [rules.w_direct_item(i, BH, nb) for i in range(BH * nb)]
        assert sorted(items) == list(range(BH * nb))
        blocks = [e % nb for e in items]
        assert all(a >= b for a, b in zip(blocks, blocks[1:]))   # longest first


@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 64, 1000, 1344])
def test_ranges_are_the_logical_ids(rules, n):
    lo, hi, end = ctypes.c_int(), ctypes.c_int(), 0
    for x in range(8):
        rules.w_range(n, x, ctypes.byref(lo), ctypes.byref(hi))
        assert lo.value == end and hi.value - lo.value == len(range(x, n, 8))
        end = hi.value
    assert end == n


@pytest.mark.parametrize("nb", [32, 33, 39, 63, 64, 127, 1000])
def test_parts_cover_every_block_once(rules, nb):
    DEALT, BY_LOAD, NONE = 0, 1, 2
    rng = random.Random(nb)
    for BH in list(range(1, 41)) + [48, 56, 64, 65, 200]:
        lp = rules.w_log_parts(BH, nb)
        NP, placing = BH << lp, rules.w_placing(BH, lp)
        if lp == 0:
            # whole heads, by load for a multiple of 8 up to 64, or head order
            assert placing == (BY_LOAD if BH % 8 == 0 and BH <= 64 else NONE)
            continue
        assert placing != NONE and NP % 8 == 0
        assert NP <= (256 if placing == DEALT else 64)
        if placing == DEALT:
            rank = list(range(BH))
            rng.shuffle(rank)
            place = [None] * NP
            for t in range(NP):
                place[rules.w_deal_slot(t & 7, rank[t >> 3], BH)] = t
        else:
            place = list(range(NP))
            rng.shuffle(place)
        assert sorted(place) == list(range(NP))
        sizes = [rules.w_part_blocks(t & ((1 << lp) - 1), lp, nb) for t in place]
        first = [sum(sizes[:t]) for t in range(NP)]
        assert first[-1] + sizes[-1] == BH * nb
        arr = (ctypes.c_int * NP)(*first)
        seen = set()
        for lid in range(BH * nb):
            slot = rules.w_slot_of(arr, NP, lid)
            assert first[slot] <= lid < first[slot] + sizes[slot]
            idx = rules.w_part_index(place[slot], lp, lid - first[slot])
            assert 0 <= idx < nb
            seen.add((place[slot] >> lp, idx))
        assert len(seen) == BH * nb


def test_short_heads_have_no_parts(rules):
    for BH in range(1, 300):
        assert all(rules.w_log_parts(BH, nb) == 0 for nb in (1, 8, 31))


def test_group_rules_agree(rules):
    """The forms that are launched exist: several groups in the d = 64 forward only
    without tables; a form picked by the plan only where the schedule runs before the
    forward, and only where it leaves its answer (where the backward goes by it)."""
    f, b = (ctypes.c_int * 2)(), (ctypes.c_int * 2)()
    for nb in list(range(1, 80)) + [128, 500, 1024]:
        for BH in list(range(1, 140)) + [200, 1000]:
            n = BH * nb
            for d in (64, 128):
                direct = rules.w_forward_direct(d, n, nb)
                rules.w_fwd_groups(d, n, nb, direct, f)
                rules.w_bwd_groups(d, n, nb, b)
                assert f[0] in ((1, 2, 4) if d == 64 else (1, 2))
                assert b[0] in ((1, 3) if d == 64 else (1, 2))
                if d == 64 and f[0] > 1:
                    assert direct and not f[1]
                if f[1]:
                    assert not direct and f[0] > 1 and b[1]
                if b[1]:
                    assert b[0] > 1
