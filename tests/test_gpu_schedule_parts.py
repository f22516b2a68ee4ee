"""The workgroup schedule of long sequences (32 or more 128-row blocks per head),
where parts of a head may run on different XCDs: every table is a permutation of
the (head, block) items, each XCD's range runs largest first, and, where heads are
split, no XCD holds much more work than the average."""
import numpy as np
import pytest
import torch

from paper_2504_06949_amd import acp, workloads
from tests.test_gpu_schedule import item_work, xcd_ranges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,L,parts,seed", [
    (1, 1, 4096, 8, 81),      # one head over all XCDs
    (1, 8, 4160, 8, 82),      # 33 blocks, the last one ragged: parts of 5 and 4 blocks
    (1, 11, 4096, 8, 83),     # 88 parts dealt out, 11 per XCD
    (1, 18, 4096, 8, 84),     # 18 heads: no multiple of 8 below 64 parts
    (2, 10, 4224, 2, 85),     # 20 heads: 40 parts placed by load
    (2, 32, 4096, 1, 86),     # 64 whole heads placed by load
    (3, 20, 4096, 1, 87),     # 60 heads: head order
])
def test_long_schedule(B, H, L, parts, seed):
    w = workloads.custom(f"parts{seed}", B, H, L, 64, "bf16", seed, mu=(0.5, 2.0, 5.0, 9.0, 20.0))
    print(f"case: schedule {w.describe()}", flush=True)
    x = workloads.generate(w, with_grad=False)
    g = {k: (v.cuda() if torch.is_tensor(v) else v) for k, v in x.items()}
    _, _, ws = acp.forward(g["q"], g["k"], g["v"], g["log_f"], w.eps)
    torch.cuda.synchronize()
    pv = {k: v.cpu().numpy() for k, v in acp.plan_views(ws, B, H, L, 64, torch.bfloat16).items()}
    BH, M, nb = B * H, L // 64, (L + 127) // 128
    rs, ce = pv["row_start"].reshape(BH, M), pv["col_end"].reshape(BH, M)
    for table in ("q", "k"):
        sched = pv["sched_" + table].astype(np.int64)
        assert sorted(sched.tolist()) == list(range(BH * nb)), "not a permutation"
        loads = []
        for lo, hi in xcd_ranges(BH * nb):
            works = [item_work(table, e // nb, e % nb, M, rs, ce) for e in sched[lo:hi].tolist()]
            assert all(a >= b for a, b in zip(works, works[1:])), "not largest first"
            loads.append(sum(works))
        if parts == 8:
            # each XCD has every 8th block of every head: within one block of the
            # longest kind (2 M tiles) per head of the average
            assert max(loads) <= sum(loads) / 8 + BH * 2 * M
        elif parts > 1:
            assert max(loads) <= 1.3 * sum(loads) / 8


@pytest.mark.parametrize("B,H,L,mu,seed", [
    (1, 16, 4096, 25.0, 91),     # nothing pruned: two whole heads per XCD
    (2, 16, 4160, 25.0, 92),     # four, the last block ragged
    (1, 24, 8192, -2.0, 93),     # two or three tiles per row everywhere: three whole heads
    (1, 20, 4096, -2.0, 94),     # two and a half heads per XCD, in head order
    (1, 3, 16384, -2.0, 95),
])
def test_equal_long_heads_stay_whole(B, H, L, mu, seed):
    """Heads of equal work are not divided: parts would balance nothing, and every XCD
    would read every head's keys and values."""
    w = workloads.custom(f"even{seed}", B, H, L, 64, "bf16", seed, mu=(mu,))
    print(f"case: schedule {w.describe()}", flush=True)
    x = workloads.generate(w, with_grad=False)
    g = {k: (v.cuda() if torch.is_tensor(v) else v) for k, v in x.items()}
    _, _, ws = acp.forward(g["q"], g["k"], g["v"], g["log_f"], w.eps)
    torch.cuda.synchronize()
    pv = acp.plan_views(ws, B, H, L, 64, torch.bfloat16)
    BH, nb = B * H, (L + 127) // 128
    for table in ("q", "k"):
        sched = pv["sched_" + table].cpu().numpy().astype(np.int64)
        assert sorted(sched.tolist()) == list(range(BH * nb)), "not a permutation"
        for lo, hi in xcd_ranges(BH * nb):
            heads = set((sched[lo:hi] // nb).tolist())
            if BH % 8 == 0:
                assert len(heads) == BH // 8
            else:
                assert heads == set(range(lo // nb, (hi - 1) // nb + 1))
