"""The bf16 kernels with several groups of waves sharing a 128-row block (chosen
for calls with few blocks), against the oracle: group counts that do and do not
divide the number of tiles, rows with fewer tiles than groups, short blocks (up to
6 tiles) that one group takes alone, a ragged last block, and both softmax variants
(fixed stabiliser; online maximum with a logit bound over 32).  Tolerances as in test_gpu_attn.py: 2e-2, relative to the largest
reference value above 1 on the bfloat16 outputs."""
import pytest
import torch

from paper_2504_06949_amd import acp, workloads
from tests._helpers import ensure_built, to_gpu
from tests.test_gpu_attn import _full_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("B,H,L,d,mu,norm,seed", [
    (1, 2, 2112, 64, (3.0, 9.0), None, 71),    # 4 groups, 3 in the backward; 33 tiles, ragged
    (1, 2, 2048, 64, (2.0, 9.0), 17.0, 72),    # the same with the online maximum
    (1, 2, 1088, 64, (1.0, 6.0), None, 73),    # 2 groups (9 blocks per head)
    (1, 2, 1024, 64, (1.0, 8.0), 17.0, 74),
    (1, 2, 1088, 128, (1.0, 8.0), None, 75),   # d = 128: 2 groups
    (1, 2, 1024, 128, (3.0, 8.0), 21.0, 76),
    (1, 1, 4160, 128, (5.0,), None, 77),       # the same through the schedule tables (33 blocks)
    (1, 1, 4160, 64, (5.0,), None, 78),        # 4 groups of a long head, without them
    (1, 1, 960, 64, (5.0,), None, 77),         # 8 blocks, the last one ragged
    (1, 1, 896, 64, (5.0,), None, 78),         # 7 blocks: one group
])
def test_groups(B, H, L, d, mu, norm, seed):
    w = workloads.custom(f"groups{seed}", B, H, L, d, "bf16", seed, mu=mu,
                         row_norms=None if norm is None else (norm,))
    print(f"case: {w.describe()}", flush=True)
    _full_parity(w)


@pytest.mark.parametrize("B,H,L,d,mu,seed", [
    (1, 2, 2112, 64, (-2.0,), 81),         # every block short: 4 and 3 groups, ragged
    (1, 2, 1088, 64, (-2.0, 1.0), 82),     # 2 and 3 groups, short and longer blocks
    (1, 2, 1088, 128, (-2.0, 1.0), 83),
    (1, 1, 4160, 128, (0.0,), 84),
])
def test_short_blocks(B, H, L, d, mu, seed):
    w = workloads.custom(f"short{seed}", B, H, L, d, "bf16", seed, mu=mu)
    print(f"case: {w.describe()}", flush=True)
    _full_parity(w)


@pytest.mark.parametrize("B,H,L,d,mu,chain", [
    (1, 16, 2176, 64, (-2.0,), 0),              # 272 blocks, all short: one group in the backward
    (1, 16, 2176, 64, (12.0,), 1),              # unpruned: 3
    (1, 16, 2112, 64, (-2.0, 1.0, 12.0), 1),    # ragged
    (1, 16, 2176, 128, (-2.0,), 0),             # 2 groups in the forward, one in dQ
    (1, 16, 2176, 128, (-2.0, 12.0), 1),
    (1, 8, 4224, 128, (0.0,), 0),               # 264 blocks, with the tables: one group
    (1, 8, 4160, 128, (0.0, 12.0), 1),          # and 2, ragged
])
def test_form_by_plan(B, H, L, d, mu, chain):
    """More than 256 blocks: both forms are launched and the plan picks one.  The longest
    last row against the mean over all rows says which (1.6 times)."""
    w = workloads.custom(f"plan{H}_{L}_{d}_{chain}", B, H, L, d, "bf16", 85, mu=mu)
    print(f"case: {w.describe()}", flush=True)
    g = to_gpu(workloads.generate(w))
    _, _, ws = acp.forward(g["q"], g["k"], g["v"], g["log_f"], w.eps)
    pv = acp.plan_views(ws, B, H, L, d, torch.bfloat16)
    M = L // 64
    longest = int((M - pv["row_start"][..., M - 1]).max())
    mean = float(pv["kept"].sum()) / (B * H * M)
    assert (longest >= 1.6 * mean) == bool(chain)
    _full_parity(w, heads=[(0, 0), (0, 1), (0, H - 1)])
