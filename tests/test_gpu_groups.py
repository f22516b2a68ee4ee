"""The bf16 kernels with several groups of waves sharing a 128-row block (chosen
for calls with few blocks), against the oracle: group counts that do and do not
divide the number of tiles, rows with fewer tiles than groups, a ragged last
block, and both softmax variants (fixed stabiliser; online maximum with a logit
bound over 32).  Tolerances as in test_gpu_attn.py: 2e-2, relative to the largest
reference value above 1 on the bfloat16 outputs."""
import pytest

from paper_2504_06949_amd import workloads
from tests._helpers import ensure_built
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
