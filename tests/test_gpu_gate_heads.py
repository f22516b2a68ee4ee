"""The gate producer at the head counts where its kernel changes (up to 20 heads on
the VALU, in steps of 4; 2, 3 or 4 groups of 16 on the matrix cores) and where its
waves get no head or an incomplete round, and with odd numbers of 64-feature tiles:
log f and c bit for bit as the oracle's."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2504_06949_amd import acp, workloads
from tests._helpers import ensure_built, to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("B,H,L,dm,seed", [
    (2, 1, 256, 64, 1),       # one tile, three waves without a head
    (1, 4, 320, 192, 2),      # the last with one head per lane
    (1, 5, 320, 128, 3),      # the first with two
    (1, 8, 320, 192, 8),
    (1, 9, 320, 64, 9),
    (1, 12, 320, 192, 10),
    (1, 13, 320, 128, 11),
    (1, 16, 512, 320, 4),
    (1, 17, 512, 64, 5),      # five heads per lane
    (1, 20, 512, 192, 12),
    (1, 21, 512, 128, 13),    # the first on the matrix cores, two groups of 16
    (1, 32, 512, 192, 14),
    (1, 33, 512, 192, 6),     # three groups
    (1, 48, 512, 64, 15),
    (1, 49, 512, 128, 16),    # four
    (1, 64, 512, 128, 7),
])
def test_gate_head_counts(B, H, L, dm, seed):
    print(f"case: gate B={B} H={H} L={L} d_model={dm}", flush=True)
    x = workloads.gate_inputs(B, L, dm, H, seed)
    g = to_gpu(x)
    log_f, ws = acp.gate_project(g["x"], g["w_f"], g["b_f"], B, H, 64)
    torch.cuda.synchronize()
    c = acp.plan_views(ws, B, H, L, 64, torch.bfloat16)["c"].cpu().numpy()
    xf = x["x"].float().numpy().reshape(B, L, dm)
    for b in range(B):
        a = orc.gate_logits(xf[b], x["w_f"].float().numpy(), x["b_f"].numpy())
        want = orc.log_sigmoid(a).T.astype(np.float32)
        np.testing.assert_array_equal(log_f[b].cpu().numpy(), want)
        np.testing.assert_array_equal(c[b], orc.cumsum_log_gates(want))
