"""The Q/K projection at sizes that take its 256 x 256 tile: a last row tile with
one 128-row chunk, row tiles across two sequences, and column tiles half in Q and
half in K.  Q and K against the float64 product (bfloat16 rounding: half an ulp is
2^-9 relative; the float32 sums of d_model products add d_model 2^-24), the norm
maxima through the bound U, bit for bit that of a forward on the same Q and K."""
import pytest
import torch

from paper_2504_06949_amd import acp, workloads
from tests._helpers import EPS, ensure_built, to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("B,H,L,d,dm,seed", [
    (1, 12, 32640, 64, 512, 1),     # 255 chunks of 128 rows
    (6, 10, 2176, 64, 576, 2),      # 17 chunks per sequence; H d = 640
    (6, 5, 2176, 128, 512, 3),
])
def test_large_tiles(B, H, L, d, dm, seed):
    print(f"case: project B={B} H={H} L={L} d={d} d_model={dm}", flush=True)
    g = to_gpu(workloads.projection_inputs(B, L, dm, H, d, seed))
    q, k, ws = acp.project_qk(g["x"], g["wq"], g["wk"], B, H, d)
    x = g["x"].double()
    for got, w in ((q, g["wq"]), (k, g["wk"])):
        want = (x @ w.double()).view(B, L, H, d).transpose(1, 2)
        err = (got.double() - want).abs()
        # the float32 sum's error is relative to the sum of |x w|, at most |x| |w| per row
        bound = want.abs() * 2.0 ** -8 + dm * 2.0 ** -24 * float((x * x).sum(1).max().sqrt()) * float(
            (w.double() ** 2).sum(0).max().sqrt())
        assert bool((err <= bound).all())
    v = torch.zeros_like(q)
    log_f = torch.full((B, H, L), -0.01, device="cuda")
    acp.forward_projected(q, k, v, log_f, EPS, ws)
    plan = acp.plan_views(ws, B, H, L, d, torch.bfloat16)
    _, _, ws2 = acp.forward(q, k, v, log_f, EPS)
    plan2 = acp.plan_views(ws2, B, H, L, d, torch.bfloat16)
    torch.cuda.synchronize()
    assert torch.equal(plan["bound_u"], plan2["bound_u"])
    assert torch.equal(plan["row_start"], plan2["row_start"])
