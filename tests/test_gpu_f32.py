"""The float32 kernels at the sizes where their launch shape changes (16, 32 or 64
rows per workgroup, chosen by the number of rows) and where a workgroup's waves
get no subtile, against the oracle; and masked entries that are not finite.

Tolerance: the float32 path's 1e-4 on every output, relative to the largest
reference value where that exceeds 1 (as in test_gpu_attn.py: float32 sums over
up to L terms carry a relative error of order sqrt(L) 2^-24)."""
import numpy as np
import pytest
import torch

from paper_2504_06949_amd import acp, workloads
from tests._helpers import EPS, ensure_built, to_gpu
from tests.test_gpu_attn import _full_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("B,H,L,d,heads", [
    (1, 1, 64, 64, None),              # one block, 16 rows per workgroup
    (1, 1, 64, 128, None),
    (1, 5, 448, 64, None),
    (4, 16, 512, 64, 2),               # 32768 rows: 32 per workgroup
    (4, 16, 448, 64, 2),               # 28672: still 16 in the backward, 16 in the forward
    (16, 16, 256, 64, 2),              # 65536: 64 per workgroup in the forward
    (4, 8, 512, 128, 2),               # 16384: 32 in the d = 128 forward
])
def test_launch_shapes(B, H, L, d, heads):
    w = workloads.custom(f"f32_{B}_{H}_{L}_{d}", B, H, L, d, "f32", 40 + L + d, mu=(0.5, 3.0, 8.0))
    print(f"case: {w.describe()}", flush=True)
    pick = None if heads is None else [(0, 0), (B - 1, H - 1)]
    _full_parity(w, heads=pick)


@pytest.mark.parametrize("d", [64, 128])
def test_masked_nonfinite_values_do_not_leak(d):
    """An infinite or NaN row of V reaches only the queries that keep it, and one of
    dO only the keys that its query keeps: the others' outputs are those of the
    same call without it."""
    w = workloads.custom("f32_nf", 1, 2, 192, d, "f32", 91, mu=(2.0, 6.0))
    print(f"case: {w.describe()}", flush=True)
    g = to_gpu(workloads.generate(w))
    o0, lse0, _ = acp.forward(g["q"], g["k"], g["v"], g["log_f"], EPS)
    v = g["v"].clone()
    v[0, 0, 70, 3] = float("inf")
    v[0, 0, 150] = float("nan")
    o, lse, ws = acp.forward(g["q"], g["k"], v, g["log_f"], EPS)
    assert torch.equal(lse, lse0) and torch.equal(o[0, 1], o0[0, 1])
    assert torch.equal(o[0, 0, :70], o0[0, 0, :70])
    assert torch.isposinf(o[0, 0, 70:75, 3]).all() and torch.isnan(o[0, 0, 150]).all()
    keep = [c for c in range(d) if c != 3]
    assert torch.equal(o[0, 0, 70:150][:, keep], o0[0, 0, 70:150][:, keep])

    o, lse, ws = acp.forward(g["q"], g["k"], g["v"], g["log_f"], EPS)
    want = acp.backward(g["q"], g["k"], g["v"], o, g["do"], ws)
    do = g["do"].clone()
    do[0, 0, 70, 3] = float("inf")
    got = acp.backward(g["q"], g["k"], g["v"], o, do, ws)
    torch.cuda.synchronize()
    for a, b in zip(got[:3], want[:3]):
        assert torch.equal(a[0, 1], b[0, 1])
    np.testing.assert_array_equal(got[2][0, 0, 71:].cpu().numpy(), want[2][0, 0, 71:].cpu().numpy())
    assert torch.isinf(got[2][0, 0, 70, 3])


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("d", [64, 128])
def test_masked_nonfinite_rows_do_not_leak_into_gradients(d, bad):
    """A row of K that is not finite reaches dQ of the queries from its own on, and a
    row of Q dK and dV of the keys up to its own: the other rows are those of the same
    call without it (they mask it).  The bound comes from QK-norm scales, so that the
    plan does not depend on the rows."""
    w = workloads.custom("f32_nfg", 1, 2, 192, d, "f32", 92, mu=(2.0, 6.0))
    print(f"case: {w.describe()} {bad}", flush=True)
    g = to_gpu(workloads.generate(w))
    gam = torch.full((2,), 1.5, device="cuda")

    def grads(q, k):
        o, _, ws = acp.forward_qknorm(q, k, g["v"], g["log_f"], gam, gam, EPS)
        return acp.backward(q, k, g["v"], o, g["do"], ws)

    want = grads(g["q"], g["k"])
    for row, col in ((70, 5), (70, slice(None)), (143, 0)):
        k = g["k"].clone()
        k[0, 0, row, col] = bad
        got = grads(g["q"], k)
        assert torch.equal(got[0][0, 0, :row], want[0][0, 0, :row])
        assert torch.isnan(got[0][0, 0, row]).any()
        for a, b in zip(got[:3], want[:3]):
            assert torch.equal(a[0, 1], b[0, 1])
        q = g["q"].clone()
        q[0, 0, row, col] = bad
        got = grads(q, g["k"])
        for a, b in zip(got[1:3], want[1:3]):
            assert torch.equal(a[0, 0, row + 1:], b[0, 0, row + 1:])
            assert torch.equal(a[0, 1], b[0, 1])
        assert torch.isnan(got[1][0, 0, row]).any()
        keep = [r for r in range(192) if r != row]
        assert torch.equal(got[0][0, 0, keep], want[0][0, 0, keep])
