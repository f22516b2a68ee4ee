"""The per-head scans where a thread's run of positions is longer than its
registers hold and ends inside a batch: the decoding set-up on prompts that are
no multiple of 4 (single loads) and of 4 only, and dlog f at L = 16448; and on both
sides of 4096, where dlog f holds 4 values per thread or 16; against the oracle (tolerances of test_gpu_decode.py and test_gpu_attn.py)."""
import pytest

from paper_2504_06949_amd import workloads
from tests._helpers import EPS, ensure_built
from tests.test_gpu_attn import _full_parity
from tests.test_gpu_decode import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("L0,C,sigma", [
    (16387, 17408, 0.5),     # 20 positions per thread, unaligned heads
    (16390, 1024, 0.5),      # a ring shorter than the prompt
    (20484, 1024, 6.0),      # whole float4s; spans over 53 bits (double-double)
])
def test_decode_setup_long_odd_prompts(L0, C, sigma):
    w = workloads.custom(f"runs{L0}", 1, 2, L0 + 2, 64, "bf16", 95, mu=(3.0, 9.0), gate_sigma=sigma,
                         qk_norm=True)
    _check(w, L0, C, EPS, 2 * L0)


@pytest.mark.parametrize("L", [4096, 4160, 16448])
def test_dlogf_run_tail(L):
    w = workloads.custom(f"tail{L}", 1, 1, L, 64, "bf16", 96, mu=(4.0,))
    print(f"case: fwd/bwd {w.describe()}", flush=True)
    _full_parity(w)
