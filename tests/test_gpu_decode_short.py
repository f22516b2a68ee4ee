"""Decoding across the key and head counts where a step changes its launch: one
workgroup of 256 keys per head, one of 1024 (up to 256 heads), then several with a
merge; and rings that keep the count there for any context.  Every step against the oracle (test_gpu_decode.py's
checks and tolerances)."""
import pytest

from paper_2504_06949_amd import workloads
from tests._helpers import EPS, ensure_built
from tests.test_gpu_decode import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


@pytest.mark.parametrize("dtype,d,L0,L,C", [
    ("bf16", 64, 252, 260, 512),       # 253 .. 260 keys
    ("bf16", 128, 252, 260, 512),
    ("f32", 64, 252, 260, 512),
    ("f32", 128, 254, 258, 320),
    ("bf16", 64, 1020, 1028, 2048),    # 1021 .. 1028 keys
    ("bf16", 128, 1021, 1027, 1088),
    ("bf16", 64, 1500, 1504, 1024),    # a full ring of 1024
    ("bf16", 64, 700, 704, 256),       # and of 256
])
def test_decode_launch_edges(dtype, d, L0, L, C):
    w = workloads.custom(f"edge{L0}_{C}", 1, 3, L, d, dtype, 97, mu=(2.0, 6.0, 12.0), qk_norm=True)
    _check(w, L0, C, EPS, 4 * L)


@pytest.mark.parametrize("dtype,d,H,L0", [
    ("bf16", 64, 256, 300),    # one workgroup of 1024 per head
    ("bf16", 64, 257, 300),    # two of 256 and a merge
    ("bf16", 128, 257, 300),
    ("f32", 64, 257, 254),     # 255 .. 257 keys: one of 256, then two
])
def test_decode_many_heads(dtype, d, H, L0):
    w = workloads.custom(f"heads{H}", 1, H, L0 + 3, d, dtype, 98, mu=(2.0, 6.0, 12.0), qk_norm=True)
    _check(w, L0, 512, EPS, 2048)


@pytest.mark.parametrize("dtype,d,H,L0,C", [
    ("bf16", 64, 384, 257, 320),   # the set-up in one launch, its last workgroup with one row
    ("bf16", 64, 385, 257, 320),   # in two
    ("f32", 128, 385, 65, 64),     # in two, a ring shorter than the prompt
    ("bf16", 128, 385, 96, 128),   # in one
    ("bf16", 64, 1, 4097, 4160),   # a run of 8 positions per thread
])
def test_decode_setup_launches(dtype, d, H, L0, C):
    w = workloads.custom(f"setup{H}", 1, H, L0 + 1, d, dtype, 99, mu=(2.0, 6.0, 12.0), qk_norm=True)
    _check(w, L0, C, EPS, 2 * L0)
