"""GPU parity of attnw_attention (bf16) on few heads whose query blocks are shared by several workgroups, each with its share of the
columns of V and O: every share (2, 3, 4 workgroups), its waves' last keys ragged, and as many blocks as still share."""
import pytest

from paper_2407_13885_amd import workloads as wl

import gpu_util as gu
from test_gpu_attention_general import _check, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


@pytest.mark.parametrize("d", [64, 96, 128, 192, 256])
@pytest.mark.parametrize("heads,N", [(1, 257), (2, 512), (1, 1000), (7, 288), (3, 1025), (6, 640), (4, 1024), (9, 801)])
def test_shared_columns(heads, N, d):
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=3800 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=3801 + N)
    O = gu.to_f64(_run(x, V))
    for h in {0, heads - 1}:
        _check(O[0, h], x, V, 0, h, (0, N), f"{heads} heads of {N} x {d}, head {h}")
