"""GPU parity of attnw_attention (fp32) on few heads, where workgroups share the columns of V and O of a query block: every number of
column blocks, head sizes that end inside one, last key ranges of one key and without keys, last query blocks of one query."""
import pytest

from paper_2407_13885_amd import workloads as wl

import gpu_util as gu
from test_gpu_attention_general import _check, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


@pytest.mark.parametrize("d", [36, 64, 68, 96, 100, 128, 132, 160, 164, 192, 196, 224, 228, 252, 256])
@pytest.mark.parametrize("heads,N", [(1, 65), (1, 96), (2, 97), (1, 129), (3, 200), (1, 385), (2, 673), (1, 1921)])
def test_columns_shared(heads, N, d):
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=4100 + N + d)
    V = wl.value_inputs(x, seed=4101 + N)
    O = gu.to_f64(_run(x, V))
    for h in {0, heads - 1}:
        _check(O[0, h], x, V, 0, h, (0, N), f"{heads} heads of {N} x {d}, head {h}")
