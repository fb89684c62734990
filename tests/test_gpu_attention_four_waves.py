"""GPU parity of attnw_attention (bf16, d of 80 and more) on both sides of the choice between workgroups of 128 and of 256 queries: one and two rounds
of either, three and four with the last one less and more than half full, ragged last strips, partial strips in a launch of their own, lengths of one strip."""
import pytest

from paper_2407_13885_amd import workloads as wl

import gpu_util as gu
from test_gpu_attention import _check_rows, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


@pytest.mark.parametrize("heads,N,d", [(128, 256, 128), (129, 256, 128), (300, 129, 96), (40, 600, 128), (24, 1377, 144), (64, 1024, 144), (65, 1025, 144),
                                       (130, 1025, 80), (61, 1057, 256), (70, 1100, 256), (130, 900, 240), (90, 700, 176), (600, 130, 208),
                                       (110, 1100, 96), (150, 1100, 96), (200, 1100, 96), (100, 1300, 224), (120, 1300, 224), (46, 4200, 256)])
def test_workgroups_of_four_waves(heads, N, d):
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=4300 + N + heads)
    V = wl.value_inputs(x, seed=4301 + N)
    O = gu.to_f64(_run(x, V))
    last = (N - 1) // 128 * 128
    for h in (0, heads // 2, heads - 1):
        _check_rows(O[0, h], x, V, 0, h, [(0, 32), (96, 129), (max(last - 32, 0), N)], f"{heads} heads of {N} x {d}, head {h}")
