"""GPU parity of attnw_attention (bf16, d = 64) on both sides of the choice between one and two query blocks per wave: as many workgroups as
compute units, one more, twice as many; whole strips, ragged ones and partial strips in a launch of their own."""
import pytest

from paper_2407_13885_amd import workloads as wl

import gpu_util as gu
from test_gpu_attention import _check_rows, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


@pytest.mark.parametrize("heads,N", [(32, 4096), (33, 4096), (51, 2560), (52, 2560), (128, 2048), (65, 1024), (130, 768), (52, 2400), (45, 2743), (86, 700),
                                     (86, 1025), (63, 1057), (129, 1025), (8, 8256), (257, 513)])
def test_blocks_per_wave(heads, N):
    x = wl.fused_inputs("t", "bf16", 1, heads, N, 64, seed=4100 + N + heads)
    V = wl.value_inputs(x, seed=4101 + N)
    O = gu.to_f64(_run(x, V))
    rows = [(0, 64), (N - 96, N)] + ([(N // 512 * 512 - 32, N // 512 * 512 + 32)] if N % 512 > 32 and N > 544 else [])
    for h in (0, heads // 2, heads - 1):
        _check_rows(O[0, h], x, V, 0, h, rows, f"{heads} heads of {N}, head {h}")
