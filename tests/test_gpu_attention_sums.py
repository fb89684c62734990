"""GPU parity of attnw_attention (bf16, d = 32 and 64, 1024 tokens and more), where the exponent of the weights follows their sums: scores that
climb by fractions of a binade and by hundreds of them a sub-tile, up to where weights against the old exponent overflow."""
import numpy as np
import pytest

from paper_2407_13885_amd import workloads as wl

import gpu_util as gu
from test_gpu_attention import _check_rows, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


# one and two query blocks per wave, whole strips and ragged ends, each with enough heads for the kernel
@pytest.mark.parametrize("heads,N,d", [(100, 1024, 32), (72, 1120, 32), (40, 3072, 32), (100, 1024, 64), (70, 1100, 64), (40, 3072, 64)])
@pytest.mark.parametrize("step", [0.05, 0.7, 9.0, 200.0])
def test_scores_climb(heads, N, d, step):
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=3700 + N + d)
    # the last column of K climbs every 32 keys, that of Q is one: the logits of a sub-tile lie `step` above those of the last
    h = heads - 1
    climb = step / float(x.scale) * (np.arange(N) // 32)
    x.Q[0, h, :, d - 1] = 0x3f80
    x.K[0, h, :, d - 1] = (climb.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    V = wl.value_inputs(x, seed=3701 + N)
    O = gu.to_f64(_run(x, V))
    _check_rows(O[0, h], x, V, 0, h, [(0, 96), (N - 96, N)], f"{heads} heads of {N} x {d}, step {step}")
    _check_rows(O[0, 0], x, V, 0, 0, [(0, 64)], f"{heads} heads of {N} x {d}, head 0")
