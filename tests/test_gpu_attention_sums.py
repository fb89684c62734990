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


# one query block per wave (d = 32 and 64, whole strips and ragged ends) and two, each on the sums
SHAPES = [(100, 1024, 32), (72, 1120, 32), (50, 1280, 64), (50, 1100, 64), (40, 3072, 64)]


def _pairs(heads, N, d, seed):
    """Small noise; the last two columns of Q are one, those of K nothing yet: they add to the logits of their key, an eighth a unit."""
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=seed, scale=0.125)
    x.Q[...] = wl.store(wl.widen(x.Q, "bf16") * 0.25, "bf16")
    x.Q[..., d - 2:] = 0x3f80
    x.K[..., d - 2:] = 0
    return x


@pytest.mark.parametrize("heads,N,d", SHAPES)
@pytest.mark.parametrize("again", [False, True])
def test_scores_jump_by_the_range_of_fp32(heads, N, d, again):
    """One key, or one of every 32 from there on, 86 to 90 logits above all others: weights against the exponent in force from 2^124 to beyond
    2^128, factors between the exponents down to 2^-130 (below 2^-126 the instruction gives 0)."""
    x = _pairs(heads, N, d, 3800 + N + d)
    keys = np.arange(N // 2 + 5, N, 32) if again else np.array([N // 2 + 5])
    for h in range(17):
        x.K[0, h, keys, d - 2] = wl.store(np.float32(512.0), "bf16")
        x.K[0, h, keys, d - 1] = wl.store(np.float32(176 + 2 * h), "bf16")
    V = wl.value_inputs(x, seed=3801 + N)
    O = gu.to_f64(_run(x, V))
    for h in range(18):
        _check_rows(O[0, h], x, V, 0, h, [(0, 32), (N - 32, N)], f"{heads} heads of {N} x {d}, jump {h} of 17")


@pytest.mark.parametrize("heads,N,d", SHAPES)
def test_exponents_of_a_million(heads, N, d):
    """Exponents of 1.5 million (an ulp is an eighth): the keys of two blocks weigh the same, whichever of them moved the exponent."""
    x = _pairs(heads, N, d, 3900 + N + d)
    x.Q[..., :d - 2] = 0
    x.K[..., d - 2] = wl.store(np.float32(2.0 ** 23), "bf16")
    V = np.zeros_like(x.K)
    first, second = slice(N // 2, N // 2 + 32), slice(N // 2 + 160, N // 2 + 192)
    V[:, :, first], V[:, :, second] = 0x3f80, 0xbf80
    for h in range(heads):
        x.K[0, h, first, d - 1] = x.K[0, h, second, d - 1] = wl.store(np.float32(80 + h), "bf16")
    O = gu.to_f64(_run(x, V))
    for h in range(heads):
        _check_rows(O[0, h], x, V, 0, h, [(0, 2), (N - 2, N)], f"{heads} heads of {N} x {d}, head {h}")
