"""GPU parity of attnw_attention (bf16, d = 176 to 256, more than 384 tokens) where the two waves of a SIMD take turns at the matrix unit: rests of the
ring of four tiles, ragged last tiles, strips with waves without queries, a last strip that another kernel takes, scores that climb from tile to
tile."""
import numpy as np
import pytest

from paper_2407_13885_amd import workloads as wl

import gpu_util as gu
from test_gpu_attention import _check_rows, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


# one full round of 256-query strips, (120, 520): 240 strips and eight queries of every head left over
@pytest.mark.parametrize("d", [176, 192, 208, 224, 240, 256])
@pytest.mark.parametrize("heads,N", [(128, 385), (128, 416), (128, 417), (128, 448), (128, 449), (128, 479), (128, 481), (128, 512), (120, 520), (16, 4066)])
def test_tiles(heads, N, d):
    names = gu.attention_kernels("bf16", heads, N, d)
    # (one full round: rows of fewer tokens than this are the other kernel's; strips with a tail of their own are not asked for their length)
    fewest = {176: 458, 192: 801, 208: 458, 224: 458, 240: 385, 256: 385}[d]
    assert ("attention_turns_kernel" in names[0]) == (N >= fewest or heads == 120) and len(names) == (2 if heads == 120 else 1)
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=5300 + N + heads)
    V = wl.value_inputs(x, seed=5301 + N)
    O = gu.to_f64(_run(x, V))
    for h in (0, heads // 2, heads - 1):
        _check_rows(O[0, h], x, V, 0, h, [(0, 33), (max(N - 40, 0), N)], f"{heads} heads of {N} x {d}, head {h}")


# the same rests where longer rows alone come here
@pytest.mark.parametrize("heads,N,d", [(128, 458, 176), (128, 500, 176), (64, 801, 192), (64, 833, 192), (64, 870, 192), (64, 896, 192), (51, 1057, 192), (128, 465, 224)])
def test_longer_rows(heads, N, d):
    assert "attention_turns_kernel" in gu.attention_kernels("bf16", heads, N, d)[0]
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=5360 + N)
    V = wl.value_inputs(x, seed=5361 + N)
    O = gu.to_f64(_run(x, V))
    for h in (0, heads - 1):
        _check_rows(O[0, h], x, V, 0, h, [(0, 33), (max(N - 40, 0), N)], f"{heads} heads of {N} x {d}, head {h}")


# rows of nine and ten tiles: the strips of 256 queries where a head's last ones are a launch of their own
@pytest.mark.parametrize("heads,N,d", [(240, 257, 176), (250, 320, 208), (256, 288, 256)])
def test_own_last_strip(heads, N, d):
    names = gu.attention_kernels("bf16", heads, N, d)
    assert "attention_turns_kernel" in names[0] and len(names) == 2
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=5350 + N)
    V = wl.value_inputs(x, seed=5351 + N)
    O = gu.to_f64(_run(x, V))
    for h in (0, heads - 1):
        _check_rows(O[0, h], x, V, 0, h, [(0, 33), (230, N)], f"{heads} heads of {N} x {d}, head {h}")


@pytest.mark.parametrize("heads,N,d", [(128, 449, 176), (128, 470, 176), (64, 850, 192), (128, 500, 208), (120, 520, 240), (128, 400, 256)])
@pytest.mark.parametrize("step", [0.05, 0.7, 9.0, 200.0])
def test_scores_climb(heads, N, d, step):
    scale = {"scale": -1.0 / 16} if d == 208 else {}
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=5400 + N + d, **scale)
    # the last column of K climbs every 32 keys, that of Q is one: the logits of a tile lie `step` above those of the last
    h = heads - 1
    climb = step / float(x.scale) * (np.arange(N) // 32)
    x.Q[0, h, :, d - 1] = 0x3f80
    x.K[0, h, :, d - 1] = (climb.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    V = wl.value_inputs(x, seed=5401 + N)
    O = gu.to_f64(_run(x, V))
    _check_rows(O[0, h], x, V, 0, h, [(0, 96), (N - 96, N)], f"{heads} heads of {N} x {d}, step {step}")
    _check_rows(O[0, 0], x, V, 0, 0, [(0, 64)], f"{heads} heads of {N} x {d}, head 0")
