"""GPU parity of attnw_attention (bf16) with the K and V of a head in LDS and a wave per 32 queries: every head size up to 128, last
blocks of one key, of 31 and whole, workgroups with and without idle waves, the largest K and V that fit (also past the reach of the
direct transfers)."""
import pytest

from paper_2407_13885_amd import workloads as wl

import gpu_util as gu
from test_gpu_attention_general import _check, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


@pytest.mark.parametrize("heads,N,d", [(2, N, d) for d in (32, 64) for N in (1, 31, 33, 64, 65, 96, 129, 197, 256, 257, 400, 511, 512)] +
                         [(3, N, d) for d in (16, 48, 80, 96, 112, 128) for N in (33, 100, 257, 320)] +
                         [(1, 640, 64), (1, 577, 64), (1, 1280, 32), (1, 1249, 32), (2, 416, 96), (700, 129, 64), (600, 257, 32)])
def test_keys_in_lds(heads, N, d, monkeypatch):
    monkeypatch.setenv("ATTNW_ATTENTION_KERNEL", "heads")
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=3900 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=3901 + N)
    O = gu.to_f64(_run(x, V))
    for h in {0, heads - 1}:
        _check(O[0, h], x, V, 0, h, (0, N), f"{heads} heads of {N} x {d}, head {h}")


def test_negative_scale(monkeypatch):
    monkeypatch.setenv("ATTNW_ATTENTION_KERNEL", "heads")
    x = wl.fused_inputs("t", "bf16", 1, 2, 333, 64, seed=3950, scale=-0.125, row_factor=(0.5, 3.0))
    V = wl.value_inputs(x, seed=3951)
    O = gu.to_f64(_run(x, V))
    for h in range(2):
        _check(O[0, h], x, V, 0, h, (0, 333), f"negative scale, head {h}")


# few heads of more than 256 tokens, and 256 tokens of d = 32: left to the kernels of 256-query strips; and the neighbours that are not
@pytest.mark.parametrize("heads,N,d", [(102, 480, 64), (263, 288, 64), (257, 336, 64), (755, 256, 32), (135, 450, 64), (346, 288, 64),
                                       (755, 255, 32)])
def test_as_dispatched(heads, N, d):
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=3960 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=3961 + N)
    O = gu.to_f64(_run(x, V))
    for h in {0, heads - 1}:
        _check(O[0, h], x, V, 0, h, (0, N), f"{heads} heads of {N} x {d}, head {h}")
