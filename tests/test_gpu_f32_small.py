"""GPU parity of the fp32 attention weights of few short heads (workgroups of 16 queries, K straight from memory): last blocks of any number of keys, waves
without blocks and with two, every padding of a row, as many workgroups as compute units, neither sign of the scale."""
import math

import numpy as np
import pytest

import oracle
from paper_2407_13885_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


@pytest.mark.parametrize("d", [20, 32, 36, 48, 52, 64, 100, 128, 132, 256])
@pytest.mark.parametrize("heads,N", [(1, 1), (3, 2), (3, 15), (256, 16), (5, 17), (1, 63), (32, 128), (2, 127), (1, 129), (8, 256), (3, 250), (2, 145)])
def test_weights(heads, N, d):
    scale = {"scale": -1.0 / math.sqrt(d)} if d in (36, 132) else {}
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=7600 + N + d, **scale)
    P = gu.to_f64(gu.run_fused(x, guard=4096))
    for h in sorted({0, heads // 2, heads - 1}):
        ref = oracle.attention_weights(x.Q[0, h], x.K[0, h], "f32", x.scale)
        gu.check_weights(P[0, h], ref, "f32", f"fused f32 {heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("N,d", [(37, 20), (128, 64), (200, 256)])
def test_not_finite(N, d):
    """Infinities and NaN give what fp32 arithmetic gives, the rows around them as ever; the first column of K is what lanes past the end of a row read."""
    x = wl.fused_inputs("t", "f32", 1, 3, N, d, seed=7700 + N)
    x.Q[0, 0, :, 0] = np.where(np.arange(N) % 2 == 0, 1.0, -1.0)
    x.K[0, 0, 5, 0] = -np.inf                     # weight 0 for even queries, NaN rows for odd ones
    x.Q[0, 1, 7, d - 1] = np.nan                  # one NaN row
    P = gu.to_f64(gu.run_fused(x, guard=4096))
    for h in range(3):
        with np.errstate(all="ignore"):
            S = float(x.scale) * (x.Q[0, h].astype(np.float64) @ x.K[0, h].astype(np.float64).T)
            E = np.exp(S - S.max(axis=1, keepdims=True))
            ref = E / E.sum(axis=1, keepdims=True)
        assert (np.isnan(P[0, h]) == np.isnan(ref)).all(), f"head {h}"
        ok = np.isfinite(ref)
        assert np.abs(P[0, h][ok] - ref[ok]).max() <= gu.ABS_F32, f"head {h}"
