"""GPU parity of fp32 attention weights and scores on 32-query strips whose scores stay in registers: ends of blocks, of strips and of
the keys that registers hold, every padding of a row, rows off the 16-byte boundaries, strip lists across heads."""
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


# one wave with keys, all of them, a second block, the steps of the registers (256, 512, 1024, 2048 keys) and past them;
# lists of one strip and of several, across heads
SHAPES = [(1, 1, 20), (2, 31, 4), (3, 33, 32), (300, 33, 36), (2, 128, 64), (1, 255, 100), (2, 257, 64), (40, 257, 128), (3, 512, 132),
          (2, 513, 256), (1, 1025, 68), (2, 1024, 128), (9, 1000, 244), (1, 2048, 64), (5, 2047, 32), (1, 2049, 128), (2, 2080, 64),
          (3, 2310, 160), (1, 4100, 32)]


@pytest.mark.parametrize("heads,N,d", SHAPES)
def test_weights(heads, N, d):
    scale = {"scale": -1.0 / math.sqrt(d)} if N % 2 else {}
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=7100 + N + d, **scale)
    P = gu.to_f64(gu.run_fused(x, guard=4096))
    assert np.abs(P.sum(axis=-1) - 1.0).max() <= gu.ROWSUM_F32
    for h in sorted({0, heads // 2, heads - 1}):
        ref = oracle.attention_weights(x.Q[0, h], x.K[0, h], "f32", x.scale)
        gu.check_weights(P[0, h], ref, "f32", f"{heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("heads,N,d", [(1, 1, 20), (3, 33, 32), (40, 257, 128), (3, 512, 132), (300, 50, 64), (1, 1025, 68), (2, 2310, 160)])
def test_scores(heads, N, d):
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=7200 + N + d)
    S = gu.to_f64(gu.run_scores(x, guard=4096))
    for h in sorted({0, heads // 2, heads - 1}):
        q, k = x.Q[0, h].astype(np.float64), x.K[0, h].astype(np.float64)
        # every product and sum in fp32: d roundings of at most the sum of magnitudes
        bound = (d + 2) * 2.0 ** -24 * float(x.scale) * (np.abs(q) @ np.abs(k).T)
        assert (np.abs(S[0, h] - float(x.scale) * (q @ k.T)) <= bound).all(), f"{heads} heads N={N} d={d} head {h}"


@pytest.mark.parametrize("N,d", [(70, 32), (300, 64), (2100, 36)])
def test_not_finite(N, d):
    """Infinities, NaN and values that bf16 rounds to infinity give what fp32 arithmetic gives, the strips around them as ever."""
    heads = 3
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=7300 + N)
    x.Q[0, 0, :, 0] = np.where(np.arange(N) % 2 == 0, 1.0, -1.0)
    x.K[0, 0, 5, 0] = -np.inf                     # weight 0 for even queries, NaN rows for odd ones
    x.Q[0, 1, 7, 1] = np.nan                      # one NaN row
    x.Q[0, 2, :, 3] = 0.0
    x.K[0, 2, 9, 3] = 3.4e38                      # finite, above the largest bf16, and multiplied by zero
    P = gu.to_f64(gu.run_fused(x, guard=4096))
    S = gu.to_f64(gu.run_scores(x, guard=4096))
    for h in range(heads):
        with np.errstate(all="ignore"):
            ref_s = float(x.scale) * (x.Q[0, h].astype(np.float64) @ x.K[0, h].astype(np.float64).T)
            E = np.exp(ref_s - ref_s.max(axis=1, keepdims=True))
            ref = E / E.sum(axis=1, keepdims=True)
        assert (np.isnan(P[0, h]) == np.isnan(ref)).all(), f"head {h}"
        ok = np.isfinite(ref)
        assert np.abs(P[0, h] - ref)[ok].max() <= gu.ABS_F32, f"head {h}"
        fin = np.isfinite(ref_s)
        assert (np.isfinite(S[0, h]) == fin).all() and (np.isnan(S[0, h]) == np.isnan(ref_s)).all(), f"scores, head {h}"
        assert np.abs(S[0, h][fin] - ref_s[fin]).max() <= 1e-5 * np.abs(ref_s[fin]).max(), f"scores, head {h}"


@pytest.mark.parametrize("what", gu.LARGE_SCORES)
@pytest.mark.parametrize("heads,N,d", [(1, 128, 64), (3, 300, 36), (1, 2100, 100)])
def test_large_scores(what, heads, N, d):
    """Scores that fp32 holds and operands times 2^24 do not, with logits of ordinary size."""
    Q, K, scale, rel = gu.large_scores(what, heads, N, d)
    P = gu.to_f64(gu.run_fused(wl.FusedInputs("t", "f32", 1, heads, N, d, scale, Q, K), guard=4096))
    ref = oracle.attention_weights(Q[0, 0], K[0, 0], "f32", scale)
    for h in {0, heads - 1}:
        gu.check_weights(P[0, h], ref, "f32", f"{what}: {heads} heads N={N} d={d} head {h}", abs_f32=2 * rel * ref.max())


@pytest.mark.parametrize("heads,N", [(1, 100), (3, 257), (400, 100), (1, 2049)])
def test_scores_of_four_columns(heads, N):
    """Four products are too few for six of their parts to be as exact as the fp32 instruction: a score that is one product is that
    product, rounded once (2^-24) and once more by the scale (a power of two: not at all)."""
    x = wl.fused_inputs("t", "f32", 1, heads, N, 4, seed=7400 + N, scale=0.5)
    x.Q[...] *= (np.arange(4) == (np.arange(N) % 4)[:, None]).astype(np.float32)
    S = gu.to_f64(gu.run_scores(x, guard=4096))
    for h in sorted({0, heads // 2, heads - 1}):
        ref = 0.5 * (x.Q[0, h].astype(np.float64) @ x.K[0, h].astype(np.float64).T)
        assert (np.abs(S[0, h] - ref) <= 2.0 ** -24 * np.abs(ref)).all(), f"{heads} heads N={N} head {h}"
