"""GPU parity of the fp32 attention weights on enough strips for the kernel that multiplies operands in three bf16 parts."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2407_13885_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


@pytest.mark.parametrize("d", [4, 32, 36, 64, 100, 128])
@pytest.mark.parametrize("N", [64, 100, 132, 260, 512])
def test_weights_f32_in_three_parts(N, d):
    """Every padding of a row; strips with waves past the end, last tiles of 4 keys, sub-tiles without keys, whole tiles."""
    heads = 128
    scale = {"scale": -1.0 / math.sqrt(d)} if d == 36 else {}
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=6100 + N + d, **scale)
    P = gu.to_f64(gu.run_fused(x, guard=4096))
    assert np.abs(P.sum(axis=-1) - 1.0).max() <= 1e-5
    for h in (0, 1, heads // 2 + 1, heads - 1):
        ref = oracle.attention_weights(x.Q[0, h], x.K[0, h], "f32", x.scale)
        gu.check_weights(P[0, h], ref, "f32", f"fused f32 in parts {heads} heads N={N} d={d} head {h}")


# (the 260 and 512 keys of some head sizes above go to the strips of 32 queries; these do not)
@pytest.mark.parametrize("heads,N,d", [(64, 400, 64), (64, 508, 36), (70, 188, 128), (9, 2996, 128), (10, 3000, 64), (8, 4096, 100)])
def test_weights_f32_in_three_parts_long_sweeps(heads, N, d):
    """Interior tiles and long sweeps of head sizes above 32: 256 to 511 keys up to d = 64, beyond 2048 keys rounds that are full."""
    strips, small = heads * ((N + 127) // 128), heads * ((N + 31) // 32)
    full = -(-small // 256) >= 4 * -(-strips // 256)
    assert 2 * strips >= 256 and (N > 2048 or N < (192 if d > 64 else 512) if full else N < (192 if d > 64 else 256))
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=6400 + N + d)
    P = gu.to_f64(gu.run_fused(x, guard=4096))
    assert np.abs(P.sum(axis=-1) - 1.0).max() <= gu.ROWSUM_F32
    for h in (0, heads - 1):
        ref = oracle.attention_weights(x.Q[0, h], x.K[0, h], "f32", x.scale)
        gu.check_weights(P[0, h], ref, "f32", f"fused f32 in parts {heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("heads", [2, 128])
@pytest.mark.parametrize("what", ["Q and K columns", "scale 2^-70", "scale 2^-90"])
def test_weights_f32_over_the_range_of_fp32(what, heads):
    """Operands of every magnitude that fp32 holds, in three bf16 parts (strips of 32 queries for two heads, of 128 for 128) and, at a
    scale of 2^-90, on the fp32 instruction: as exact as ordinary ones."""
    N, d = 132, 64
    scale = {"Q and K columns": 2.0 ** 20, "scale 2^-70": 2.0 ** -70, "scale 2^-90": 2.0 ** -90}[what]
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=6300 + len(what), scale=scale / math.sqrt(d))
    if what == "Q and K columns":                 # (products of 2^-20: the scale brings them back)
        e = np.linspace(-100, 100, d)
        x.Q[...] *= (2.0 ** e).astype(np.float32)
        x.K[...] *= (2.0 ** (-e - 20)).astype(np.float32)
    else:
        x.Q[...] *= np.float32(scale ** -0.5)
        x.K[...] *= np.float32(scale ** -0.5)
    P = gu.to_f64(gu.run_fused(x, guard=4096))
    for h in sorted({0, heads // 2, heads - 1}):
        ref = oracle.attention_weights(x.Q[0, h], x.K[0, h], "f32", x.scale)
        gu.check_weights(P[0, h], ref, "f32", f"{what}, {heads} heads, head {h}")


def test_weights_f32_in_three_parts_not_finite():
    """Infinities, NaN and values that bf16 rounds to infinity give what fp32 arithmetic gives."""
    heads, N, d = 128, 132, 32
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=6200)
    x.Q[0, 0, :, 0] = np.where(np.arange(N) % 2 == 0, 1.0, -1.0)
    x.K[0, 0, 5, 0] = -np.inf                     # weight 0 for even queries, NaN rows for odd ones
    x.Q[0, 1, 7, 1] = np.nan                      # one NaN row
    x.Q[0, 2, :, 3] = 0.0
    x.K[0, 2, 9, 3] = 3.4e38                      # finite, above the largest bf16, and multiplied by zero
    P = gu.to_f64(gu.run_fused(x, guard=4096))
    for h in range(4):
        with np.errstate(all="ignore"):
            S = float(x.scale) * (x.Q[0, h].astype(np.float64) @ x.K[0, h].astype(np.float64).T)
            E = np.exp(S - S.max(axis=1, keepdims=True))
            ref = E / E.sum(axis=1, keepdims=True)
        assert (np.isnan(P[0, h]) == np.isnan(ref)).all(), f"head {h}"
        ok = np.isfinite(ref)
        assert np.abs(P[0, h] - ref)[ok].max() <= gu.ABS_F32, f"head {h}"


@pytest.mark.parametrize("what", gu.LARGE_SCORES)
@pytest.mark.parametrize("heads,N,d", [(128, 132, 64), (9, 3000, 100)])
def test_weights_f32_in_three_parts_large_scores(what, heads, N, d):
    """Scores that fp32 holds and operands times 2^24 do not, with logits of ordinary size."""
    Q, K, scale, rel = gu.large_scores(what, heads, N, d)
    P = gu.to_f64(gu.run_fused(wl.FusedInputs("t", "f32", 1, heads, N, d, scale, Q, K), guard=4096))
    ref = oracle.attention_weights(Q[0, 0], K[0, 0], "f32", scale)
    for h in {0, heads - 1}:
        gu.check_weights(P[0, h], ref, "f32", f"{what}: {heads} heads N={N} d={d} head {h}", abs_f32=2 * rel * ref.max())
