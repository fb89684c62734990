"""GPU parity of attnw_attention (fp32, d = 36 to 128, many heads) on operands in three bf16 parts where the two waves of a SIMD take turns at the matrix
unit: few tiles of 32 keys, ragged last tiles, waves without queries, scores that climb from tile to tile, waves that start again in fp32."""
import numpy as np
import pytest

import oracle
from paper_2407_13885_amd import workloads as wl

import gpu_util as gu
from test_gpu_attention_general import _check, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


@pytest.mark.parametrize("d", [36, 64, 68, 96, 128])
@pytest.mark.parametrize("N", [129, 160, 161, 191, 193, 224, 256, 257])
def test_tiles(N, d):
    heads = 256
    assert "attention_f32_turns_kernel" in gu.attention_kernels("f32", heads, N, d)[0]
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=5500 + N + d)
    V = wl.value_inputs(x, seed=5501 + N)
    O = gu.to_f64(_run(x, V))
    for h in (0, heads // 2 + 1, heads - 1):
        _check(O[0, h], x, V, 0, h, (0, N), f"{heads} heads of {N} x {d}, head {h}")


# on both sides of the line between this instruction and the fp32 one: more than half of the waves busy and no keys to share, or not
@pytest.mark.parametrize("heads,N,d", [(27, 1187, 20), (26, 1187, 20), (130, 235, 32), (21, 1187, 40), (20, 1187, 64), (64, 257, 100), (56, 257, 100), (14, 1187, 128),
                                       (13, 1187, 68), (9, 2084, 96)])
def test_few_strips(heads, N, d):
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=5800 + N + d)
    V = wl.value_inputs(x, seed=5801 + N)
    O = gu.to_f64(_run(x, V))
    for h in (0, heads - 1):
        for rows in ((0, 40), (max(0, N - 40), N)):
            _check(O[0, h], x, V, 0, h, rows, f"{heads} heads of {N} x {d}, head {h}")


# Keys shared between waves make sums of a quarter of the terms, and every product of the fp32 instruction is whole: 2-norm error 3.7e-7, 4.3e-7 and 6.7e-7 (seven of
# eight values zero: 2.4e-7, 3.0e-7, 3.8e-7) where operands in parts, one sum per output, have 5.6e-7, 5.6e-7 and 1.05e-6 (4.2e-7, 4.0e-7, 7.1e-7).  The bounds lie
# between (geometric mean).
@pytest.mark.parametrize("heads,N,d,dense,sparse", [(27, 1187, 20, 4.6e-7, 3.2e-7), (32, 1111, 56, 4.9e-7, 3.5e-7), (28, 4192, 68, 8.4e-7, 5.2e-7)])
def test_shared_keys_keep_their_precision(heads, N, d, dense, sparse):
    assert "attention_f32_kernel" in gu.attention_kernels("f32", heads, N, d)[0]
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=5900 + N)
    V = wl.value_inputs(x, seed=5901 + N)
    for bound in (dense, sparse):
        if bound == sparse:
            V = V * (np.random.default_rng(N).random(V.shape) < 0.125).astype(np.float32)
        O = gu.to_f64(_run(x, V))
        off = size = 0.0
        for h in (0, heads // 2, heads - 1):
            for rows in ((0, 64), (N - 64, N)):
                ref = oracle.attention_output(x.Q[0, h], x.K[0, h], V[0, h], "f32", x.scale, rows=rows)
                off += np.square(O[0, h, rows[0]:rows[1]] - ref).sum()
                size += np.square(ref).sum()
        assert np.sqrt(off / size) <= bound, f"{heads} heads of {N} x {d}: {np.sqrt(off / size):.2e}"


@pytest.mark.parametrize("N,d", [(161, 64), (250, 100), (200, 128)])
@pytest.mark.parametrize("step", [0.7, 9.0, 200.0])
def test_scores_climb(N, d, step):
    heads = 256
    assert "attention_f32_turns_kernel" in gu.attention_kernels("f32", heads, N, d)[0]
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=5600 + N + d)
    # the last column of K climbs every 32 keys, that of Q is one: the logits of a tile lie `step` above those of the last
    h = heads - 1
    x.Q[0, h, :, d - 1] = 1.0
    x.K[0, h, :, d - 1] = step / float(x.scale) * (np.arange(N) // 32)
    V = wl.value_inputs(x, seed=5601 + N)
    O = gu.to_f64(_run(x, V))
    for g in (0, h):
        _check(O[0, g], x, V, 0, g, (0, N), f"{heads} heads of {N} x {d}, step {step}, head {g}")


@pytest.mark.parametrize("N,d", [(161, 64), (257, 128)])
def test_not_finite(N, d):
    """Infinities, NaN and values that bf16 rounds to infinity give what fp32 arithmetic gives."""
    heads = 256
    assert "attention_f32_turns_kernel" in gu.attention_kernels("f32", heads, N, d)[0]
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=5700 + N)
    V = wl.value_inputs(x, seed=5701)
    x.Q[0, 0, :, 0] = np.where(np.arange(N) % 2 == 0, 1.0, -1.0)
    x.K[0, 0, 5, 0] = -np.inf                     # weight 0 for even queries, NaN rows for odd ones
    V[0, 1, 3, 2] = np.inf                        # a column of infinities
    x.Q[0, 2, 7, 1] = np.nan                      # one NaN row
    # From 2^104 on an operand in parts is NaN.  (A weight is at most 2^8 before it is divided by the row's sum, the exponent following the maximum
    # that far behind: 2^8 x 1e36 is below the largest fp32 number, 3.4e38 in a row this late is not.)
    V[0, 3, N - 1, d - 1] = 1e36
    O = gu.to_f64(_run(x, V))
    for h in range(5):
        with np.errstate(all="ignore"):
            S = float(x.scale) * (x.Q[0, h].astype(np.float64) @ x.K[0, h].astype(np.float64).T)
            E = np.exp(S - S.max(axis=1, keepdims=True))
            ref = (E / E.sum(axis=1, keepdims=True)) @ V[0, h].astype(np.float64)
        assert (np.isnan(O[0, h]) == np.isnan(ref)).all() and (np.isinf(O[0, h]) == np.isinf(ref)).all(), f"head {h}"
        ok = np.isfinite(ref)
        size = np.abs(V[0, h][np.isfinite(V[0, h])]).max()
        # (weights and sums good to a few 2^-24 of sum_j P_ij |V_jt| <= the largest value; scores below 10)
        assert np.abs(O[0, h][ok] - ref[ok]).max() <= 2.0 ** -16 * size, f"head {h}"


@pytest.mark.parametrize("N,d", [(161, 36), (129, 64), (200, 68), (250, 96), (161, 100), (257, 128)])
def test_masked_tail(N, d):
    """A mask through a column of K that operands in parts cannot hold: every wave starts again on the fp32 instruction."""
    heads = 256
    assert "attention_f32_turns_kernel" in gu.attention_kernels("f32", heads, N, d)[0]
    scale = {"scale": -1.0 / np.sqrt(d)} if d == 68 else {}
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=5950 + N + d, **scale)
    V = wl.value_inputs(x, seed=5951)
    x.Q[..., d - 1] = 1.0
    x.K[..., d - 1] = np.where(np.arange(N) >= N - 40, np.float32(-1e20), np.float32(0.0)) * np.sign(x.scale)
    O = gu.to_f64(_run(x, V))
    for h in (0, heads // 2, heads - 1):
        ref = oracle.attention_output(x.Q[0, h], x.K[0, h], V[0, h], "f32", x.scale)
        # (weights and sums good to a few 2^-24 of sum_j P_ij |V_jt| <= the largest value; scores of the keys left below 10)
        assert np.abs(O[0, h] - ref).max() <= 2.0 ** -16 * np.abs(V[0, h]).max(), f"head {h}"
