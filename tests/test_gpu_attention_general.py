"""GPU parity of attnw_attention on the element types and head sizes that the tiled bf16 kernel does not
take -- fp32 (d a multiple of 4 up to 256) and bf16 with 128 < d <= 256 -- against the fp64 oracle.

bf16: the bar of test_gpu_attention.py (weights rounded to bf16 before they multiply V, the output once more).

fp32: both contractions run on the fp32 matrix instruction and nothing is rounded but in fp32.  With
B_i = |scale| max_j sum_t |q_it| |k_jt| (what the rounding errors of one score are relative to),
A_it = sum_j P_ij |V_jt| and u = 2^-24:
  * a score is a sum of d fp32 products: |scale| |s^ - s| <= d u B_i, which moves every weight by that
    relative amount (numerator), and the normaliser by at most as much;
  * the exponent argument c s - ref is formed with one rounding and c itself is rounded (2 u |c s|, counted
    with the first item since |c s| <= 1.45 B_i), the exponential is good to a few u, the running sum and
    the rescalings by powers of two add N u at worst;
  * the output is a sum of N fp32 products: N u A_it at worst.
Bar: |O - O_ref| <= ((2 d + 4) u B_i + 2^-20 + 2 N u) (A_it + |O_ref|).  (At d = 64, N = 600 and rows
of spread 2 that is about 2e-4 relative -- twenty times tighter than one bf16 rounding.)"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2407_13885_amd as attnw
from paper_2407_13885_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


def _run(x, V, guard=4096):
    Q, K, Vd = gu.to_dev(x.Q, x.dtype), gu.to_dev(x.K, x.dtype), gu.to_dev(V, x.dtype)
    O, canary = gu.empty_like_out((x.B, x.H, x.N, x.d), x.dtype, guard)
    attnw.attnw_attention(Q, K, Vd, O, x.B, x.H, x.N, x.d, float(x.scale), gu.DT[x.dtype])
    torch.cuda.synchronize()
    assert gu.guards_intact(canary), "attention kernel wrote outside O"
    return O


def _check(got, x, V, b, h, rows, what, floor=0.0):
    r0, r1 = rows
    ref, P = oracle.attention_output(x.Q[b, h], x.K[b, h], V[b, h], x.dtype, x.scale, rows=rows, return_weights=True)
    A = P @ np.abs(wl.widen(V[b, h], x.dtype))
    if x.dtype == "bf16":
        tol = 2.0 ** -8 * (A + np.abs(ref)) * 1.02 + 1e-6 * A
    else:
        u = 2.0 ** -24
        Bi = abs(float(np.float32(x.scale))) * (np.abs(wl.widen(x.Q[b, h, r0:r1], "f32")) @ np.abs(wl.widen(x.K[b, h], "f32")).T).max(axis=1)
        tol = ((2 * x.d + 4) * u * Bi[:, None] + 2.0 ** -20 + 2 * x.N * u) * (A + np.abs(ref)) + floor
    err = np.abs(got[r0:r1] - ref)
    assert np.isfinite(got[r0:r1]).all(), f"{what}: non-finite output"
    if (err > tol).any():
        i = np.unravel_index(np.argmax(err / tol), err.shape)
        raise AssertionError(f"{what} rows {r0}..{r1}: {int((err > tol).sum())} elements beyond the bound; worst at {i}: "
                             f"got {got[r0:r1][i]:.8e} ref {ref[i]:.8e} err {err[i]:.3e} tol {tol[i]:.3e}")


@pytest.mark.parametrize("d", [4, 8, 12, 20, 32, 36, 64, 100, 128, 132, 200, 256])
@pytest.mark.parametrize("N", [1, 31, 32, 33, 100, 257, 600])
def test_attention_f32(N, d):
    x = wl.fused_inputs("t", "f32", 1, 2, N, d, seed=3100 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=3101 + N)
    O = gu.to_f64(_run(x, V))
    for h in range(2):
        _check(O[0, h], x, V, 0, h, (0, N), f"fp32 attention N={N} d={d} head {h}")


@pytest.mark.parametrize("d", [144, 160, 192, 208, 256])
@pytest.mark.parametrize("N", [1, 33, 128, 257, 600])
def test_attention_bf16_large_heads(N, d):
    x = wl.fused_inputs("t", "bf16", 1, 2, N, d, seed=3300 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=3301 + N)
    O = gu.to_f64(_run(x, V))
    for h in range(2):
        _check(O[0, h], x, V, 0, h, (0, N), f"bf16 attention N={N} d={d} head {h}")


@pytest.mark.parametrize("dtype,B,H,N,d", [("f32", 2, 3, 2048, 64), ("f32", 1, 2, 1500, 128), ("f32", 1, 1, 1024, 256),
                                           ("bf16", 2, 2, 2048, 256), ("bf16", 1, 3, 1500, 160)])
def test_attention_general_long(dtype, B, H, N, d):
    """Many sub-tiles per wave, several heads and batches (addressing of the heads), sampled row ranges."""
    x = wl.fused_inputs("t", dtype, B, H, N, d, seed=3500 + H + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=3501 + N)
    O = gu.to_f64(_run(x, V))
    assert np.isfinite(O).all()
    for b in range(B):
        for h in range(H):
            for rows in [(0, 40), (N // 2 - 3, N // 2 + 30), (N - 40, N)]:
                _check(O[b, h], x, V, b, h, rows, f"{dtype} attention {B}x{H}x{N}x{d} head ({b},{h})")


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 20), ("bf16", 192)])
def test_attention_general_negative_and_zero_scale_constant_values(dtype, d):
    N = 333
    x = wl.fused_inputs("t", dtype, 1, 2, N, d, seed=3700 + d, scale=-1.0 / math.sqrt(d), row_factor=(0.5, 3.0))
    V = wl.value_inputs(x, seed=3701 + d)
    O = gu.to_f64(_run(x, V))
    for h in range(2):
        _check(O[0, h], x, V, 0, h, (0, N), f"{dtype} negative scale d={d} head {h}")
    Vw = wl.widen(V[0, 0], dtype)
    one = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -20
    # scale 0: uniform weights, every output row is the column mean of V
    x0 = wl.fused_inputs("t", dtype, 1, 2, N, d, seed=3700 + d, scale=0.0)
    O0 = gu.to_f64(_run(x0, V))
    assert np.abs(O0[0, 0] - Vw.mean(axis=0)).max() <= one * np.abs(Vw).mean(axis=0).max() + 1e-7
    # constant V rows: every output row equals that row (weights sum to 1, up to their rounding)
    Vc = np.broadcast_to(V[:, :, :1, :], V.shape).copy()
    Oc = gu.to_f64(_run(x, Vc))
    v = wl.widen(Vc[0, 1, 0], dtype)
    assert np.abs(Oc[0, 1] - v).max() <= 2 * one * np.abs(v).max()


def test_attention_f32_scores_climbing_along_the_keys():
    """Every sub-tile brings a new row maximum: the reference exponent moves and the accumulators are rescaled."""
    N, d = 1024, 32
    x = wl.fused_inputs("t", "f32", 1, 2, N, d, seed=97)
    a = 4.0
    for step in (0.02, 0.4):
        Kw = wl.widen(x.K, "f32") * 0.05
        Kw[..., 0] = (np.arange(N, dtype=np.float64) * step / (a * float(x.scale)))[None, None, :]
        Qw = wl.widen(x.Q, "f32") * 0.05
        Qw[..., 0] = a
        Qw[0, 1, ::2, 0] = -a
        x.Q[...] = wl.store(Qw, "f32")
        x.K[...] = wl.store(Kw, "f32")
        V = wl.value_inputs(x, seed=98)
        O = gu.to_f64(_run(x, V))
        for h in range(2):
            _check(O[0, h], x, V, 0, h, (0, N), f"fp32 climbing scores step={step} head {h}")


def test_attention_general_is_deterministic():
    x = wl.fused_inputs("t", "f32", 1, 2, 300, 36, seed=6)
    V = wl.value_inputs(x, seed=7)
    a, b = _run(x, V, guard=64), _run(x, V, guard=64)
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("d", [4, 36, 64, 96, 128, 256])
@pytest.mark.parametrize("N", [1, 100, 129])
def test_attention_f32_many_heads(N, d):
    """Enough heads that every wave takes all keys (fewer heads share the keys of a query block between the waves of a
    workgroup): one key, 128-query workgroups with a wave that is not full (N = 100, and 129 with d = 256), operands in three bf16
    parts (N = 129 up to d = 128)."""
    heads = 512
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=3900 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=3901 + N)
    O = gu.to_f64(_run(x, V))
    assert np.isfinite(O).all()
    for h in (0, 1, heads // 2 + 1, heads - 1):
        _check(O[0, h], x, V, 0, h, (0, N), f"fp32 attention {heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("d", [4, 32, 36, 64, 100, 128])
def test_attention_f32_several_strips_of_all_keys(d):
    """Forty heads of 700 keys: several 128-query workgroups per head on the fp32 instruction (too few 256-query strips for operands in
    parts), the last with a wave of 28 queries and waves past the end."""
    heads, N = 40, 700
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=4000 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=4001 + N)
    O = gu.to_f64(_run(x, V))
    assert np.isfinite(O).all()
    for h in (0, heads // 2 + 1, heads - 1):
        _check(O[0, h], x, V, 0, h, (0, N), f"fp32 attention {heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("d", [144, 160, 176, 192, 208, 224, 240, 256])
@pytest.mark.parametrize("N", [65, 129, 256, 257])
def test_attention_bf16_large_heads_many(N, d):
    """Enough heads that a wave takes all keys (fewer share the keys of a query block between four waves): every padding of
    a row, a last tile of one key, waves and strips past the end."""
    heads = 300
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=4100 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=4101 + N)
    O = gu.to_f64(_run(x, V))
    assert np.isfinite(O).all()
    for h in (0, 1, heads // 2 + 1, heads - 1):
        _check(O[0, h], x, V, 0, h, (0, N), f"bf16 attention {heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("d", [4, 32, 36, 64, 100, 128])
@pytest.mark.parametrize("N", [257, 600])
def test_attention_f32_in_three_parts(N, d):
    """Enough heads for the kernel that multiplies operands in three bf16 parts: every padding of a row, last tiles of one
    key and of 24, waves past the end; rows of scores of both signs of the scale."""
    heads = 256
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=4300 + N + d, row_factor=(0.5, 2.0),
                        **({"scale": -1.0 / math.sqrt(d)} if d == 36 else {}))
    V = wl.value_inputs(x, seed=4301 + N)
    O = gu.to_f64(_run(x, V))
    assert np.isfinite(O).all()
    for h in (0, 1, heads // 2 + 1, heads - 1):
        _check(O[0, h], x, V, 0, h, (0, N), f"fp32 attention in parts {heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("heads", [2, 256])
@pytest.mark.parametrize("what", ["V", "V columns", "V rows", "Q and K columns", "tiny weights", "scale 2^-70", "scale 2^-90"])
def test_attention_f32_over_the_range_of_fp32(what, heads):
    """Operands of every magnitude that fp32 holds, on the fp32 instruction (two heads) and in three bf16 parts (256): the same
    bound, relative to sum_j P_ij |V_jt|, with the spacing of fp32's smallest numbers per product as a floor."""
    N, d = 257, 4 if what == "tiny weights" else 64
    scale = {"Q and K columns": 2.0 ** 20, "scale 2^-70": 2.0 ** -70, "scale 2^-90": 2.0 ** -90}.get(what, 1.0)
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=4500 + len(what), scale=scale / math.sqrt(d))
    V = wl.value_inputs(x, seed=4501)
    if what == "V":
        V *= np.float32(2.0 ** -124)
    elif what == "V columns":
        V *= (2.0 ** -np.linspace(0, 125, d)).astype(np.float32)
    elif what == "V rows":
        V *= (2.0 ** -(np.arange(N) % 125.0)).astype(np.float32)[:, None]
    elif what == "Q and K columns":               # (products of 2^-20: the scale brings them back)
        e = np.linspace(-100, 100, d)
        x.Q[...] *= (2.0 ** e).astype(np.float32)
        x.K[...] *= (2.0 ** (-e - 20)).astype(np.float32)
    elif what == "tiny weights":                  # the only key with a value weighs 2^-124: scores -86, the others near 0
        x.Q[...] *= np.float32(0.01)
        x.Q[..., 0] = 2.0
        x.K[..., 0] = 0.0
        x.K[..., 100, 0] = -86.0
        V[...] = 0.0
        V[..., 100, :] = 256.0 + np.arange(d) / 7.0
    else:
        x.Q[...] *= np.float32(scale ** -0.5)
        x.K[...] *= np.float32(scale ** -0.5)
    O = gu.to_f64(_run(x, V))
    for h in sorted({0, heads // 2, heads - 1}):
        _check(O[0, h], x, V, 0, h, (0, N), f"{what}, {heads} heads, head {h}", floor=N * 2.0 ** -149)


def test_attention_f32_in_three_parts_not_finite():
    """Infinities, NaN and values that bf16 rounds to infinity give what fp32 arithmetic gives."""
    heads, N, d = 256, 257, 32
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=4400)
    V = wl.value_inputs(x, seed=4401)
    x.Q[0, 0, :, 0] = np.where(np.arange(N) % 2 == 0, 1.0, -1.0)
    x.K[0, 0, 5, 0] = -np.inf                     # weight 0 for even queries, NaN rows for odd ones
    V[0, 1, 3, 2] = np.inf                        # a column of infinities
    x.Q[0, 2, 7, 1] = np.nan                      # one NaN row
    V[0, 3, 9, 4] = 3.4e38                        # finite, and above the largest bf16
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
        assert np.abs(O[0, h] - ref)[ok].max() <= 2.0 ** -16 * size, f"head {h}"


@pytest.mark.parametrize("heads,N,d", [(2, 100, 36), (2, 600, 36), (2, 600, 200), (300, 20, 20), (300, 50, 132), (512, 100, 100), (256, 257, 36)])
def test_attention_f32_infinite_key(heads, N, d):
    """A key with -inf in the first chunk of a row that is padded on chip: weight 0 for the queries that meet it with a positive
    number, NaN rows for those with a negative one, as in fp32 arithmetic.  On every shape of workgroup."""
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=4600 + N + d)
    V = wl.value_inputs(x, seed=4601)
    h = heads - 1
    x.Q[0, h, :, 0] = np.where(np.arange(N) % 2 == 0, 1.0, -1.0)
    x.K[0, h, 5, 0] = -np.inf
    O = gu.to_f64(_run(x, V))
    assert np.isfinite(O[0, :h]).all()
    assert np.isnan(O[0, h, 1::2]).all()
    Q, K = x.Q[0, h, ::2].astype(np.float64), np.delete(x.K[0, h].astype(np.float64), 5, axis=0)
    W = np.delete(V[0, h].astype(np.float64), 5, axis=0)
    S = float(x.scale) * (Q @ K.T)
    E = np.exp(S - S.max(axis=1, keepdims=True))
    P = E / E.sum(axis=1, keepdims=True)
    ref, u = P @ W, 2.0 ** -24
    B = abs(float(x.scale)) * (np.abs(Q) @ np.abs(K).T).max(axis=1)
    tol = ((2 * d + 4) * u * B[:, None] + 2.0 ** -20 + 2 * N * u) * (P @ np.abs(W) + np.abs(ref))
    assert (np.abs(O[0, h, ::2] - ref) <= tol).all()


@pytest.mark.parametrize("heads,N,d", [(256, 257, 36), (256, 257, 64), (256, 600, 32)])
def test_attention_f32_in_three_parts_infinite_last_value(heads, N, d):
    """An infinity in the last row of V, which the rows past the end of a last tile are read as: that column is infinite in every
    row of the head, nothing else changes."""
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=4700 + N + d)
    V = wl.value_inputs(x, seed=4701)
    h = heads - 1
    V[0, h, N - 1, 2] = np.inf
    O = gu.to_f64(_run(x, V))
    assert (O[0, h, :, 2] == np.inf).all()
    V[0, h, N - 1, 2] = O[0, h, :, 2] = 0.0
    ref = oracle.attention_output(x.Q[0, h], x.K[0, h], V[0, h], "f32", x.scale, rows=(0, N))
    ref[:, 2] = 0.0
    # (as in the bound above: d and N enough for B below 16)
    assert np.abs(O[0, h] - ref).max() <= ((2 * d + 4) * 16 + 2 * N + 16) * 2.0 ** -24 * 2 * np.abs(V[0, h]).max()
    assert np.isfinite(O[0, :h]).all()


@pytest.mark.parametrize("d", [144, 160, 176, 192, 208, 224, 240, 256])
@pytest.mark.parametrize("heads,N", [(3, 1), (3, 17), (3, 31), (600, 32), (300, 33), (300, 49), (300, 64)])
def test_attention_bf16_large_heads_of_one_or_two_query_blocks(heads, N, d):
    """One query block per head: a wave without LDS.  Two query blocks and enough heads: workgroups of two waves."""
    x = wl.fused_inputs("t", "bf16", 1, heads, N, d, seed=4800 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=4801 + N)
    O = gu.to_f64(_run(x, V))
    for h in (0, 1, heads // 2 + 1, heads - 1):
        _check(O[0, h], x, V, 0, h, (0, N), f"bf16 attention {heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("d", [132, 160, 164, 196, 224, 228, 256])
@pytest.mark.parametrize("heads,N", [(1, 1), (5, 17), (5, 31), (600, 32)])
def test_attention_f32_large_heads_of_one_query_block(heads, N, d):
    """A wave per head without LDS: every padding of a row, rows past the end; both signs of the scale."""
    scale = {"scale": -1.0 / math.sqrt(d)} if N == 17 else {}
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=4900 + N + d, row_factor=(0.5, 2.0), **scale)
    V = wl.value_inputs(x, seed=4901 + N)
    O = gu.to_f64(_run(x, V))
    for h in sorted({0, heads // 2, heads - 1}):
        _check(O[0, h], x, V, 0, h, (0, N), f"fp32 attention {heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("d", [4, 36, 64, 100, 128])
@pytest.mark.parametrize("heads,N", [(300, 33), (300, 64), (300, 65), (300, 96), (300, 129), (300, 160)])
def test_attention_f32_one_wave_workgroups_of_a_few_blocks(heads, N, d):
    """More heads than compute units, each of two, three or five query blocks: a workgroup per block, the last of one query or full."""
    x = wl.fused_inputs("t", "f32", 1, heads, N, d, seed=5000 + N + d, row_factor=(0.5, 2.0))
    V = wl.value_inputs(x, seed=5001 + N)
    O = gu.to_f64(_run(x, V))
    for h in (0, heads // 2 + 1, heads - 1):
        _check(O[0, h], x, V, 0, h, (0, N), f"fp32 attention {heads} heads N={N} d={d} head {h}")


@pytest.mark.parametrize("what", gu.LARGE_SCORES)
@pytest.mark.parametrize("heads,N,d", [(2, 257, 64), (256, 257, 64), (256, 200, 128)])
def test_attention_f32_large_scores(what, heads, N, d):
    """Scores that fp32 holds and operands times 2^24 do not, with logits of ordinary size, on the fp32 instruction (two heads) and in
    three bf16 parts."""
    Q, K, scale, rel = gu.large_scores(what, heads, N, d)
    x = wl.FusedInputs("t", "f32", 1, heads, N, d, scale, Q, K)
    V = wl.value_inputs(x, seed=4901)
    O = gu.to_f64(_run(x, V))
    for h in {0, heads - 1}:
        ref = oracle.attention_output(Q[0, h], K[0, h], V[0, h], "f32", scale, rows=(0, N))
        # weights off by `rel` relative to each other, sums of N products
        assert np.abs(O[0, h] - ref).max() <= (2 * rel + (N + 8) * 2.0 ** -24) * np.abs(V[0, h]).max(), f"{what}, {heads} heads, head {h}"


@pytest.mark.parametrize("q,k", [(20, 52), (52, 20), (21, 52), (20, 53), (53, 20)])
@pytest.mark.parametrize("d", [32, 64, 96, 128])
def test_attention_f32_operands_at_the_limits_of_parts(d, q, k):
    """|Q| and |K| at 2^20 and 2^52, up to which no score in three bf16 parts overflows, and beyond, where the fp32 instruction takes over:
    only one key is so large, in the last tile, and its score of up to -2^80 must leave its weight."""
    N, heads = 200, 256
    Q = np.full((1, heads, N, d), 2.0 ** q, np.float32)
    K = np.full((1, heads, N, d), -2.0 ** (k - 1), np.float32)
    K[0, :, 197] *= 2.0 * (1.0 - 2.0 ** -8)
    scale = np.float32(4.0 / d * 2.0 ** -(q + k))  # logits of -2 and about -4, every product and sum exact
    x = wl.FusedInputs("t", "f32", 1, heads, N, d, scale, Q, K)
    V = wl.value_inputs(x, seed=4907)
    V[0, :, 197] = 1000.0                         # (a weight of e^-2 / 200 in a sum of some 1)
    O = gu.to_f64(_run(x, V))
    for h in (0, heads - 1):
        ref = oracle.attention_output(Q[0, h], K[0, h], V[0, h], "f32", scale, rows=(0, N))
        # weights as in the test above (exponents below 15), sums of N products
        assert np.abs(O[0, h] - ref).max() <= (2 * 3 * 15 * 2.0 ** -24 + (N + 8) * 2.0 ** -24) * np.abs(V[0, h]).max(), f"d={d} head {h}"
