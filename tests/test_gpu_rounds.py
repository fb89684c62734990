"""GPU parity of attnw_fused on whole tiles (bf16, d = 64 and 128: the round-based kernel, whose sums are taken against the maximum of a
round's first keys) where later scores lie far above those: by some binades, and by more than fp32 sums hold."""
import numpy as np
import pytest

import oracle
from paper_2407_13885_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


def _bf16(a):
    return (np.asarray(a, np.float32).view(np.uint32) >> 16).astype(np.uint16)


def _inputs(BH, N, d, seed):
    """Small noise, the last column of Q one: the last column of K adds to every logit of its key (after the scale)."""
    x = wl.fused_inputs("t", "bf16", 1, BH, N, d, seed=seed)
    x.Q[...] = wl.store(wl.widen(x.Q, "bf16") * 0.25, "bf16")
    x.K[...] = wl.store(wl.widen(x.K, "bf16") * 0.25, "bf16")
    x.Q[..., d - 1] = 0x3f80
    x.K[..., d - 1] = 0
    return x


# 64-query strips of 256-key tiles, 128-query strips with one and two tiles staged, lists of one strip and of several
@pytest.mark.parametrize("BH,N,d", [(3, 512, 64), (40, 1536, 64), (80, 1792, 64), (3, 512, 128), (2, 768, 128), (40, 1024, 128)])
@pytest.mark.parametrize("what", ["climbs", "jumps", "jumps in one head"])
def test_scores_far_above_the_first(BH, N, d, what, monkeypatch):
    x = _inputs(BH, N, d, 6900 + N + d)
    h = BH - 1
    j = np.arange(N)
    if what == "climbs":                          # 60 logits in all
        logits, heads = 60.0 * (j // 32) / (N // 32), slice(None)
    elif what == "jumps":                         # by 290 binades
        logits, heads = np.where(j < N // 2 + 5, 0.0, 201.0), slice(None)
    else:
        logits, heads = np.where(j < N // 2 + 5, 0.0, 201.0), slice(h, h + 1)
    x.K[0, heads, :, d - 1] = _bf16(logits / float(x.scale))
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "rounds")
    got = gu.run_fused(x, guard=8192)[0]
    for head in sorted({0, h}):
        ref = oracle.attention_weights(x.Q[0, head], x.K[0, head], "bf16", x.scale)
        gu.check_weights(gu.to_f64(got[head]), ref, "bf16", f"{BH} heads of {N} x {d}, {what}, head {head}")


def test_a_nan_poisons_its_own_row_only(monkeypatch):
    x = wl.fused_inputs("t", "bf16", 1, 2, 1024, 128, seed=6950)
    x.Q[0, 1, 40, 3] = 0x7fc0
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "rounds")
    got = gu.to_f64(gu.run_fused(x))[0]
    bad = np.isnan(got)
    assert bad[1, 40].all()
    bad[1, 40] = False
    assert not bad.any()


# the second half-wave's first keys lie `units` eighths of a logit above everything that the first half-wave sees before one key of its own
@pytest.mark.parametrize("BH,N,d", [(3, 512, 64), (80, 1792, 64), (3, 512, 128), (2, 768, 128)])
@pytest.mark.parametrize("units", [700, 704, 708])
def test_half_waves_far_apart(BH, N, d, units, monkeypatch):
    """Sums of 2^126 to 2^128 in one half-wave, its exponent 126 binades and more below the other's."""
    x = wl.fused_inputs("t", "bf16", 1, BH, N, d, seed=6960 + N + d, scale=0.125)
    x.Q[...] = wl.store(wl.widen(x.Q, "bf16") * 0.25, "bf16")
    x.K[...] = wl.store(wl.widen(x.K, "bf16") * 0.25, "bf16")
    x.Q[..., d - 1] = 0x3f80
    j = np.arange(N)
    # (keys j % 8 < 4 are the first half-wave's, j % 64 < 32 in a first sub-tile)
    high = (j % 64 == 4) | ((j >= N - 128) & (j % 64 == 33))
    x.K[..., d - 1] = wl.store(np.where(high, np.float32(units), np.float32(0.0)), "bf16")
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "rounds")
    got = gu.run_fused(x, guard=8192)[0]
    for head in sorted({0, BH - 1}):
        ref = oracle.attention_weights(x.Q[0, head], x.K[0, head], "bf16", x.scale)
        gu.check_weights(gu.to_f64(got[head]), ref, "bf16", f"{BH} heads of {N} x {d}, {units}, head {head}")
