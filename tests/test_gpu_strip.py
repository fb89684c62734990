"""GPU parity of attnw_fused / attnw_gemm_scores on 129 to 1280 tokens (bf16: the kernel that shares the keys of 32 queries between
the waves of a workgroup and stages the strip as it lies in memory) against the fp64 oracle: every element of sampled heads at the
bf16 bar, the guard bands around the output, scores bit for bit against the general kernel."""
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


def _check(BH, N, d, monkeypatch, scale=None):
    x = wl.fused_inputs("t", "bf16", 1, BH, N, d, seed=6300 + N + d, scale=scale, row_factor=(0.5, 2.0))
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "strip")
    got = gu.to_f64(gu.run_fused(x, guard=8192))[0]
    S = gu.run_scores(x, guard=8192)
    for h in sorted({0, BH - 1}):
        ref = oracle.attention_weights(x.Q[0, h], x.K[0, h], "bf16", x.scale)
        gu.check_weights(got[h], ref, "bf16", f"{BH} heads of {N} x {d}, head {h}")
    assert np.isfinite(got).all()
    assert np.abs(got.sum(-1) - 1.0).max() <= gu.ROWSUM_BF16
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "twopass")
    S2 = gu.run_scores(x, guard=8192)
    assert torch.equal(S.view(torch.int16), S2.view(torch.int16))


# four waves (up to 640 keys) and eight, with equal and unequal numbers of blocks, last blocks of one key, of 31 and whole, rows on
# and off the 16-byte boundaries (multiples of 16 with padded staging, of 8, of 4, even, odd), last strips of one query
@pytest.mark.parametrize("N", [129, 160, 161, 197, 255, 256, 257, 385, 387, 392, 447, 448, 511, 512, 577, 578, 608, 639, 640, 641, 700, 766,
                               768, 769, 896, 1000, 1023, 1024, 1025, 1151, 1152, 1215, 1217, 1264, 1279, 1280])
def test_lengths(N, monkeypatch):
    _check(3, N, 64, monkeypatch)


# head sizes that fill the steps of the contraction and that are padded to them
@pytest.mark.parametrize("d", [16, 32, 48, 80, 96, 112, 128])
@pytest.mark.parametrize("N", [333, 640, 1025, 1280])
def test_head_sizes(N, d, monkeypatch):
    _check(2, N, d, monkeypatch)


@pytest.mark.parametrize("BH,N,d,scale", [(150, 577, 64, None), (1, 1025, 64, -0.25), (2, 385, 32, 0.0), (90, 401, 128, None)])
def test_many_heads_and_scales(BH, N, d, scale, monkeypatch):
    _check(BH, N, d, monkeypatch, scale)


def test_a_nan_poisons_its_own_row_only(monkeypatch):
    x = wl.fused_inputs("t", "bf16", 1, 2, 577, 80, seed=6002)
    x.Q[0, 1, 40, 3] = 0x7fc0
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "strip")
    got = gu.to_f64(gu.run_fused(x))[0]
    bad = np.isnan(got)
    assert bad[1, 40].all()
    bad[1, 40] = False
    assert not bad.any()


@pytest.mark.parametrize("N,d", [(577, 80), (333, 112), (700, 64)])
def test_an_infinite_key_weighs_nothing(N, d, monkeypatch):
    """-inf in the last column of a key, for every head size that was once padded: weight 0 where the query is positive there, a score of
    -inf, everything else as without the key."""
    x = wl.fused_inputs("t", "bf16", 1, 2, N, d, seed=6350 + N + d)
    x.Q[0, 1, :, d - 1] = 0x3f80                  # 1.0
    x.K[0, 1, 5, d - 1] = 0xff80                  # -inf
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "strip")
    got = gu.to_f64(gu.run_fused(x))[0]
    S = gu.to_f64(gu.run_scores(x))[0]
    assert (got[1, :, 5] == 0.0).all() and np.isneginf(S[1, :, 5]).all()
    rest = np.arange(N) != 5
    ref = oracle.attention_weights(x.Q[0, 1][rest], x.K[0, 1][rest], "bf16", x.scale)
    gu.check_weights(got[1][rest][:, rest], ref, "bf16", f"N={N} d={d}")
    assert np.isfinite(S[1][:, rest]).all() and np.isfinite(got[0]).all() and np.isfinite(S[0]).all()
