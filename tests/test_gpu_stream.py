"""GPU parity of attnw_fused / attnw_gemm_scores on more than 512 tokens (bf16: the persistent kernel whose waves share the keys of 32
queries) against the fp64 oracle: every element of sampled heads at the bf16 bar, the guard bands around the output, scores bit for bit
against the general kernel."""
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


def _check(BH, N, d, monkeypatch, scale=None, factors=(0.5, 2.0), kernel="stream"):
    x = wl.fused_inputs("t", "bf16", 1, BH, N, d, seed=6700 + N + d, scale=scale, row_factor=factors)
    if kernel is None:
        monkeypatch.delenv("ATTNW_FUSED_KERNEL", raising=False)
    else:
        monkeypatch.setenv("ATTNW_FUSED_KERNEL", kernel)
    P = gu.run_fused(x, guard=8192)[0]
    S = gu.run_scores(x, guard=8192)
    assert torch.isfinite(P).all()
    assert float((P.double().sum(-1) - 1.0).abs().max()) <= gu.ROWSUM_BF16
    for h in sorted({0, BH - 1}):
        ref = oracle.attention_weights(x.Q[0, h], x.K[0, h], "bf16", x.scale)
        gu.check_weights(gu.to_f64(P[h]), ref, "bf16", f"{BH} heads of {N} x {d}, head {h}")
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "twopass")
    S2 = gu.run_scores(x, guard=8192)
    assert torch.equal(S.view(torch.int16), S2.view(torch.int16))


# two windows and a key more, windows cut off after one key, after one block and one key before a whole one, rows on 16-byte boundaries,
# even and odd ones; d = 64: 16 waves and windows of 512 keys, d = 128: eight and 256, six of them (five off the boundaries) held
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [513, 520, 767, 768, 769, 1023, 1024, 1025, 1281, 1537, 1544, 1790, 1793, 2049, 2080])
def test_lengths(N, d, monkeypatch):
    _check(2, N, d, monkeypatch)


# every number of contraction steps: pieces of one to four, whole and overlapping, one to four of a block
@pytest.mark.parametrize("d", range(16, 257, 16))
@pytest.mark.parametrize("N", [1100, 1801])
def test_head_sizes(N, d, monkeypatch):
    _check(1, N, d, monkeypatch)


# several strips per workgroup, across heads; sharp rows, whose reference exponent moves; scales of both signs and none
@pytest.mark.parametrize("BH,N,d,scale,factors", [(40, 600, 32, None, (0.5, 2.0)), (33, 777, 96, None, (0.5, 3.0)), (20, 1030, 144, None, (0.5, 3.0)), (30, 1025, 64, None, (0.5, 2.0)), (70, 513, 48, None, (0.5, 2.0)),
                                                  (2, 700, 64, -0.25, (0.5, 2.0)), (2, 1500, 80, 0.0, (0.5, 2.0)),
                                                  (1, 1667, 128, 3.0, (0.5, 2.0)), (1, 4100, 16, 2.0, (1.0, 3.0))])
def test_many_strips_and_scales(BH, N, d, scale, factors, monkeypatch):
    _check(BH, N, d, monkeypatch, scale, factors)


# calls that take the kernel without being asked to
@pytest.mark.parametrize("BH,N,d", [(2, 1283, 64), (8, 1659, 128), (1, 2100, 208), (24, 641, 256), (3, 1536, 32), (20, 608, 96)])
def test_calls_of_its_own(BH, N, d, monkeypatch):
    _check(BH, N, d, monkeypatch, kernel=None)


def test_a_nan_poisons_its_own_row_only(monkeypatch):
    x = wl.fused_inputs("t", "bf16", 1, 2, 1301, 80, seed=6002)
    x.Q[0, 1, 40, 3] = 0x7fc0
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "stream")
    got = gu.to_f64(gu.run_fused(x))[0]
    bad = np.isnan(got)
    assert bad[1, 40].all()
    bad[1, 40] = False
    assert not bad.any()


# the first keys that a lane sees weigh nothing: its reference exponent comes from later ones
@pytest.mark.parametrize("N,d", [(1301, 80), (700, 64), (1792, 208)])
def test_infinite_keys_weigh_nothing(N, d, monkeypatch):
    x = wl.fused_inputs("t", "bf16", 1, 2, N, d, seed=6750 + N + d)
    x.Q[0, 1, :, d - 1] = 0x3f80                  # 1.0
    gone = np.zeros(N, bool)
    gone[5] = True
    gone[32:96] = True
    x.K[0, 1, gone, d - 1] = 0xff80               # -inf
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "stream")
    got = gu.to_f64(gu.run_fused(x))[0]
    S = gu.to_f64(gu.run_scores(x))[0]
    assert (got[1][:, gone] == 0.0).all() and np.isneginf(S[1][:, gone]).all()
    rest = ~gone
    ref = oracle.attention_weights(x.Q[0, 1][rest], x.K[0, 1][rest], "bf16", x.scale)
    gu.check_weights(got[1][rest][:, rest], ref, "bf16", f"N={N} d={d}")
    assert np.isfinite(S[1][:, ~gone]).all() and np.isfinite(got[0]).all() and np.isfinite(S[0]).all()


# windows held in registers, all of them; N = 1536: workgroups start at different ones
@pytest.mark.parametrize("N,d", [(1100, 128), (1536, 128), (1280, 96)])
def test_exponents_of_a_million(N, d, monkeypatch):
    """Exponents of 1.5 million (an ulp is an eighth): keys of the same score weigh the same, whether their block moved the reference or not."""
    x = wl.fused_inputs("t", "bf16", 1, 4, N, d, seed=6800 + N + d, scale=0.125)
    x.Q[...] = 0
    x.Q[..., d - 2:] = 0x3f80
    x.K[..., d - 2] = wl.store(np.float32(2.0 ** 23), "bf16")
    x.K[..., d - 1] = 0
    block = np.arange(N) // 32
    for h in range(4):
        # (one wave of eight has these blocks)
        x.K[0, h, (block == 11) | (block == 19), d - 1] = wl.store(np.float32(81 + 11 * h), "bf16")
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "stream")
    got = gu.to_f64(gu.run_fused(x))[0]
    for h in range(4):
        ref = oracle.attention_weights(x.Q[0, h], x.K[0, h], "bf16", x.scale)
        gu.check_weights(got[h], ref, "bf16", f"N={N} d={d} head {h}")


# K of a head beyond 8 MiB (scores 6), more strips per compute unit than the heads' K in L2 bears, and the last shape in front of each line
@pytest.mark.parametrize("BH,N,d,taken", [(1, 32776, 128, False), (128, 1544, 64, False), (104, 1544, 64, True), (34, 4104, 128, False), (19, 4104, 128, True), (30, 3080, 176, False),
                                          (300, 2056, 32, False),
                                          (1, 17152, 112, False), (1, 17160, 128, True), (1, 16640, 224, False), (1, 16384, 224, True), (1, 20000, 176, False)])
def test_where_the_other_kernels_are_faster(BH, N, d, taken, monkeypatch):
    """Weights of these are those of one kernel, bit for bit, and not of the other (2.1 to 1.05 times as fast here)."""
    out = {}
    Q = torch.randn((BH, N, d), device="cuda", generator=torch.Generator("cuda").manual_seed(6890)).bfloat16()
    K = torch.randn((BH, N, d), device="cuda", generator=torch.Generator("cuda").manual_seed(6891)).bfloat16()
    for kernel in (None, "stream", "rounds"):
        monkeypatch.delenv("ATTNW_FUSED_KERNEL", raising=False)
        if kernel is not None:
            monkeypatch.setenv("ATTNW_FUSED_KERNEL", kernel)
        out[kernel] = torch.empty((BH, N, N), device="cuda", dtype=torch.bfloat16)
        attnw.attnw_fused(Q, K, out[kernel], 1, BH, N, d, d ** -0.5, attnw.ATTNW_BF16)
    torch.cuda.synchronize()
    same = {kernel: torch.equal(out[None].view(torch.int16), out[kernel].view(torch.int16)) for kernel in ("stream", "rounds")}
    assert same == {"stream": taken, "rounds": not taken}


# one wave's blocks in three windows held in registers: 1, 2^14.9 and 2^134.9 against the first
@pytest.mark.parametrize("N,d", [(1100, 128), (1536, 96), (1280, 208)])
def test_weights_far_below_a_later_key(N, d, monkeypatch):
    """Weights of 2^-120, whose block was taken against a reference that then moves by 135 binades (a factor of 2^-127 and less is 0)."""
    x = wl.fused_inputs("t", "bf16", 1, 2, N, d, seed=6810 + N + d, scale=0.125)
    x.Q[...] = 0
    x.Q[..., d - 1] = 0x3f80
    x.K[..., d - 1] = 0
    for window, units in ((1, 82.5), (2, 748.0)):
        x.K[0, :, (window * 8 + 3) * 32, d - 1] = wl.store(np.float32(units), "bf16")
    monkeypatch.setenv("ATTNW_FUSED_KERNEL", "stream")
    got = gu.to_f64(gu.run_fused(x))[0]
    for h in range(2):
        ref = oracle.attention_weights(x.Q[0, h], x.K[0, h], "bf16", x.scale)
        gu.check_weights(got[h], ref, "bf16", f"N={N} d={d} head {h}")
