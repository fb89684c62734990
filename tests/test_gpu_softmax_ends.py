"""GPU parity of attnw_softmax on rows of a few elements fewer or more than a shape's chunks hold, off the 16-byte boundaries: the ends of a row one to a lane.  Both edges
of the dispatch (five elements fewer in bf16, three in fp32, one a lane more) for every shape, in place and not, rows of the lowest value, a last block of one row."""
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


def _kernel(dtype, cols):
    S = torch.empty((16, cols), device="cuda", dtype=gu.TORCH_DT[dtype])
    P = torch.empty_like(S)
    name, = gu.kernels(lambda stream: attnw.attnw_softmax(S, P, 16, cols, gu.DT[dtype], stream))
    return name


# chunks per lane, lanes per row
@pytest.mark.parametrize("r,lanes", [(2, 64), (3, 64), (2, 128), (3, 128), (2, 256), (3, 256), (4, 256), (6, 256), (2, 1024), (3, 1024), (4, 1024), (6, 1024)])
@pytest.mark.parametrize("dtype,vec", [("bf16", 8), ("f32", 4)])
def test_rows(dtype, vec, r, lanes):
    held = r * vec * lanes
    fewest = held - 5 if dtype == "bf16" else held - 3
    for cols in (fewest, held + lanes - 1):       # the edges themselves: of the kernel with the ends, one element further of another
        assert "softmax_rows_ends" in _kernel(dtype, cols)
    assert "softmax_rows_ends" not in _kernel(dtype, fewest - 1 - (dtype == "f32")) and "softmax_rows_ends" not in _kernel(dtype, held + lanes + 1)
    for i, cols in enumerate((held - 5, fewest, held - 1, held + 1, held + 2, held + lanes - 1)):
        rows, inplace = (13, True) if i % 2 else (9, False)
        s = wl.softmax_inputs("t", dtype, rows, cols, seed=7800 + cols, sigma=2.0, peak_fraction=0.01)
        S = s.S.copy()
        low = np.float32(-3.3895314e38) if dtype == "f32" else np.uint16(0xff7f)
        S[5, :] = low                             # a fully masked row: uniform
        S[rows - 1, : cols // 2] = low
        P = gu.run_softmax(gu.to_dev(S, dtype), rows, cols, dtype, guard=0 if inplace else 4096, inplace=inplace)
        got = gu.to_f64(P)
        gu.check_weights(got, oracle.softmax(S, dtype), dtype, f"softmax {dtype} {rows} x {cols}")
        assert np.abs(got[5] - 1.0 / cols).max() <= (2.0 ** -8 if dtype == "bf16" else 1e-6) / cols
