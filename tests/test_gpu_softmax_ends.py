"""GPU parity of attnw_softmax on rows of a few elements fewer or more than a shape's chunks hold, off the 16-byte boundaries: the ends of a row one to a lane.  Both edges
of the dispatch (five elements fewer, one a lane more) for every shape, in place and not, rows of the lowest value, a last block of one row."""
import numpy as np
import pytest

import oracle
from paper_2407_13885_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    gu.require_gpu()


# chunks per lane, lanes per row
@pytest.mark.parametrize("r,lanes", [(2, 64), (3, 64), (2, 128), (3, 128), (2, 256), (3, 256), (4, 256), (6, 256), (2, 1024), (3, 1024), (4, 1024), (6, 1024)])
@pytest.mark.parametrize("dtype,vec", [("bf16", 8), ("f32", 4)])
def test_rows(dtype, vec, r, lanes):
    held = r * vec * lanes
    for i, cols in enumerate((held - 5, held - 1, held + 1, held + 2, held + lanes - 1)):
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
