"""3x3 average pooling at stride 1 with 16 channels per thread, one and four
output rows per thread, byte for byte against the oracle: every window cut by
an edge, rows that are no multiple of four, both types and roundings, counted
padding, and values that make ties and both ends of the range."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import Q, O, dev, assert_equal  # noqa: E402

# 65536 or more 16-channel outputs take this kernel; 131072 or more threads of four rows the second form
SHAPES = [(64, 33, 2, 256), (64, 3, 22, 256), (8, 13, 64, 1024), (9, 30, 64, 256), (700, 1, 6, 256)]


@pytest.mark.parametrize("dt", ["u8", "i8"])
@pytest.mark.parametrize("rounding", ["half_up", "half_away"])
@pytest.mark.parametrize("shape", SHAPES)
def test_avg3(dt, rounding, shape):
    rng = np.random.default_rng(shape[1])
    lo, hi = O.DTYPE_RANGE[dt]
    kinds = [rng.integers(lo, hi + 1, size=shape), rng.choice([lo, hi], size=shape),
             rng.integers((lo + hi) // 2 - 1, (lo + hi) // 2 + 3, size=shape)]
    for i, x in enumerate(kinds):
        x = x.astype(O.NAME_TO_NP[dt])
        for pads in ((1, 1, 1, 1), (2, 1, 2, 2), (1, 2, 1, 0)):
            if shape[1] + pads[0] + pads[2] < 3 or shape[2] + pads[1] + pads[3] < 3:
                continue
            for count_pad in (False, True):
                zp = int(rng.integers(lo, hi + 1))
                y = Q.pool2d(dev(x), "avg", (3, 3), (1, 1), pads, count_pad, zp, rounding)
                want = O.pool2d(x, "avg", (3, 3), (1, 1), pads, count_pad, zp, rounding)
                assert_equal(y.cpu().numpy(), want, f"avg3 {dt} {rounding} {shape} {pads} {count_pad} kind {i}")
