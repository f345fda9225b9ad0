"""Standalone requantize at the edges of its 32-bit form: shifts at and just
outside [33, 53], accumulators at the int32 ends and on ties, counts that make
a thread walk several groups with its channel records kept, channel counts
that do and do not allow that."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import Q, O, dev, assert_equal  # noqa: E402

ROUNDINGS = ("half_up", "half_away", "two_stage")


@pytest.mark.parametrize("shift", [32, 33, 34, 52, 53, 54])
@pytest.mark.parametrize("frac", [0.5, 0.75, 0.9999998])
def test_shift_edges(shift, frac):
    s_in = float(np.float32(frac * 2.0 ** (31 - shift)))
    assert Q.quantize_multiplier(s_in)[1] == shift
    rng = np.random.default_rng(shift)
    ends = np.array([-2**31, -2**31 + 1, -1, 0, 1, 2**31 - 2, 2**31 - 1], np.int64)
    step = 2 ** (shift - 31)                       # one output step and its halves: ties
    near = (np.arange(-600, 600)[:, None] * (step // 2) + np.arange(-2, 3)).reshape(-1)
    x = np.concatenate([ends, near, rng.integers(-2**31, 2**31, 5001)])
    x = np.clip(x, -2**31, 2**31 - 1).astype(np.int32)
    for yt, zp in (("u8", 0), ("u8", 255), ("i8", -128), ("i8", 127)):
        for rounding in ROUNDINGS:
            y = Q.requantize(dev(x), s_in, 0, 1.0, zp, yt, None, rounding).cpu().numpy()
            assert_equal(y, O.requantize(x, s_in, 0, 1.0, zp, yt, None, rounding), f"{yt} {zp} {rounding}")


@pytest.mark.parametrize("xt,yt", [("i32", "u8"), ("i32", "i8"), ("u8", "i8"), ("i8", "u8")])
@pytest.mark.parametrize("C", [1, 3, 16, 30, 321, 4999])
def test_channels(xt, yt, C):
    rng = np.random.default_rng(C)
    count = (9 if xt != "i32" else 2) * 2048 * 256 * 4 + 77   # several groups per thread
    shape = (count // C, C)
    lo, hi = {"u8": (0, 256), "i8": (-128, 128), "i32": (-60000, 60000)}[xt]
    x = rng.integers(lo, hi, size=shape).astype({"u8": np.uint8, "i8": np.int8, "i32": np.int32}[xt])
    s_in = (10.0 ** rng.uniform(-0.9, -0.7, size=C) * (1e-3 if xt == "i32" else 1.0)).astype(np.float32)
    zp_in = np.zeros(C, np.int32) if xt == "i32" else rng.integers(lo, hi, size=C).astype(np.int32)
    ylo, yhi = {"u8": (0, 256), "i8": (-128, 128)}[yt]
    zp_out = rng.integers(ylo, yhi, size=C).astype(np.int32)
    for rounding in ROUNDINGS:
        y = Q.requantize(dev(x), s_in, zp_in, 1.0, zp_out, yt, None, rounding).cpu().numpy()
        assert_equal(y, O.requantize(x, s_in, zp_in, np.ones(C, np.float32), zp_out, yt, None, rounding),
                     f"{xt}->{yt} C={C} {rounding}")
