"""Term 3 (window sums) where its kernels divide the work: one lane to a whole
wave per pixel, 16- and 4-byte loads, row and column tiles with remainders,
strides and dilations, and a patch too large for the tiled form."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import Q, O, dev, assert_equal  # noqa: E402

# N, H, W, C, R, S, stride, pads, dilation
SHAPES = [
    (2, 9, 7, 3, 1, 1, 1, 0, 1),
    (1, 5, 6, 16, 1, 1, 2, 0, 1),
    (3, 1, 300, 1040, 1, 1, 1, 0, 1),
    (2, 11, 13, 20, 3, 3, 1, 1, 1),
    (1, 7, 150, 32, 1, 7, 1, (0, 3, 0, 3), 1),
    (2, 40, 66, 48, 5, 3, 2, (2, 1, 2, 1), 1),
    (64, 33, 33, 16, 3, 3, 1, 1, 1),
    (1, 80, 140, 16, 3, 3, 1, 1, 36),
    (2, 17, 17, 160, 7, 1, 1, (3, 0, 3, 0), 2),
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("xt", ["u8", "i8"])
def test_window_sums(shape, xt):
    N, H, W, C, R, S, stride, pads, dil = shape
    rng = np.random.default_rng(H * W + C)
    lo, hi = (0, 256) if xt == "u8" else (-128, 128)
    x = rng.integers(lo, hi, size=(N, H, W, C)).astype(np.uint8 if xt == "u8" else np.int8)
    K = 5
    w = rng.integers(-4, 5, size=(K, R, S, C)).astype(np.int8)
    zpw = rng.integers(-100, 100, size=K).astype(np.int32)
    zpx = int(rng.integers(lo, hi))
    pads4 = (pads,) * 4 if isinstance(pads, int) else pads
    y = Q.conv2d(dev(x), 0.02, zpx, dev(w), 0.01, zpw, None, stride, pads, dil, 1.0, 0, "i32").cpu().numpy()
    ref = O.conv2d(x, 0.02, zpx, w, np.full(K, 0.01, np.float32), zpw, None, 1.0, 0, "i32",
                   stride=(stride, stride), pads=pads4, dil=(dil, dil))
    assert_equal(y, ref, f"window sums {shape} {xt}")
