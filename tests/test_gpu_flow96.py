"""The 96-channel tiles of the short-loop conv kernel, whose last waves load
two row blocks twice: channel counts of one tile, of several, and ending inside
one; linear and tabulated taps; term 3, int32 output, a fused add; and counts
for which they are not offered."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import Q, O, dev, env, make_plan, run_gpu, run_oracle, assert_equal  # noqa: E402

L = W.ConvLayer
SHAPES = [
    (L("1x1", 9, 9, 64, 96, 1, 1), 5, {}),
    (L("1x1c16", 13, 7, 16, 192, 1, 1), 3, dict(x_dtype="i8", yt="i8")),
    (L("1x1c100", 11, 9, 100, 260, 1, 1, 2), 2, {}),
    (L("3x3", 23, 21, 64, 96, 3, 3, 1, (1, 1, 1, 1)), 2, {}),
    (L("3x3z", 12, 13, 48, 70, 3, 3, 1, (1, 1, 1, 1)), 1, dict(zp_w="channel")),
    (L("3x3i32", 16, 15, 128, 288, 3, 3, 2, (0, 0, 1, 1)), 3, dict(yt="i32")),
    (L("5x5c36", 9, 9, 36, 80, 5, 5, 1, (2, 2, 2, 2)), 2, dict(rounding="two_stage")),
]


@pytest.mark.parametrize("tile", [19, 20, 21, 22])
def test_tiles_of_96_channels(tile):
    ran = 0
    for i, (layer, N, kw) in enumerate(SHAPES):
        c = W.conv_case(layer, N, seed=1500 + i, **kw)
        with env(QNN_FLOW=tile):
            p, keep = make_plan(c)
            d = p.describe()
            p.close()
            if "cands=1 " not in d + " ":
                continue   # a short form with fewer stages
            ran += 1
            assert "tile=96x" in d, d
            assert_equal(run_gpu(c), run_oracle(c), f"flow {tile} {layer.name}: {d}")
    assert ran >= 2


@pytest.mark.parametrize("tile", [19, 20, 21])
def test_fused_add_96(tile):
    c = W.conv_case(L("f", 12, 13, 64, 96, 1, 1), 3, seed=31, yt="i8")
    mid = run_oracle(c)
    with env(QNN_FLOW=tile):
        p, keep = make_plan(c)
    assert "tile=96x" in p.describe(), p.describe()
    r = np.random.default_rng(tile).integers(0, 256, size=mid.shape).astype(np.uint8)
    p.set_residual("u8", 0.031, 7, 0.047, -3, "i8")
    y = p.run(dev(c.x), residual=dev(r)).cpu().numpy()
    p.close()
    assert_equal(y, O.add(mid, c.s_y, c.zp_y, r, 0.031, 7, 0.047, -3, "i8"), f"fused flow {tile}")


@pytest.mark.parametrize("cout", [64, 128, 200])   # 64-wide tiles fit better; past the padded tables
def test_not_offered(cout):
    c = W.conv_case(L("n", 9, 9, 64, cout, 1, 1), 2, seed=1)
    with env(QNN_FLOW=20):
        p, keep = make_plan(c)
    assert "tile=96x" not in p.describe(), p.describe()
    p.close()
