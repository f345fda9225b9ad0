"""The short-loop LDS-direct kernel (conv_flow_kernel.h), every configuration
forced where it holds the reduction, on the shapes at which its forms differ:
linear (1x1 inside the image, dense) with channel counts that end inside a
K-step or a 16-byte chunk, strided; tabulated taps with several taps in a
K-step, channels padded to 16 per tap, padding, dilation; row pairs; ragged
channel and pixel tiles; 1 to 20 K-steps; term 3, int32 output, the three
roundings."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import Q, O, dev, env, make_plan, run_gpu, run_oracle, assert_equal  # noqa: E402

STAGES = [0] * 10 + [1, 1, 1, 2, 2, 2, 4, 4, 4]   # K-steps a short form holds (0: ring)
L = W.ConvLayer
SHAPES = [
    (L("1x1", 9, 9, 64, 300, 1, 1), 5, {}),
    (L("1x1s2", 9, 11, 128, 72, 1, 1, 2), 3, dict(yt="i8")),
    (L("1x1c24", 13, 7, 24, 144, 1, 1), 3, dict(x_dtype="i8")),
    (L("1x1c20", 11, 9, 20, 70, 1, 1), 2, {}),
    (L("1x1c7", 11, 9, 7, 33, 1, 1), 2, {}),
    (L("1x1c208", 5, 5, 208, 130, 1, 1), 7, dict(zp_w="channel")),
    (L("1x1c520", 10, 10, 520, 260, 1, 1), 4, dict(yt="i32")),
    (L("1x1pad", 8, 8, 64, 96, 1, 1, 1, (1, 1, 1, 1)), 2, dict(x_dtype="i8")),
    (L("3x3", 23, 21, 64, 200, 3, 3, 1, (1, 1, 1, 1)), 2, {}),
    (L("3x3z", 23, 21, 64, 200, 3, 3, 1, (1, 1, 1, 1)), 1, dict(zp_w="channel")),
    (L("3x3c48", 12, 14, 48, 64, 3, 3, 1, (1, 1, 1, 1)), 3, dict(rounding="half_away")),
    (L("3x3c16", 12, 14, 16, 40, 3, 3, 2, (0, 0, 1, 1)), 3, {}),
    (L("5x5c36", 9, 9, 36, 70, 5, 5, 1, (2, 2, 2, 2)), 2, dict(rounding="two_stage")),
    (L("7x1c160", 17, 17, 160, 160, 7, 1, 1, (3, 0, 3, 0)), 1, dict(yt="i8")),
    (L("1x15c20", 5, 31, 20, 24, 1, 15, 1, (0, 7, 0, 7)), 2, {}),
    (L("3x3i32", 16, 15, 128, 96, 3, 3, 2, (0, 0, 1, 1)), 3, dict(yt="i32")),
    (L("stem", 29, 31, 3, 64, 7, 7, 2, (3, 3, 3, 3)), 2, {}),
    (L("c8", 17, 16, 8, 24, 3, 3, 1, (1, 1, 1, 1)), 2, dict(x_dtype="i8")),
]


@pytest.mark.parametrize("tile", range(len(STAGES)))
def test_every_flow_tile(tile):
    ran = 0
    for i, (layer, N, kw) in enumerate(SHAPES):
        c = W.conv_case(layer, N, seed=1200 + i, **kw)
        with env(QNN_FLOW=tile):
            p, keep = make_plan(c)
            d = p.describe()
            p.close()
            if "cands=1 " not in d + " ":
                continue   # a short form with fewer stages, or the largest tile beyond its shapes
            ran += 1
            assert d.startswith("conv_dma_flow"), d
            print(f"flow {tile} {layer.name}: {d}", flush=True)
            assert_equal(run_gpu(c), run_oracle(c), f"flow {tile} {layer.name} {kw}: {d}")
    assert ran >= (3 if STAGES[tile] else 6)


@pytest.mark.parametrize("tile", [0, 3, 4, 7])
def test_dilation_and_zero_point_zero(tile):
    layer = L("dil", 15, 13, 40, 40, 3, 3, 1, (2, 1, 2, 3))
    c = W.conv_case(layer, 2, seed=3)
    for zp in (c.zp_x, 0):
        c.zp_x = zp
        with env(QNN_FLOW=tile):
            p = Q.conv2d_plan(c.x.shape, "u8", c.s_x, c.zp_x, dev(c.w), c.s_w, c.zp_w, dev(c.bias), 1, c.pads, (2, 2),
                              c.s_y, c.zp_y, c.yt, c.act, c.rounding)
        assert p.describe().startswith("conv_dma_flow"), p.describe()
        y = p.run(dev(c.x))
        torch.cuda.synchronize()
        p.close()
        ref = O.conv2d(c.x, c.s_x, c.zp_x, c.w, c.s_w, c.zp_w, c.bias, c.s_y, c.zp_y, c.yt, c.act, c.rounding, (1, 1),
                       c.pads, (2, 2))
        assert_equal(y.cpu().numpy(), ref, f"dilated flow {tile} zp {zp}")


@pytest.mark.parametrize("tile", [0, 1, 5, 7, 10, 17])
@pytest.mark.parametrize("layer", [L("f1", 12, 13, 64, 72, 1, 1), L("f3", 12, 13, 48, 80, 3, 3, 1, (1, 1, 1, 1))],
                         ids=["linear", "taps"])
def test_fused_add_and_slice(tile, layer):
    """A residual add in the epilogue, and a channel slice of a wider output."""
    c = W.conv_case(layer, 3, seed=31, yt="i8")
    mid = run_oracle(c)
    with env(QNN_FLOW=tile):
        p, keep = make_plan(c, y_ldc=80)
        s, keep2 = make_plan(c, y_ldc=160, y_coff=64)
    if "cands=1 " not in p.describe() + " ":
        pytest.skip("short form with fewer stages than K-steps")
    rng = np.random.default_rng(tile)
    r = rng.integers(0, 256, size=mid.shape[:3] + (80,), dtype=np.int64).astype(np.uint8)
    p.set_residual("u8", 0.031, 7, 0.047, -3, "i8", r_ldc=80)
    y = p.run(dev(c.x), residual=dev(r)).cpu().numpy()[..., :layer.Cout]
    assert_equal(y, O.add(mid, c.s_y, c.zp_y, r[..., :layer.Cout], 0.031, 7, 0.047, -3, "i8"), f"fused flow {tile}")
    out = torch.full(mid.shape[:3] + (160,), 77, dtype=torch.int8, device="cuda")
    s.run(dev(c.x), out=out)
    got = out.cpu().numpy()
    assert_equal(got[..., 64:64 + layer.Cout], mid, f"slice flow {tile}")
    assert (got[..., :64] == 77).all() and (got[..., 64 + layer.Cout:] == 77).all()


@pytest.mark.parametrize("M,K,N", [(300, 1000, 1001), (1030, 320, 520), (5, 4096, 64)])
def test_dense_largest_tile_grouped(M, K, N):
    """Dense through the 256 x 256 tile, and through 64 x 64 with weights past
    the size at which four pixel tiles are interleaved."""
    for tile, (m, k, n) in ((6, (M, K, N)), (0, (M, 4096, 1100))):
        c = W.dense_case(W.DenseLayer("d", m, k, n), seed=M)
        with env(QNN_FLOW=tile):
            assert_equal(run_gpu(c), run_oracle(c), f"dense {m} {k} {n} flow {tile}")


@pytest.mark.parametrize("layer,knobs", [
    # weights beyond 4 MB: the channel tiles of four pixel tiles in turn, the last group of fewer
    (L("il", 9, 37, 4100, 1100, 1, 1), [dict(QNN_FLOW=t) for t in (0, 3, 4, 6, 9, 19)]),
    # 900 K-steps: a chunk table of 29 KB; 938 without one
    (L("15x15", 8, 8, 256, 32, 15, 15, 1, (7, 7, 7, 7)), [dict(QNN_FLOW=0), dict(QNN_FLOW=4), dict(QNN_SMALL=0)]),
    (L("long", 2, 3, 60000, 48, 1, 1), [dict(QNN_FLOW=0), dict(QNN_FLOW=7), dict(QNN_SMALL=3)]),
], ids=lambda v: getattr(v, "name", None))
def test_large_weights_and_long_reductions(layer, knobs):
    c = W.conv_case(layer, 1, seed=5)
    ref = run_oracle(c)
    for knob in knobs:
        with env(**knob):
            p, keep = make_plan(c)
        d = p.describe()
        y = p.run(dev(c.x)).cpu().numpy()
        p.close()
        print(layer.name, knob, d, flush=True)
        assert "cands=1" in d.split() and d.startswith("conv_dma_flow" if "QNN_FLOW" in knob else "conv_dma_small"), d
        assert_equal(y, ref, f"{layer.name} {knob}: {d}")
