"""Plan preparation makes the tables that the chosen kernel reads, and no
others: border classes and corrections over pads, strides, dilations and pixel
counts at which they differ, recorded choices of every kernel family (plans and
one-shot calls), and the time that padding adds to a creation."""
import time

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import Q, O, dev, env, make_plan, run_gpu, run_oracle, assert_equal  # noqa: E402

L = W.ConvLayer


@pytest.mark.parametrize("knob", [dict(QNN_FLOW=0), dict(QNN_SMALL=0), dict(QNN_DMA=0), {}],
                         ids=["flow", "small", "dma", "untuned"])
@pytest.mark.parametrize("layer,N,dil", [
    (L("3x3", 1, 1, 64, 33, 3, 3, 1, (1, 1, 1, 1)), 1, 1),          # one pixel, every tap but one outside
    (L("5x5s2", 11, 13, 20, 17, 5, 5, 2, (2, 4, 3, 1)), 3, 1),      # one-sided pads, 84 pixels a row pair
    (L("3x3d", 9, 7, 128, 40, 3, 3, 1, (4, 5, 2, 3)), 2, 3),        # dilated: the middle taps outside too
    (L("15x15", 16, 17, 4, 20, 15, 15, 1, (7, 7, 7, 7)), 1, 1),     # 225 taps
    (L("1x7", 17, 17, 160, 300, 1, 7, 1, (0, 3, 0, 3)), 2, 1),      # two channel blocks of the records
], ids=lambda v: getattr(v, "name", None))
def test_border_tables(layer, N, dil, knob):
    c = W.conv_case(layer, N, seed=layer.Cin)
    ref = O.conv2d(c.x, c.s_x, c.zp_x, c.w, c.s_w, c.zp_w, c.bias, c.s_y, c.zp_y, c.yt, c.act, c.rounding,
                   (layer.stride,) * 2, c.pads, (dil, dil))
    w, b = dev(c.w), dev(c.bias)
    with env(**(knob or dict(QNN_AUTOTUNE=0))):
        p = Q.conv2d_plan(c.x.shape, "u8", c.s_x, c.zp_x, w, c.s_w, c.zp_w, b, layer.stride, c.pads, dil, c.s_y,
                          c.zp_y, c.yt, c.act, c.rounding)
        y = p.run(dev(c.x)).cpu().numpy()
        d = p.describe()
        p.close()
    print(layer.name, knob, d, flush=True)
    assert_equal(y, ref, f"{layer.name} {knob}: {d}")


RECORDED = [   # layer, batch, {describe prefix: family, tile, split}
    (L("c64", 12, 14, 64, 64, 3, 3, 1, (1, 1, 1, 1)), 2,
     {"conv_tap": (1, 0, 1), "conv_dma tile": (2, 0, 1), "conv_wave": (3, 2, 1), "conv_halo": (4, 8, 1),
      "conv_window": (5, 0, 1), "conv_dma_flow": (6, 0, 1), "conv_dma_small": (7, 0, 1)}),
    (L("c48", 12, 14, 48, 64, 3, 3, 1, (1, 1, 1, 1)), 2,
     {"conv_mfma": (0, 3, 1), "conv_dma_flow": (6, 1, 1), "conv_dma_small": (7, 4, 1)}),
    (L("stem", 29, 31, 3, 64, 7, 7, 2, (3, 3, 3, 3)), 2,
     {"conv_dma tile": (2, 4, 1), "conv_dma_flow": (6, 0, 1), "conv_dma_small": (7, 1, 1)}),
    (L("c80", 9, 9, 80, 70, 1, 1), 2,
     {"conv_mfma": (0, 3, 1), "conv_tap": (1, 0, 1), "conv_dma tile": (2, 4, 1), "conv_dma_flow": (6, 0, 1),
      "conv_dma_small": (7, 2, 1)}),
]


@pytest.mark.parametrize("i", range(len(RECORDED)), ids=[r[0].name for r in RECORDED])
def test_recorded_family(i, tmp_path):
    layer, N, choices = RECORDED[i]
    c = W.conv_case(layer, N, seed=70 + i)
    ref = run_oracle(c)
    path = tmp_path / "choices.txt"
    try:
        Q.set_tuning_file(str(path))
        p, keep = make_plan(c)
        p.close()
        key = path.read_text().split()[0]
        for prefix, (fam, tile, split) in choices.items():
            path.write_text(f"{key} {fam} {tile} {split}\n")
            Q.set_tuning_file(str(path))
            p, keep = make_plan(c)
            d = p.describe()
            assert d.startswith(prefix), d
            y = p.run(dev(c.x)).cpu().numpy()
            p.close()
            print(layer.name, d, flush=True)
            assert_equal(y, ref, f"{layer.name} recorded {prefix}")
            assert_equal(run_gpu(c, one_shot=True), ref, f"{layer.name} one-shot {prefix}")
    finally:
        Q.set_tuning_file(None)


def test_recorded_without_border_classes(tmp_path):
    """Files written when padded layers of such channel counts had no border
    classes name them with none."""
    c = W.conv_case(L("old", 12, 14, 48, 64, 3, 3, 1, (1, 1, 1, 1)), 2, seed=5)
    path = tmp_path / "choices.txt"
    try:
        Q.set_tuning_file(str(path))
        p, keep = make_plan(c)
        p.close()
        key = path.read_text().split()[0]
        assert ":b9:" in key, key
        path.write_text(key.replace(":b9:", ":b0:") + " 0 3 1\n")
        Q.set_tuning_file(str(path))
        p, keep = make_plan(c)
        d = p.describe()
        assert d.startswith("conv_mfma tile=64x64x128"), d
        y = p.run(dev(c.x)).cpu().numpy()
        p.close()
        assert_equal(y, run_oracle(c), "recorded without classes")
        assert len(path.read_text().split("\n")) == 2   # nothing timed anew
    finally:
        Q.set_tuning_file(None)


@pytest.mark.parametrize("cout,tile", [(32, "64x128x64"), (64, "64x128x64"), (100, "128x128x64"), (130, "64x128x64")])
def test_untimed_tile_fits_the_channels(cout, tile):
    """What a one-shot call takes where 128 x 128 tiles fill the chip: no block
    of 64 channels that the layer does not have."""
    c = W.conv_case(L("u", 92, 93, 32, cout, 3, 3, 1, (1, 1, 1, 1)), 8, seed=cout)
    with env(QNN_AUTOTUNE=0):
        p, keep = make_plan(c)
    d = p.describe()
    y = p.run(dev(c.x)).cpu().numpy()
    p.close()
    assert d.startswith(f"conv_dma_flow tile={tile} "), d
    assert_equal(y, run_oracle(c), d)


def test_padding_adds_little_to_creation():
    """Without timing of candidates, as a one-shot call prepares. Padding took
    7 times the unpadded layer's time while each pixel's class was worked out
    on the host and each correction summed by one thread; 1.1 times now."""
    t = {0: [], 1: []}
    w = dev(np.random.default_rng(0).integers(-60, 61, size=(32, 3, 3, 36)).astype(np.int8))
    s_w, z = np.full(32, 0.01, np.float32), np.zeros(32, np.int32)
    with env(QNN_AUTOTUNE=0):
        for i in range(12):
            for pad in (0, 1):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                p = Q.conv2d_plan((32, 160, 160, 36), "u8", 0.02, 117, w, s_w, z, None, 1, pad, 1, 2.0, 128, "u8")
                t[pad].append(time.perf_counter() - t0)
                p.close()
    plain, padded = (float(np.median(t[k][2:])) * 1e6 for k in (0, 1))
    print(f"creation: {plain:.0f} us, padded {padded:.0f} us", flush=True)
    assert padded < 3 * plain
