"""GPU parity of the split-reduction form of the LDS-direct ring kernel:
each tile's K-steps in S parts run by separate workgroups, whose int32
partial sums the last-arriving workgroup adds before the requantize
epilogue (terms of Eq. (3), requantize of Eq. (5)).  Every configuration
with a split form is forced at several part counts on ragged shapes with
padding, strides, int8 inputs and outputs, term 3 and int32 outputs, and
compared byte for byte with the oracle; repeated runs check that the
arrival counters return to zero, two streams with their own workspaces
that runs do not share state."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import assert_equal, dev, env, log, make_plan, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

SPLIT_TILES = [0, 1, 2, 3, 4, 5, 6, 8, 9, 12]

SHAPES = [
    (W.ConvLayer("t", 23, 21, 64, 200, 3, 3, 1, (1, 1, 1, 1)), 2, {}),
    (W.ConvLayer("t", 23, 21, 64, 200, 3, 3, 1, (1, 1, 1, 1)), 2, dict(zp_w="channel")),
    (W.ConvLayer("t", 13, 11, 64, 130, 3, 3, 1, (1, 1, 1, 1)), 1, dict(yt="i32")),
    (W.ConvLayer("t", 16, 15, 128, 96, 3, 3, 2, (0, 0, 1, 1)), 3, dict(x_dtype="i8")),
    (W.ConvLayer("t", 17, 17, 128, 72, 1, 7, 1, (0, 3, 0, 3)), 2, dict(rounding="half_away")),
    (W.ConvLayer("t", 9, 9, 512, 300, 1, 1), 5, dict(yt="i8")),
    (W.ConvLayer("t", 7, 7, 512, 512, 3, 3, 1, (1, 1, 1, 1)), 2, dict(rounding="two_stage")),
]


@pytest.mark.parametrize("parts", [2, 3, 5])
@pytest.mark.parametrize("tile", SPLIT_TILES)
def test_every_split_tile(tile, parts):
    with env(QNN_DMA=tile, QNN_KSPLIT=parts):
        for i, (layer, N, kw) in enumerate(SHAPES):
            c = W.conv_case(layer, N, seed=500 + tile * 10 + i, **kw)
            if layer.R * layer.S * layer.Cin // 64 < parts:
                continue
            p, keep = make_plan(c)
            d = p.describe()
            assert d.startswith("conv_dma tile") and f"ksplit={parts}" in d, d
            x = dev(c.x)
            ref = run_oracle(c)
            log(f"split tile {tile} parts {parts} shape {i}: {d}")
            for rep in range(2):   # the counters must be back at zero for the second run
                y = p.run(x)
                torch.cuda.synchronize()
                assert_equal(y.cpu().numpy(), ref, f"tile {tile} parts {parts} shape {i} run {rep} {kw}")
            p.close()


def test_split_channel_slice_and_streams():
    """A split plan writing a channel slice, run on two streams at once with
    a workspace each, twice: every run equals the oracle and leaves the
    bytes outside the slice untouched."""
    layer = W.ConvLayer("t", 14, 14, 256, 96, 3, 3, 1, (1, 1, 1, 1))
    c = W.conv_case(layer, 4, seed=77)
    ref = run_oracle(c)
    with env(QNN_DMA=0, QNN_KSPLIT=4):
        p, keep = make_plan(c, y_ldc=256, y_coff=64)
    assert "ksplit=4" in p.describe(), p.describe()
    x = dev(c.x)
    ws = [torch.zeros(p.workspace_size, dtype=torch.uint8, device="cuda") for _ in range(2)]
    st = [torch.cuda.Stream(), torch.cuda.Stream()]
    ys = [torch.full((4, 14, 14, 256), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    for rep in range(2):
        for k in range(2):
            with torch.cuda.stream(st[k]):
                p.run(x, ys[k], workspace=ws[k], stream=st[k])
        torch.cuda.synchronize()
        for k in range(2):
            y = ys[k].cpu().numpy()
            assert_equal(y[..., 64:160], ref, f"stream {k} run {rep}")
            assert (y[..., :64] == 0x5A).all() and (y[..., 160:] == 0x5A).all()
    p.close()


@pytest.mark.parametrize("forced,prefix", [({}, "conv_dma_"), (dict(QNN_DMA=4, QNN_KSPLIT=8), "conv_dma tile")],
                         ids=["auto", "split"])
def test_small_grid(forced, prefix):
    """The stage-7 3x3 ResNet-50 layer at batch 1 (49 pixels, 512 channels,
    72 K-steps) has too few tiles for the chip: the plan's own choice, and
    eight workgroups per tile."""
    layer = [l for l in W.resnet50() if l.name == "s7b1_3x3"][0]
    c = W.conv_case(layer, 1, seed=3)
    with env(**forced):
        p, keep = make_plan(c)
        d = p.describe()
        log(f"s7b1_3x3 b1: {d}")
        p.close()
        assert d.startswith(prefix), d
        assert_equal(run_gpu(c), run_oracle(c), "s7b1_3x3 b1")
