"""The kernel for few output pixels (conv_small.hip), every configuration
forced, on the shapes of the short-loop kernel's test (they share the packing
and the chunk table) and on reductions of one K-step, of an odd count, and of
more steps than the workgroup holds in flight."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import Q, O, dev, env, make_plan, run_gpu, run_oracle, assert_equal  # noqa: E402
from test_gpu_flow import SHAPES  # noqa: E402

L = W.ConvLayer
MORE = [
    (L("one", 1, 1, 64, 64, 1, 1), 1, {}),
    (L("3x3c512", 7, 7, 512, 40, 3, 3, 1, (1, 1, 1, 1)), 1, dict(yt="i8")),
    (L("1x1c2100", 3, 3, 2100, 70, 1, 1), 1, dict(zp_w="channel", rounding="two_stage")),
    (L("5x5c512", 6, 6, 512, 20, 5, 5, 2), 2, dict(x_dtype="i8")),
]


@pytest.mark.parametrize("tile", range(6))
def test_every_small_tile(tile):
    for i, (layer, N, kw) in enumerate(SHAPES + MORE):
        c = W.conv_case(layer, N, seed=1300 + i, **kw)
        with env(QNN_SMALL=tile):
            p, keep = make_plan(c)
            d = p.describe()
            p.close()
            assert d.startswith("conv_dma_small"), d
            print(f"small {tile} {layer.name}: {d}", flush=True)
            assert_equal(run_gpu(c), run_oracle(c), f"small {tile} {layer.name} {kw}: {d}")


@pytest.mark.parametrize("tile", [0, 2, 4, 5])
@pytest.mark.parametrize("dts", [("i8", "u8", "i8"), ("u8", "i8", "u8")])
def test_fused_add_and_slice(tile, dts):
    """A residual add in the epilogue (aligned residual rows and byte by byte,
    both add forms), and a channel slice of a wider output."""
    yt, rt, ot = dts
    c = W.conv_case(L("f3", 12, 13, 48, 77, 3, 3, 1, (1, 1, 1, 1)), 2, seed=31, yt=yt)
    mid = run_oracle(c)
    rng = np.random.default_rng(tile)
    r = rng.integers(0, 256, size=mid.shape[:3] + (96,)).astype(np.uint8)
    r = r if rt == "u8" else r.view(np.int8)
    for coff, s_o, rounding in ((0, 0.047, "half_up"), (3, 0.011, "half_away")):
        with env(QNN_SMALL=tile):
            p, keep = make_plan(c, y_ldc=80)
        p.set_residual(rt, 0.031, 7, s_o, 5, ot, r_ldc=96, r_coff=coff, rounding=rounding)
        y = p.run(dev(c.x), residual=dev(r)).cpu().numpy()[..., :77]
        ref = O.add(mid, c.s_y, c.zp_y, np.ascontiguousarray(r[..., coff:coff + 77]), 0.031, 7, s_o, 5, ot, None,
                    rounding)
        assert_equal(y, ref, f"fused small {tile} {dts} {coff}")
        p.close()
    with env(QNN_SMALL=tile):
        p, keep = make_plan(c, y_ldc=150, y_coff=65)
    out = torch.full(mid.shape[:3] + (150,), 77, dtype=torch.int8 if yt == "i8" else torch.uint8, device="cuda")
    p.run(dev(c.x), out=out)
    got = out.cpu().numpy()
    assert_equal(got[..., 65:142], mid, f"slice small {tile}")
    assert (got[..., :65] == 77).all() and (got[..., 142:] == 77).all()


@pytest.mark.parametrize("M,K,N", [(1, 655, 267), (16, 768, 1001), (130, 93, 64)])
def test_dense(M, K, N):
    for tile in (0, 3, 5):
        c = W.dense_case(W.DenseLayer("d", M, K, N), seed=M, yt="i8")
        with env(QNN_SMALL=tile):
            assert_equal(run_gpu(c), run_oracle(c), f"dense {M} {K} {N} small {tile}")
