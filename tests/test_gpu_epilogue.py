"""The epilogue of the short-loop conv kernel: records with the bias folded
into the 64-bit product (full-range and narrower clamps, staged rows and rows
stored from registers, reductions too long for them), the residual add with
f32 terms (ties, equal scales, every byte pair of types, scales whose terms
need the tables or the long form), and a 256 x 256 tile that gives way when a
residual is fused."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import Q, O, dev, env, make_plan, run_gpu, run_oracle, assert_equal  # noqa: E402

L = W.ConvLayer


@pytest.mark.parametrize("yt", ["u8", "i8"])
@pytest.mark.parametrize("act", ["none", "relu", "narrow"])
@pytest.mark.parametrize("cout", [16, 24, 96, 130])
def test_record_forms(yt, act, cout):
    for layer in (L("p", 9, 9, 48, cout, 1, 1), L("t", 9, 8, 32, cout, 3, 3, 1, (1, 1, 1, 1))):
        c = W.conv_case(layer, 3, seed=cout, yt=yt, act=None, zp_w="zero")
        hi = 255 if yt == "u8" else 127
        c.act = {"none": None, "relu": (c.zp_y, hi), "narrow": (c.zp_y - 9, min(c.zp_y + 40, hi))}[act]
        for tile in (0, 5):
            with env(QNN_FLOW=tile):
                assert_equal(run_gpu(c), run_oracle(c), f"{layer.name} {yt} {act} K={cout} flow {tile}")


@pytest.mark.parametrize("J", [26000, 26400])
def test_long_reduction(J):
    """Weight zero points: up to J = 26214 the records hold the bias."""
    c = W.conv_case(L("long", 1, 1, J, 40, 1, 1), 3, seed=J, zp_w="channel")
    with env(QNN_FLOW=0):
        assert_equal(run_gpu(c), run_oracle(c), f"1x1 J={J}")


@pytest.mark.parametrize("yt,rt,ot", [("u8", "u8", "u8"), ("i8", "u8", "i8"), ("u8", "i8", "i8"), ("i8", "i8", "u8")])
@pytest.mark.parametrize("ratios", [(0.5, 0.5), (1.0, 1.0), (2.0, 0.25), (0.7371, 1.2519), (3e-4, 37.0), (3e5, 1.0)])
@pytest.mark.parametrize("knob", [dict(QNN_FLOW=2), dict(QNN_SMALL=2)], ids=["flow", "small"])
def test_add_terms(yt, rt, ot, ratios, knob):
    c = W.conv_case(L("a", 16, 16, 64, 64, 1, 1), 4, seed=9, yt=yt, act=None)
    mid = run_oracle(c)
    assert len(np.unique(mid)) > 200   # nearly every byte of the first operand
    s_o = c.s_y / ratios[0]
    s_r = s_o * ratios[1]
    r = np.random.default_rng(4).integers(0, 256, size=mid.shape).astype(np.uint8)
    r = r if rt == "u8" else r.view(np.int8)
    zp_r, zp_o = (131 if rt == "u8" else -5), (120 if ot == "u8" else 7)
    ref = O.add(mid, c.s_y, c.zp_y, r, s_r, zp_r, s_o, zp_o, ot)
    for force in (None, 0):
        with env(**knob):
            p, keep = make_plan(c)
        with env(**({} if force is None else dict(QNN_FLOAT_ADD=force))):
            p.set_residual(rt, s_r, zp_r, s_o, zp_o, ot)
        y = p.run(dev(c.x), residual=dev(r)).cpu().numpy()
        p.close()
        assert_equal(y, ref, f"add {yt} {rt} {ot} {ratios} {knob} float={force}")


def test_largest_tile_gives_way(tmp_path):
    """A recorded choice of the 256 x 256 tile, which has no fused add."""
    c = W.conv_case(L("g", 16, 16, 256, 512, 1, 1), 4, seed=2)
    path = tmp_path / "choices.txt"
    try:
        Q.set_tuning_file(str(path))
        p, keep = make_plan(c)
        p.close()
        key = path.read_text().split()[0]
        path.write_text(f"{key} 6 6 1\n")
        Q.set_tuning_file(str(path))
        p, keep = make_plan(c)
    finally:
        Q.set_tuning_file(None)
    assert "tile=256x256" in p.describe(), p.describe()
    mid = run_oracle(c)
    assert_equal(p.run(dev(c.x)).cpu().numpy(), mid, "largest tile")
    r = np.random.default_rng(1).integers(0, 256, size=mid.shape, dtype=np.int64).astype(np.uint8)
    p.set_residual("u8", 0.03, 7, 0.05, 9, "u8")
    assert "conv_dma_flow" in p.describe() and "256x256" not in p.describe(), p.describe()
    y = p.run(dev(c.x), residual=dev(r)).cpu().numpy()
    p.close()
    assert_equal(y, O.add(mid, c.s_y, c.zp_y, r, 0.03, 7, 0.05, 9, "u8"), "fused after giving way")


@pytest.mark.parametrize("choice,prefix", [("6 4 1", "conv_dma_flow tile=256x128x64 threads=512 stages=4 tiles=16 "),
                                           ("6 16 1", "conv_dma_flow tile=64x64x64 threads=256 stages=4s tiles=128 "),
                                           ("7 5 1", "conv_dma_small tile=32x64x64 threads=512 stages=1 tiles=256 ")])
def test_largest_tile_gives_way_as_recorded(choice, prefix, tmp_path):
    """The kernel that takes over is recorded beside the choice."""
    c = W.conv_case(L("g", 16, 16, 256, 512, 1, 1), 4, seed=2)
    path = tmp_path / "choices.txt"
    try:
        Q.set_tuning_file(str(path))
        p, keep = make_plan(c)
        p.close()
        key = path.read_text().split()[0]
        path.write_text(f"{key} 6 6 1\n{key}+add {choice}\n")
        Q.set_tuning_file(str(path))
        p, keep = make_plan(c)
    finally:
        Q.set_tuning_file(None)
    mid = run_oracle(c)
    r = np.random.default_rng(1).integers(0, 256, size=mid.shape, dtype=np.int64).astype(np.uint8)
    p.set_residual("u8", 0.03, 7, 0.05, 9, "u8")
    assert p.describe().startswith(prefix), p.describe()
    y = p.run(dev(c.x), residual=dev(r)).cpu().numpy()
    p.close()
    assert_equal(y, O.add(mid, c.s_y, c.zp_y, r, 0.03, 7, 0.05, 9, "u8"), "fused after giving way")


def test_second_plan_gives_way_alike():
    """A plan created from the choice that timing an equal one left behind."""
    w = dev(np.random.default_rng(0).integers(-90, 91, size=(4096, 1, 1, 4096)).astype(np.int8))
    seen = []
    for _ in range(2):
        p = Q.conv2d_plan((1, 64, 64, 4096), "u8", 0.02, 100, w, 0.01, 0, None, 1, 0, 1, 2.0, 3, "i8")
        own = p.describe()
        p.set_residual("i8", 0.03, 7, 0.05, 9, "i8")
        seen.append((own, p.describe()))
        p.close()
    print(seen, flush=True)
    assert seen[0] == seen[1], seen


@pytest.mark.parametrize("knob", [dict(QNN_FLOW=0), dict(QNN_FLOW=3), dict(QNN_SMALL=0), dict(QNN_TILE=0)],
                         ids=lambda d: "".join(f"{k[4:].lower()}{v}" for k, v in d.items()))
@pytest.mark.parametrize("R", [1, 3])
@pytest.mark.parametrize("sign", [1, -1])
def test_constant_outside_int32(R, sign, knob):
    """One input channel, padded to four, with weight zero points and the
    largest bias that is accepted: every sum fits int32, the constant that
    bias, zero points and padded channels fold into does not."""
    K, w_v, zp_w = 20, (127, -128)[sign < 0], (-128, 127)[sign < 0]
    bias = sign * (2**31 - 1 - 255 * 255 * R * R)
    assert abs(bias + 128 * w_v * R * R + 4 * R * R * -128 * zp_w) > 2**31   # x less 128 has zero point -128
    rng = np.random.default_rng(R)
    x = rng.integers(0, 256, size=(2, 7, 9, 1)).astype(np.uint8)
    x[0, 0, :2, 0] = 0, 255
    w = np.full((K, R, R, 1), w_v, np.int8)
    zpw, b = np.full(K, zp_w, np.int32), np.full(K, bias, np.int32)
    s_w, pad = np.full(K, 2.0**-23, np.float32), R // 2     # shift 53, the largest of the 32-bit form
    with env(**knob):
        y = Q.conv2d(dev(x), 1.0, 0, dev(w), s_w, zpw, dev(b), 1, pad, 1, 1.0, 128, "u8").cpu().numpy()
    ref = O.conv2d(x, 1.0, 0, w, s_w, zpw, b, 1.0, 128, "u8", pads=(pad,) * 4)
    assert (ref == (255 if sign > 0 else 0)).all()
    assert_equal(y, ref, f"constant beyond int32: {knob} {R}x{R}")
