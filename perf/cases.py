"""The calls whose time is watched: what a program that runs quantized
networks on this library has it do, through the public Python entry points.

A case is a dict of plain values with a "kind":

  conv        one conv2d plan run: N, H, W, C, K, R, S, stride, pad_h, pad_w, act
  depthwise   one depthwise plan run: N, H, W, C, R, stride, act
  dense       one dense plan run: M, Kd, Nd
  ffn         a transformer feed-forward pair (dense up, dense down): M, Kd, Nd
  add         one qnn.add: N, H, W, C
  requantize  one per-channel requantize plan run (int32 in): N, H, W, C
  pool        one pool2d: N, H, W, C, R, stride, pad_h, mode
  network     a whole network body with int8 hand-off between its steps,
              captured once in a HIP graph and replayed, as a server runs it:
              net, N

with the data types and options of each ("xt", "wt", "yt", "zpw",
"rounding").  Inputs, weights and quantization parameters are drawn from the
seed; shapes are those of workloads/shapes.py and bench.py, or generic.
"""
import math

import numpy as np
import torch

from paper_2006_10226_amd import qnn as Q
from paper_2006_10226_amd.fusion import residual_fusions

_RANGE = {"u8": (0, 255), "i8": (-128, 127), "i32": (-2**31, 2**31 - 1)}
_TORCH = {"u8": torch.uint8, "i8": torch.int8, "i32": torch.int32}
_SIZE = {"u8": 1, "i8": 1, "i32": 4}


def listed():
    conv = {"kind": "conv", "xt": "u8", "wt": "i8", "yt": "u8", "zpw": "zero", "rounding": "half_up"}
    dense = {"xt": "u8", "wt": "i8", "yt": "i8", "zpw": "zero", "rounding": "half_up"}
    return [
        # the smallest call: one 3x3 conv of one 14x14x64 image, all latency
        dict(conv, name="conv3x3_14x14x64_b1", N=1, H=14, W=14, C=64, K=64, R=3, S=3, stride=1, pad_h=1, pad_w=1,
             act="none"),
        # one BERT-base feed-forward pair, one sequence of 128 tokens
        dict(dense, kind="ffn", name="ffn_128_tokens", M=128, Kd=768, Nd=3072),
        # the same pair on a batch of 32 sequences (and not quite full ones)
        dict(dense, kind="ffn", name="ffn_4000_tokens", M=4000, Kd=768, Nd=3072),
        # a large square product: the matrix cores at work
        dict(dense, kind="dense", name="dense_4096", M=4096, Kd=4096, Nd=4096),
        # a classifier head: 1001 classes (odd), int32 logits
        dict(dense, kind="dense", name="head_1001_b64", M=64, Kd=2048, Nd=1001, yt="i32"),
        # a 1x7 branch conv at 160 channels (not a multiple of 64) with asymmetric uint8 weights,
        # zero points per channel, ties away from zero
        dict(conv, name="conv1x7_17x17x160_b64", N=64, H=17, W=17, C=160, K=160, R=1, S=7, stride=1, pad_h=0,
             pad_w=3, act="relu", wt="u8", zpw="channel", rounding="half_away"),
        # whole bodies: a server's batch, and one image (the setting of the published measurements)
        {"kind": "network", "name": "resnet50_b32", "net": "resnet50", "N": 32},
        {"kind": "network", "name": "resnet50_b1", "net": "resnet50", "N": 1},
        {"kind": "network", "name": "mobilenet_v2_b64", "net": "mobilenet_v2", "N": 64},
        {"kind": "network", "name": "inception_mixed5_b64", "net": "inception_mixed5", "N": 64},
        # the unfused forms: an int32 conv output requantized per channel, and a residual add
        {"kind": "requantize", "name": "requantize_56x56x256_b32", "N": 32, "H": 56, "W": 56, "C": 256, "yt": "u8",
         "rounding": "half_up"},
        {"kind": "add", "name": "add_56x56x256_b32", "N": 32, "H": 56, "W": 56, "C": 256, "xt": "u8", "yt": "u8",
         "rounding": "half_up"},
    ]


# the largest listed product and the largest listed tensors bound what is drawn
_MOST_MACS = 4096**3
_MOST_BYTES = 32 * 56 * 56 * 256 * 5


def draw(rng):
    def log(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    opts = {"xt": rng.choice(["u8", "u8", "i8"]), "wt": rng.choice(["i8", "i8", "i8", "u8"]),
            "yt": rng.choice(["u8", "u8", "i8", "i32"]), "rounding": rng.choice(["half_up", "half_up", "half_away", "two_stage"])}
    opts["zpw"] = "channel" if opts["wt"] == "u8" else rng.choice(["zero", "zero", "zero", "channel"])
    kind = rng.choice(["conv"] * 7 + ["dense"] * 4 + ["ffn", "network", "network", "network", "depthwise", "depthwise",
                                                      "add", "requantize", "pool"])
    while True:
        if kind == "network":
            net = rng.choice(["resnet50", "mobilenet_v2", "inception_mixed5"])
            return {"kind": kind, "net": net, "N": log(1, 32 if net == "resnet50" else 64)}
        if kind in ("dense", "ffn"):
            c = dict(opts, kind=kind, M=log(1, 8192), Kd=log(64, 8192), Nd=log(32, 8192))
            if kind == "ffn":
                c.update(yt="i8", Kd=64 * rng.randint(4, 32))
                c["Nd"] = 4 * c["Kd"]
            if work(c)["flops"] <= 2 * _MOST_MACS and work(c)["bytes"] <= _MOST_BYTES:
                return c
            continue
        H = log(5, 160)
        c = {"kind": kind, "N": log(1, 64), "H": H, "W": max(5, H + rng.choice([0, 0, 0, -1, 2, 5]))}
        if kind == "conv":
            C = log(3, 1024) if rng.random() < 0.3 else rng.choice([16, 24, 32, 48, 64, 64, 80, 96, 128, 128, 144, 160, 192,
                                                                   256, 256, 288, 384, 448, 512, 768, 1024])
            K = log(8, 1024) if rng.random() < 0.3 else rng.choice([24, 32, 64, 64, 96, 128, 128, 160, 192, 256, 256, 320,
                                                                   384, 512, 1024])
            R, S = rng.choice([(1, 1), (1, 1), (3, 3), (3, 3), (5, 5), (1, 7), (7, 1), (1, 3), (7, 7)])
            c.update(opts, C=C, K=K, R=R, S=S, stride=rng.choice([1, 1, 1, 2]),
                     pad_h=rng.choice([R // 2, R // 2, 0]), act=rng.choice(["relu", "none"]))
            c["pad_w"] = S // 2 if c["pad_h"] == R // 2 else 0
        elif kind == "depthwise":
            c.update(opts, C=rng.choice([16, 24, 32, 96, 144, 192, 384, 576, 960, log(8, 1024)]), R=rng.choice([3, 3, 3, 5]),
                     stride=rng.choice([1, 1, 2]), act=rng.choice(["relu", "none"]))
        elif kind == "pool":
            c.update(xt=opts["xt"], C=log(8, 1280), mode=rng.choice(["avg", "max"]), R=rng.choice([2, 3, 3]),
                     stride=rng.choice([1, 2]), pad_h=rng.choice([0, 1]))
        else:
            c.update(C=log(8, 1024), xt=opts["xt"], yt=rng.choice(["u8", "i8"]), rounding=opts["rounding"])
            if kind == "requantize":
                del c["xt"]
        if c["H"] < c.get("R", 1) or c["W"] < c.get("S", c.get("R", 1)):
            continue
        w = work(c)
        if w["flops"] <= 2 * _MOST_MACS and 4096 <= w["bytes"] <= _MOST_BYTES:
            return c


# ---------------------------------------------------------------- drawing inputs

class _Rng:
    """Draws from one seed: large tensors on the GPU, small vectors on the host."""

    def __init__(self, seed):
        self.host = np.random.default_rng(seed)
        self.dev = torch.Generator(device="cuda").manual_seed(seed)

    def uniform(self, shape, dt):
        lo, hi = _RANGE[dt]
        return torch.randint(lo, hi + 1, shape, dtype=_TORCH[dt], device="cuda", generator=self.dev)

    def normal(self, shape, sigma, mean=0.0):
        return torch.round(torch.randn(shape, device="cuda", generator=self.dev) * sigma + mean)


def _f32(v):
    return float(np.float32(v))


def _weights(r, shape, K, wt, zpw, channel_dim):
    """Weights round(normal(zp, 30)) and their zero points, per channel where asked."""
    if wt == "u8":
        zp = r.host.integers(96, 161, size=K).astype(np.int32)
    elif zpw == "channel":
        zp = r.host.integers(-20, 21, size=K).astype(np.int32)
    else:
        zp = np.zeros(K, np.int32)
    lo, hi = (0, 255) if wt == "u8" else (-127, 127)
    view = [1] * len(shape)
    view[channel_dim] = K
    mean = torch.from_numpy(zp).cuda().float().view(view) if wt == "u8" else 0.0
    return r.normal(shape, 30.0, mean).clamp_(lo, hi).to(_TORCH[wt]), zp


def _layer(r, shape, K, J, channel_dim, xt, zp_x, wt, zpw, yt, act, s_x=0.02, spread2=None):
    """A layer's weights and quantization: the median channel spans about +-48
    output steps, the bias a quarter of the accumulator's spread."""
    w, zp_w = _weights(r, shape, K, wt, zpw, channel_dim)
    lo, hi = _RANGE[xt]
    if spread2 is None:   # of uniform activations about their zero point
        spread2 = 65535.0 / 12.0 + ((lo + hi) / 2.0 - zp_x) ** 2
    sig = math.sqrt(J * spread2 * 900.0)
    s_w = (48.0 / sig * 10.0 ** r.host.uniform(-0.5, 0.5, size=K)).astype(np.float32)
    s_y = _f32(s_x * math.exp(float(np.mean(np.log(s_w.astype(np.float64))))) * sig / 48.0)
    bias = np.rint(r.host.normal(0.0, sig / 4.0, size=K)).astype(np.int32)
    if yt == "i32":
        zp_y, clamp = 0, None
    elif act in ("relu", "relu6"):
        zp_y = _RANGE[yt][0] + 28
        top = _RANGE[yt][1]
        clamp = (zp_y, top if act == "relu" else min(top, zp_y + int(round(6.0 / s_y))))
    else:
        zp_y, clamp = int(r.host.integers(_RANGE[yt][0] + 100, _RANGE[yt][1] - 99)), None
    return {"w": w, "zp_w": zp_w, "s_w": s_w, "bias": torch.from_numpy(bias).cuda(), "s_y": s_y, "zp_y": zp_y,
            "clamp": clamp, "s_x": s_x, "zp_x": zp_x, "xt": xt, "yt": yt}


def _inputs(case, seed):
    """All that a case's call is given, without the library."""
    r, kind = _Rng(seed), case["kind"]
    if kind == "network":
        return _network(r, case["net"], case["N"])
    if kind in ("dense", "ffn"):
        M, Kd, Nd = case["M"], case["Kd"], case["Nd"]
        zp_x = int(r.host.integers(*_RANGE[case["xt"]]))
        x = r.uniform((M, Kd), case["xt"])
        up = _layer(r, (Nd, Kd), Nd, Kd, 0, case["xt"], zp_x, case["wt"], case["zpw"], case["yt"],
                    "relu" if kind == "ffn" else "none")
        if kind == "dense":
            return {"x": x, "layers": [up]}
        down = _layer(r, (Kd, Nd), Kd, Nd, 0, case["yt"], up["zp_y"], case["wt"], case["zpw"], case["yt"], "none",
                      up["s_y"], 48.0**2 / 2)
        return {"x": x, "layers": [up, down]}
    shape = (case["N"], case["H"], case["W"], case["C"])
    C = case["C"]
    if kind in ("conv", "depthwise"):
        zp_x = int(r.host.integers(*_RANGE[case["xt"]]))
        x = r.uniform(shape, case["xt"])
        if kind == "conv":
            K, R, S = case["K"], case["R"], case["S"]
            L = _layer(r, (K, R, S, C), K, R * S * C, 0, case["xt"], zp_x, case["wt"], case["zpw"], case["yt"],
                       case["act"])
        else:
            R = case["R"]
            L = _layer(r, (R, R, C), C, R * R, 2, case["xt"], zp_x, case["wt"], case["zpw"], case["yt"], case["act"])
        return {"x": x, "layers": [L]}
    if kind == "add":
        s = [_f32(v) for v in 10.0 ** r.host.uniform(-2.5, -1.0, size=2)]
        z = [int(v) for v in r.host.integers(*_RANGE[case["xt"]], size=2)]
        return {"x": r.uniform(shape, case["xt"]), "b": r.uniform(shape, case["xt"]), "s": s, "z": z,
                "s_y": _f32(1.1 * (s[0] + s[1])), "zp_y": int(r.host.integers(*_RANGE[case["yt"]]))}
    if kind == "requantize":   # accumulators of a conv: near normal, most of them inside the output's range
        return {"x": r.normal(shape, 40000.0).to(torch.int32),
                "s": (2e-5 * 10.0 ** r.host.uniform(-0.5, 0.5, size=C)).astype(np.float32), "s_y": 0.02,
                "zp_y": int(r.host.integers(_RANGE[case["yt"]][0] + 100, _RANGE[case["yt"]][1] - 99))}
    return {"x": r.uniform(shape, case["xt"])}   # pool


def _pads(h, w):
    return (h, w, h, w)


# ---------------------------------------------------------------- network bodies

def _net_steps(net):
    """(kind, name, inputs, geometry) of every step, in order.  Tensors are
    named by the step that writes them; geometry is (K, R, S, stride, pads,
    act) of a conv, with its channel offset in a concat tensor where it writes
    a slice of one."""
    out = []

    def conv(name, src, K, R=1, S=1, stride=1, pads=(0, 0, 0, 0), act="relu", kind="conv", into=None):
        out.append({"kind": kind, "src": (src,), "dst": into[0] if into else name, "K": K, "R": R, "S": S,
                    "stride": stride, "pads": pads, "act": act, "into": into})
        return name

    def pool(name, src, mode, k, stride, pads):
        out.append({"kind": "pool", "src": (src,), "dst": name, "mode": mode, "k": k, "stride": stride, "pads": pads})
        return name

    def add(name, a, b, act):
        out.append({"kind": "add", "src": (a, b), "dst": name, "act": act})
        return name

    if net == "resnet50":
        cur, cin = pool("pool", conv("stem", "x0", 64, 7, 7, 2, _pads(3, 3)), "max", 3, 2, _pads(1, 1)), 64
        for si, (width, blocks) in enumerate([(64, 3), (128, 4), (256, 6), (512, 3)]):
            for b in range(blocks):
                n, stride = f"s{si}b{b}", 2 if b == 0 and si > 0 else 1
                a = conv(n + "a", cur, width)
                m = conv(n + "b", a, width, 3, 3, stride, _pads(1, 1))
                c = conv(n + "c", m, 4 * width, act="none")
                short = conv(n + "p", cur, 4 * width, stride=stride, act="none") if b == 0 else cur
                cur = add(n + "_out", c, short, "relu")
        pool("gap_out", cur, "avg", 7, 1, _pads(0, 0))
    elif net == "mobilenet_v2":
        cur, cin = "x0", 16
        for c, blocks, s in [(24, 2, 2), (32, 3, 2), (64, 4, 2), (96, 3, 1), (160, 3, 2), (320, 1, 1)]:
            for b in range(blocks):
                n, stride = f"c{c}_{b}", s if b == 0 else 1
                e = conv(n + "e", cur, 6 * cin, act="relu6")
                d = conv(n + "d", e, 6 * cin, 3, 3, stride, _pads(1, 1) if stride == 1 else (0, 0, 1, 1), "relu6",
                         "dw")
                p = conv(n + ("p" if stride == 1 and cin == c else "_out"), d, c, act="none")
                cur, cin = add(n + "_out", p, cur, "none") if stride == 1 and cin == c else p, c
    else:
        cur = "x0"
        for tag, pool_c in (("5b", 32), ("5c", 64)):
            g = tag + "_out"
            total = 64 + 64 + 96 + pool_c
            pooled = pool(tag + "_pool", cur, "avg", 3, 1, _pads(1, 1))
            b2 = conv(tag + "_b2", cur, 48)
            b3 = conv(tag + "_b3", conv(tag + "_b3a", cur, 64), 96, 3, 3, 1, _pads(1, 1))
            conv(tag + "_b1", cur, 64, into=(g, 0, total))
            conv(tag + "_b2b", b2, 64, 5, 5, 1, _pads(2, 2), into=(g, 64, total))
            conv(tag + "_b3b", b3, 96, 3, 3, 1, _pads(1, 1), into=(g, 128, total))
            conv(tag + "_b4", pooled, pool_c, into=(g, 224, total))
            cur = g
    return out


_NET_INPUT = {"resnet50": (224, 224, 3), "mobilenet_v2": (112, 112, 16), "inception_mixed5": (35, 35, 192)}


def _net_shapes(net, N):
    """Shape of every tensor of a network body."""
    sh = {"x0": (N,) + _NET_INPUT[net]}
    for st in _net_steps(net):
        n, H, W, C = sh[st["src"][0]]
        if st["kind"] == "add":
            sh[st["dst"]] = (n, H, W, C)
            continue
        R, S = (st["k"], st["k"]) if st["kind"] == "pool" else (st["R"], st["S"])
        pt, pl, pb, pr = st["pads"]
        ho, wo = (H + pt + pb - R) // st["stride"] + 1, (W + pl + pr - S) // st["stride"] + 1
        K = C if st["kind"] == "pool" else (st["into"][2] if st["into"] else st["K"])
        sh[st["dst"]] = (n, ho, wo, K)
    return sh


def _network(r, net, N):
    """Input, weights and quantization of a network body: int8 throughout,
    every scale near its input's, ReLU outputs with zero point -100."""
    sh = _net_shapes(net, N)
    q, spread = {"x0": (0.02, -10)}, {"x0": 65535.0 / 12.0 + 9.5**2}
    steps = []
    for st in _net_steps(net):
        st, src, dst = dict(st), st["src"][0], st["dst"]
        relu = st.get("act") in ("relu", "relu6")
        if st["kind"] == "pool":
            q[dst], spread[dst] = q[src], spread[src]
        elif st["kind"] == "add":
            q[dst] = (_f32(1.5 * max(q[s][0] for s in st["src"])), -100 if relu else 0)
            spread[dst] = 48.0**2 / 2 if relu else 48.0**2
            st["clamp"] = (-100, 127) if relu else None
        else:
            C, dw = sh[src][3], st["kind"] == "dw"
            shape = (st["R"], st["S"], C) if dw else (st["K"], st["R"], st["S"], C)
            J = st["R"] * st["S"] * (1 if dw else C)
            L = _layer(r, shape, st["K"], J, 2 if dw else 0, "i8", q[src][1], "i8", "zero", "i8", st["act"], q[src][0],
                       spread[src])
            if st["into"]:   # the branches of a concat share its quantization
                L["s_y"] = q[dst][0] if dst in q else L["s_y"]
            if not relu:
                L["zp_y"] = 0
            st["L"] = L
            q[dst] = (L["s_y"], L["zp_y"])
            spread[dst] = 48.0**2 / 2 if relu else 48.0**2
        steps.append(st)
    return {"x": r.uniform(sh["x0"], "i8"), "q": q, "steps": steps}


def _capture_network(inp, case):
    """The plans and tensors of a body, residual adds in the epilogue of the
    conv that takes them, the whole captured in a HIP graph."""
    sh = _net_shapes(case["net"], case["N"])
    q, steps = inp["q"], inp["steps"]
    graph_steps = [("conv_slice" if st.get("into") else st["kind"], st["src"], st["dst"]) for st in steps]
    by_conv = {c: (i, res) for i, (c, res) in residual_fusions(graph_steps).items()}
    t, calls, skip, keep = {"x0": inp["x"]}, [], set(), []

    def tensor(name):
        if name not in t:
            t[name] = torch.empty(sh[name], dtype=torch.int8, device="cuda")
        return t[name]

    for i, st in enumerate(steps):
        if i in skip:
            continue
        x, dst = t[st["src"][0]], st["dst"]
        if st["kind"] == "pool":
            calls.append(lambda x=x, y=tensor(dst), st=st: Q.pool2d(x, st["mode"], st["k"], st["stride"], st["pads"],
                                                                    out=y))
        elif st["kind"] == "add":
            (sa, za), (sb, zb), (so, zo) = q[st["src"][0]], q[st["src"][1]], q[dst]
            calls.append(lambda a=x, b=t[st["src"][1]], y=tensor(dst), sa=sa, za=za, sb=sb, zb=zb, so=so, zo=zo,
                         act=st["clamp"]: Q.add(a, sa, za, b, sb, zb, so, zo, "i8", act, out=y))
        else:
            L = st["L"]
            args = (x.shape, "i8", L["s_x"], L["zp_x"], L["w"], L["s_w"], L["zp_w"], L["bias"], st["stride"],
                    st["pads"], 1, L["s_y"], L["zp_y"], "i8", L["clamp"])
            if st["kind"] == "dw":
                p = Q.depthwise_conv2d_plan(*args)
            elif st["into"]:
                p = Q.conv2d_plan(*args, y_ldc=st["into"][2], y_coff=st["into"][1])
            else:
                p = Q.conv2d_plan(*args)
            res = None
            if i in by_conv:
                add = steps[by_conv[i][0]]
                (sr, zr), (so, zo) = q[by_conv[i][1]], q[add["dst"]]
                try:
                    p.set_residual("i8", sr, zr, so, zo, "i8", act=add["clamp"])
                except Q.QnnError:
                    pass   # this plan's kernel has no fused add: the add runs on its own
                else:
                    res, dst = t[by_conv[i][1]], add["dst"]
                    skip.add(by_conv[i][0])
            ws = torch.zeros(p.workspace_size, dtype=torch.uint8, device="cuda") if p.workspace_size else None
            keep.append((p, ws))
            calls.append(lambda p=p, x=x, y=tensor(dst), ws=ws, res=res: p.run(x, y, ws, residual=res))
    for c in calls:
        c()
    torch.cuda.synchronize()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(s), torch.cuda.graph(g, stream=s):
        for c in calls:
            c()
    torch.cuda.synchronize()
    return {"graph": g, "stream": s, "keep": keep, "tensors": t, "out": {k: v for k, v in t.items() if k.endswith("_out")}}


# ---------------------------------------------------------------- the calls

def prepare(case, seed):
    inp, kind = _inputs(case, seed), case["kind"]
    if kind == "network":
        return dict(_capture_network(inp, case), kind=kind)
    state = {"kind": kind, "x": inp["x"]}
    if kind == "add":
        (sa, sb), (za, zb) = inp["s"], inp["z"]
        state.update(b=inp["b"], args=(sa, za), more=(sb, zb, inp["s_y"], inp["zp_y"], case["yt"], None, case["rounding"]),
                     out=torch.empty(inp["x"].shape, dtype=_TORCH[case["yt"]], device="cuda"))
        return state
    if kind == "pool":
        state.update(args=(case["mode"], case["R"], case["stride"], case["pad_h"]))
        state["out"] = Q.pool2d(inp["x"], *state["args"])
        return state
    if kind == "requantize":
        plans = [Q.requantize_plan(tuple(inp["x"].shape), "i32", inp["s"], 0, inp["s_y"], inp["zp_y"], case["yt"],
                                   rounding=case["rounding"])]
    else:
        plans = []
        for L in inp["layers"]:
            w = (L["w"], L["s_w"], L["zp_w"], L["bias"])
            y = (L["s_y"], L["zp_y"], L["yt"], L["clamp"], case["rounding"])
            if kind in ("dense", "ffn"):
                plans.append(Q.dense_plan(case["M"], L["w"].shape[1], L["xt"], L["s_x"], L["zp_x"], *w, *y))
            elif kind == "conv":
                plans.append(Q.conv2d_plan(inp["x"].shape, L["xt"], L["s_x"], L["zp_x"], *w, case["stride"],
                                           _pads(case["pad_h"], case["pad_w"]), 1, *y))
            else:
                plans.append(Q.depthwise_conv2d_plan(inp["x"].shape, L["xt"], L["s_x"], L["zp_x"], *w, case["stride"],
                                                     case["R"] // 2, 1, *y))
    state["plans"] = plans
    state["outs"] = [p.new_output() for p in plans]
    state["ws"] = [torch.zeros(p.workspace_size, dtype=torch.uint8, device="cuda") if p.workspace_size else None
                   for p in plans]
    return state


def run(state):
    kind = state["kind"]
    if kind == "network":
        state["graph"].replay()
        return state["out"]
    if kind == "add":
        return Q.add(state["x"], *state["args"], state["b"], *state["more"], out=state["out"])
    if kind == "pool":
        return Q.pool2d(state["x"], *state["args"], out=state["out"])
    x = state["x"]
    for p, y, ws in zip(state["plans"], state["outs"], state["ws"]):
        x = p.run(x, y, ws)
    return state["outs"]


def _out_hw(case):
    """Output height and width of a conv, depthwise or pool case."""
    R, S = case["R"], case.get("S", case["R"])
    ph = case["R"] // 2 if case["kind"] == "depthwise" else case["pad_h"]
    pw = case.get("pad_w", ph)
    return (case["H"] + 2 * ph - R) // case["stride"] + 1, (case["W"] + 2 * pw - S) // case["stride"] + 1


def work(case):
    """Bytes of every call's operands and result, once each, and int8
    operations (two per multiply-accumulate).  A network is its calls, the
    adds that run inside a conv counted as the tensors they cannot do without."""
    kind = case["kind"]
    if kind in ("dense", "ffn"):
        M, Kd, Nd, e = case["M"], case["Kd"], case["Nd"], _SIZE[case["yt"]]
        if kind == "ffn":
            return {"bytes": 2 * (M * Kd + Kd * Nd + M * Nd), "flops": 4 * M * Kd * Nd}
        return {"bytes": M * Kd + Kd * Nd + M * Nd * e, "flops": 2 * M * Kd * Nd}
    if kind == "network":
        b, macs = 0, 0
        sh = _net_shapes(case["net"], case["N"])
        steps = _net_steps(case["net"])
        fused = residual_fusions([("conv_slice" if s.get("into") else s["kind"], s["src"], s["dst"]) for s in steps])
        convs = {c: r for c, r in fused.values()}
        for i, st in enumerate(steps):
            size = {n: math.prod(sh[n]) for n in st["src"] + (st["dst"],)}
            if i in fused:
                continue
            if st["kind"] in ("conv", "dw"):
                C = sh[st["src"][0]][3]
                wts = st["R"] * st["S"] * (C if st["kind"] == "dw" else C * st["K"])
                out = size[st["dst"]] // sh[st["dst"]][3] * st["K"]
                b += size[st["src"][0]] + wts + out
                macs += out // st["K"] * wts
                if i in convs:   # the residual it adds
                    b += math.prod(sh[convs[i]])
            else:
                b += sum(math.prod(sh[s]) for s in st["src"]) + size[st["dst"]]
        return {"bytes": b, "flops": 2 * macs}
    x = case["N"] * case["H"] * case["W"] * case["C"]
    if kind == "add":
        return {"bytes": 3 * x, "flops": 2 * x}
    if kind == "requantize":
        return {"bytes": 5 * x, "flops": 2 * x}
    ho, wo = _out_hw(case)
    m = case["N"] * ho * wo
    if kind == "pool":
        return {"bytes": x + m * case["C"], "flops": m * case["C"] * case["R"] ** 2}
    if kind == "depthwise":
        J = case["R"] ** 2
        return {"bytes": x + J * case["C"] + m * case["C"] * _SIZE[case["yt"]], "flops": 2 * m * J * case["C"]}
    J = case["R"] * case["S"] * case["C"]
    return {"bytes": x + J * case["K"] + m * case["K"] * _SIZE[case["yt"]], "flops": 2 * m * case["K"] * J}


def tolerance(case):
    return "exact"   # whole numbers throughout: every correct implementation gives the same bytes


# ---------------------------------------------------------------- the same in 64 bits

def _multiplier(s_in, s_out):
    """Mantissa in [2^30, 2^31) and right shift of s_in / s_out, per element."""
    M = np.asarray(s_in, np.float64)
    f, e = np.frexp(M / np.float64(np.float32(s_out)))
    m = np.floor(f * 2.0**31 + 0.5).astype(np.int64)
    over = m == 1 << 31
    m = np.where(over, 1 << 30, m)
    e = np.where(over, e + 1, e)
    return torch.from_numpy(np.atleast_1d(m)).cuda(), torch.from_numpy(np.atleast_1d(31 - e.astype(np.int64))).cuda()


def _scaled(v, mult, shift, rounding):
    """round(v * mult / 2^shift) of int64 v, as the rounding says."""
    p = v * mult

    def away(p, n):   # nearest, ties away from zero
        half = torch.where(n > 0, torch.ones_like(n) << (n - 1).clamp(min=0), torch.zeros_like(n))
        return torch.where(p >= 0, (p + half) >> n, -((-p + half) >> n))

    if rounding == "half_away":
        return away(p, shift)
    if rounding == "two_stage":
        one = (p + (torch.ones_like(shift) << (shift - 1))) >> shift
        return torch.where(shift >= 31, away((p + (1 << 30)) >> 31, (shift - 31).clamp(min=0)), one)
    return (p + (torch.ones_like(shift) << (shift - 1))) >> shift


def _finish(acc, L, rounding):
    if L["yt"] == "i32":
        return acc.to(torch.int32)
    s = np.float64(np.float32(L["s_x"])) * np.asarray(L["s_w"], np.float64)
    v = _scaled(acc, *_multiplier(s, L["s_y"]), rounding) + L["zp_y"]
    lo, hi = _RANGE[L["yt"]]
    if L["clamp"]:
        lo, hi = max(lo, L["clamp"][0]), min(hi, L["clamp"][1])
    return v.clamp(lo, hi).to(_TORCH[L["yt"]])


def _exact_conv(x, L, R, S, stride, pads, depthwise, rounding="half_up"):
    """One image at a time; float64 holds every sum exactly."""
    pt, pl, pb, pr = pads
    w = L["w"].to(torch.float64) - torch.from_numpy(L["zp_w"]).cuda().to(torch.float64).view(
        (1, 1, -1) if depthwise else (-1, 1, 1, 1))
    out = []
    step = max(1, int(2e8 / (x[0].numel() * R * S + 1)))
    for xs in x.split(step):
        xd = torch.nn.functional.pad(xs.to(torch.float64) - L["zp_x"], (0, 0, pl, pr, pt, pb))
        n, H, W, C = xd.shape
        ho, wo = (H - R) // stride + 1, (W - S) // stride + 1
        acc = 0
        for r in range(R):
            for s in range(S):
                cells = xd[:, r:r + (ho - 1) * stride + 1:stride, s:s + (wo - 1) * stride + 1:stride]
                acc = acc + (cells * w[r, s] if depthwise else
                             (cells.reshape(-1, C) @ w[:, r, s].t().contiguous()).view(n, ho, wo, -1))
        out.append(_finish(acc.to(torch.int64) + L["bias"].to(torch.int64), L, rounding))
    return torch.cat(out)


def _exact_add(a, b, qa, qb, qo, yt, clamp, rounding):
    v = sum(_scaled(t.to(torch.int64) - z, *_multiplier(np.float64(np.float32(s)), qo[0]), rounding)
            for t, (s, z) in ((a, qa), (b, qb))) + qo[1]
    lo, hi = _RANGE[yt]
    if clamp:
        lo, hi = max(lo, clamp[0]), min(hi, clamp[1])
    return v.clamp(lo, hi).to(_TORCH[yt])


def _exact_pool(x, mode, k, stride, pads):
    pt, pl, pb, pr = pads

    def cells(fill, t):
        t = torch.nn.functional.pad(t, (0, 0, pl, pr, pt, pb), value=fill)
        ho, wo = (t.shape[1] - k) // stride + 1, (t.shape[2] - k) // stride + 1
        return [t[:, r:r + (ho - 1) * stride + 1:stride, s:s + (wo - 1) * stride + 1:stride]
                for r in range(k) for s in range(k)]

    if mode == "max":
        return torch.stack(cells(-1000, x.to(torch.int16))).amax(0).to(x.dtype)
    total = sum(cells(0, x.to(torch.int64)))
    count = sum(cells(0, torch.ones_like(x[:1, :, :, :1], dtype=torch.int64)))
    mag = torch.div(2 * total.abs() + count, 2 * count, rounding_mode="floor")   # ties away from zero
    return torch.where(total < 0, -mag, mag).to(x.dtype)


def exact(case, seed):
    inp, kind = _inputs(case, seed), case["kind"]
    x = inp["x"]
    if kind == "add":
        (sa, sb), (za, zb) = inp["s"], inp["z"]
        return _exact_add(x, inp["b"], (sa, za), (sb, zb), (inp["s_y"], inp["zp_y"]), case["yt"], None,
                          case["rounding"])
    if kind == "pool":
        return _exact_pool(x, case["mode"], case["R"], case["stride"], _pads(case["pad_h"], case["pad_h"]))
    if kind == "requantize":
        L = {"s_x": 1.0, "s_w": inp["s"], "s_y": inp["s_y"], "zp_y": inp["zp_y"], "yt": case["yt"], "clamp": None}
        return [_finish(x.to(torch.int64), L, case["rounding"])]
    if kind in ("dense", "ffn"):
        outs = []
        for L in inp["layers"]:
            L = dict(L, w=L["w"][:, None, None, :])
            x = _exact_conv(x[None, None], L, 1, 1, 1, _pads(0, 0), False, case["rounding"])[0, 0]
            outs.append(x)
        return outs
    if kind == "conv":
        return [_exact_conv(x, inp["layers"][0], case["R"], case["S"], case["stride"],
                            _pads(case["pad_h"], case["pad_w"]), False, case["rounding"])]
    if kind == "depthwise":
        p = case["R"] // 2
        return [_exact_conv(x, inp["layers"][0], case["R"], case["R"], case["stride"], _pads(p, p), True,
                            case["rounding"])]
    t, q = {"x0": x}, inp["q"]
    sh = _net_shapes(case["net"], case["N"])
    for st in inp["steps"]:
        src, dst = st["src"], st["dst"]
        if st["kind"] == "pool":
            t[dst] = _exact_pool(t[src[0]], st["mode"], st["k"], st["stride"], st["pads"])
        elif st["kind"] == "add":
            t[dst] = _exact_add(t[src[0]], t[src[1]], q[src[0]], q[src[1]], q[dst], "i8", st["clamp"], "half_up")
        else:
            y = _exact_conv(t[src[0]], st["L"], st["R"], st["S"], st["stride"], st["pads"], st["kind"] == "dw")
            if st["into"]:
                if dst not in t:
                    t[dst] = torch.zeros(sh[dst], dtype=torch.int8, device="cuda")
                t[dst][..., st["into"][1]:st["into"][1] + st["K"]] = y
            else:
                t[dst] = y
    return {k: v for k, v in t.items() if k.endswith("_out")}
