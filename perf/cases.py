"""The work a user of this library has it do, as cases that can be timed and compared.

Kinds of case (key "kind"):
  pw          one ternary pointwise layer                       prom_pw_conv
  pw_seq      every pointwise layer of a network at once        PwSequence.run
  dw_seq      every depthwise layer of MobileNetV2 at once      DwSequence.run
  gconv_seq   every grouped 3x3 layer of a network at once      GconvSequence.run
  block       one inverted-residual block                       prom_block
  chain       MobileNetV2's body, each block on the output of the one before
                                                                prom_dw_conv, prom_pw_conv, prom_block
  bottleneck  RegNetX's or ResNeXt's body, layer after layer    prom_pw_conv, prom_gconv3x3
  dynq        a pointwise layer with the dynamic output scale   prom_pw_conv_dynq
  quant       dynamic quantisation of float32 activations       prom_quantize_activation_absmax

Weights, folded requantisation parameters, packed forms, layer tables, output buffers and the block
workspace are what a program sets up once; a pass is the calls a forward pass makes.  The multipliers
are drawn so that a layer's outputs have a spread of about 40 codes, as calibrated scales give.
Every result is a whole number, or a float32 whose operations and roundings the interface fixes, so
the tolerance is "exact" throughout."""
import math

import numpy as np
import torch

import paper_2505_03254_amd as P
from workloads.grouped import (regnetx_400mf_grouped_layers, regnetx_400mf_pointwise_layers,
                               resnext50_32x4d_grouped_layers, resnext50_32x4d_pointwise_layers)
from workloads.mobilenetv2 import (mobilenetv2_blocks, mobilenetv2_depthwise_layers,
                                   mobilenetv2_pointwise_layers)

PW_TABLES = {"mobilenetv2": mobilenetv2_pointwise_layers, "regnetx400": regnetx_400mf_pointwise_layers,
             "resnext50": resnext50_32x4d_pointwise_layers}
GCONV_TABLES = {"regnetx400": regnetx_400mf_grouped_layers, "resnext50": resnext50_32x4d_grouped_layers}


def listed():
    return [
        # one small layer for one image: what a call costs when there is hardly any work in it
        dict(name="pw 14x14 64-384 b1", kind="pw", n=1, h=14, w=14, cin=64, cout=384, residual=False, prelu=False),
        # an early expansion layer at a serving batch: few input channels, many pixels, mostly output
        dict(name="pw 56x56 24-144 b32", kind="pw", n=32, h=56, w=56, cin=24, cout=144, residual=False, prelu=False),
        # a deep projection layer with the skip connection: many input channels, few pixels
        dict(name="pw 7x7 960-160 res b256", kind="pw", n=256, h=7, w=7, cin=960, cout=160, residual=True, prelu=False),
        # a wide layer of a ResNeXt bottleneck: the contraction itself is the work
        dict(name="pw 14x14 512-1024 b128", kind="pw", n=128, h=14, w=14, cin=512, cout=1024, residual=False, prelu=False),
        # the benchmark's sweep: the 34 pointwise layers of MobileNetV2 in one call
        dict(name="pw sweep mobilenetv2 b128", kind="pw_seq", net="mobilenetv2", n=128, prelu=False),
        # the 17 depthwise layers of MobileNetV2 in one call
        dict(name="dw sweep mobilenetv2 b128", kind="dw_seq", n=128, prelu=False),
        # the 22 grouped layers of RegNetX-400MF in one call
        dict(name="gconv sweep regnetx b128", kind="gconv_seq", net="regnetx400", n=128, prelu=True),
        # one inverted-residual block with its skip connection
        dict(name="block 28x28 32-192-32 b64", kind="block", n=64, h=28, w=28, cin=32, t=6, cout=32, stride=1, prelu=False),
        # MobileNetV2's body on a few images, with the PReLU activations of the paper's models
        dict(name="chain mobilenetv2 b8", kind="chain", n=8, hw=112, prelu=True),
        # MobileNetV2's body at a throughput batch
        dict(name="chain mobilenetv2 b128", kind="chain", n=128, hw=112, prelu=False),
        # ResNeXt-50's body: 36 pointwise and 16 grouped layers, each on the output of the one before
        dict(name="bottlenecks resnext50 b64", kind="bottleneck", net="resnext50", n=64, prelu=False),
        # a layer that quantises its own output with the dynamic scale of each image
        dict(name="dynq 56x56 24-144 b128", kind="dynq", n=128, h=56, w=56, cin=24, cout=144, relu=True, bias=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """A channel count of a network: a multiple of 8, now and then of 4 only."""
    c = _log(rng, lo, hi)
    return max(lo, c // 8 * 8) if rng.random() < 0.9 else max(lo, c // 4 * 4)


def _pixels(rng, hw, channels, most):
    """A batch for h x w images of so many channels (in and out) that the layer moves at most `most` bytes."""
    h = hw if rng.random() < 0.6 else max(1, hw + rng.randint(-3, 3))
    w = h if rng.random() < 0.7 else max(1, hw + rng.randint(-3, 3))
    n = _log(rng, 1, max(1, min(256, most // (h * w * channels))))
    return n, h, w


def draw(rng):
    kind = rng.choice(["pw", "pw", "pw", "pw", "pw_seq", "dw_seq", "gconv_seq", "block", "block", "chain",
                       "bottleneck", "dynq", "quant"])
    prelu = rng.random() < 0.3
    if kind == "pw":
        hw = rng.choice([7, 14, 28, 56, 112])
        top = {7: 2048, 14: 1024, 28: 512, 56: 256, 112: 96}[hw]
        cin, cout = _channels(rng, 16, top), _channels(rng, 16, top)
        n, h, w = _pixels(rng, hw, cin + cout, 150_000_000)
        return dict(kind="pw", n=n, h=h, w=w, cin=cin, cout=cout, residual=rng.random() < 0.4, prelu=prelu)
    if kind == "pw_seq":
        net = rng.choice(sorted(PW_TABLES))
        return dict(kind="pw_seq", net=net, n=_log(rng, 1, 64 if net == "resnext50" else 128), prelu=prelu)
    if kind == "dw_seq":
        return dict(kind="dw_seq", n=_log(rng, 1, 160), prelu=prelu)
    if kind == "gconv_seq":
        return dict(kind="gconv_seq", net=rng.choice(sorted(GCONV_TABLES)), n=_log(rng, 1, 128), prelu=prelu)
    if kind == "block":
        hw = rng.choice([7, 14, 28, 56, 112])
        cin = _channels(rng, *{7: (96, 192), 14: (32, 128), 28: (24, 64), 56: (16, 32), 112: (16, 24)}[hw])
        t = rng.choice([3, 4, 6, 6, 6])
        stride = rng.choice([1, 1, 2])
        cout = cin if stride == 1 and rng.random() < 0.7 else _channels(rng, cin, min(320, 2 * cin))
        n, h, w = _pixels(rng, hw, cin * t * 2, 300_000_000)
        return dict(kind="block", n=n, h=h, w=w, cin=cin, t=t, cout=cout, stride=stride, prelu=prelu)
    if kind == "chain":
        return dict(kind="chain", n=_log(rng, 1, 128), hw=rng.choice([112, 112, 112, 96, 80, 64, 113]), prelu=prelu)
    if kind == "bottleneck":
        return dict(kind="bottleneck", net=rng.choice(sorted(GCONV_TABLES)), n=_log(rng, 1, 64), prelu=prelu)
    if kind == "dynq":
        hw = rng.choice([7, 14, 28, 56])
        cin = _channels(rng, 16, {7: 960, 14: 576, 28: 192, 56: 144}[hw])
        cout = max(16, _channels(rng, 16, {7: 960, 14: 576, 28: 192, 56: 144}[hw]) // 16 * 16)
        n, h, w = _pixels(rng, hw, cin + cout, 80_000_000)
        return dict(kind="dynq", n=n, h=h, w=w, cin=cin, cout=cout, relu=rng.random() < 0.5, bias=rng.random() < 0.7)
    hw = rng.choice([7, 14, 28, 56, 112])
    c = _channels(rng, 16, {7: 1280, 14: 576, 28: 256, 56: 144, 112: 96}[hw])
    n, h, w = _pixels(rng, hw, 5 * c, 300_000_000)
    return dict(kind="quant", n=n, h=h, w=w, c=c)


# ---- inputs ---------------------------------------------------------------------------------------
class _Draw:
    """Seeded inputs on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def ints(self, lo, hi, shape, dtype):
        return torch.randint(lo, hi + 1, shape, generator=self.g, device="cuda", dtype=dtype)

    def acts(self, *shape):
        return self.ints(0, 127, shape, torch.int8)

    def ternary(self, cout, cin):
        u = self.ints(0, 3, (cout, cin), torch.int8)
        return torch.where(u == 2, -1, torch.where(u == 3, 0, u)).to(torch.int8)

    def requant(self, c, acc_std, lo, hi, prelu):
        """Scales around 40 / (standard deviation of the accumulators), as multiplier and shift."""
        u = torch.rand(c, generator=self.g, device="cuda", dtype=torch.float64)
        scale = ((0.7 + 0.7 * u) * 40.0 / acc_std).cpu().numpy()
        shift = np.maximum(0, np.floor(-np.log2(scale)).astype(np.int32))
        mult = np.minimum(np.floor(scale * 2.0 ** (31 + shift)), 2.0 ** 31 - 1).astype(np.int64)
        bias = (self.ints(-1000, 1000, (c,), torch.int32).to(torch.float64) * (acc_std / 1000.0)).to(torch.int32)
        neg = None
        if prelu:  # slopes of -0.25 .. 1, folded into the multiplier
            k = self.ints(-64, 255, (c,), torch.int32).cpu().numpy().astype(np.int64)
            neg = torch.from_numpy(((mult * k) >> 8).astype(np.int32)).cuda()
            lo, hi = -128, 127
        return P.Requant(bias, torch.from_numpy(mult.astype(np.int32)).cuda(), torch.from_numpy(shift).cuda(), lo, hi, neg)


def _pw_std(cin):
    return 52.0 * math.sqrt(cin)  # half of the weights are zero, inputs have a mean square of about 74^2


def _pw_layer(d, cin, cout, lo, hi, prelu):
    w = d.ternary(cout, cin)
    packed = torch.from_numpy(P.prom_pack_ternary(w.cpu().numpy())).cuda()
    return dict(w=w, packed=packed, cout=cout, rq=d.requant(cout, _pw_std(cin), lo, hi, prelu))


def _dw_layer(d, c, stride, prelu):
    return dict(w=d.ints(-127, 127, (3, 3, c), torch.int8), stride=stride, rq=d.requant(c, 3 * 74.0 * 73.0, 0, 127, prelu))


def _gconv_layer(d, c, gs, stride, prelu):
    w = d.ints(-127, 127, (3, 3, c, gs), torch.int8)
    frag = torch.from_numpy(P.prom_gconv_pack(w.cpu().numpy())).cuda() if P.prom_gconv_frag_size(c, gs) else None
    return dict(w=w, frag=frag, stride=stride, rq=d.requant(c, 3 * math.sqrt(gs) * 74.0 * 73.0, 0, 127, prelu))


def _empty(*shape):
    return torch.empty(shape, dtype=torch.int8, device="cuda")


def _down(hw, stride):
    return (hw - 1) // stride + 1


def _bottlenecks(case):
    """(name, kind, ...) of a bottleneck network's layers in order: the grouped layer stands between a
    block's first and last pointwise layer."""
    pw = {s.name: s for s in PW_TABLES[case["net"]]()}
    return [(g, pw[g.name + ".reduce"], pw.get(g.name + ".shortcut"), pw[g.name + ".expand"])
            for g in GCONV_TABLES[case["net"]]()]


def _inputs(case, seed):
    """Everything random of a case: the input and the layers."""
    d, k = _Draw(seed), case["kind"]
    n, prelu = case["n"], case.get("prelu", False)
    s = {"case": case}
    if k == "pw":
        s["x"] = d.acts(n, case["h"], case["w"], case["cin"])
        lo = -128 if case["residual"] else 0
        s["L"] = _pw_layer(d, case["cin"], case["cout"], lo, 127, prelu)
        s["res"] = d.ints(-64, 63, (n, case["h"], case["w"], case["cout"]), torch.int8) if case["residual"] else None
    elif k == "pw_seq":
        s["layers"] = []
        for p in PW_TABLES[case["net"]]():
            x = d.acts(n, p.hw, p.hw, p.cin)
            s["layers"].append((x, _pw_layer(d, p.cin, p.cout, 0, 127, prelu)))
    elif k == "dw_seq":
        s["layers"] = [(d.acts(n, p.hw_in, p.hw_in, p.c), _dw_layer(d, p.c, p.stride, prelu))
                       for p in mobilenetv2_depthwise_layers()]
    elif k == "gconv_seq":
        s["layers"] = [(d.acts(n, p.hw_in, p.hw_in, p.c), _gconv_layer(d, p.c, p.gs, p.stride, prelu))
                       for p in GCONV_TABLES[case["net"]]()]
    elif k == "block":
        cin, chid, cout = case["cin"], case["cin"] * case["t"], case["cout"]
        s["x"] = d.acts(n, case["h"], case["w"], cin)
        s["B"] = (_pw_layer(d, cin, chid, 0, 127, prelu), _dw_layer(d, chid, case["stride"], prelu),
                  _pw_layer(d, chid, cout, -128, 127, False))
    elif k == "chain":
        s["blocks"] = mobilenetv2_blocks(case["hw"])
        s["x"] = d.acts(n, case["hw"], case["hw"], s["blocks"][0].cin)
        s["layers"] = [(_pw_layer(d, b.cin, b.cin * b.t, 0, 127, prelu) if b.t > 1 else None,
                        _dw_layer(d, b.cin * b.t, b.stride, prelu),
                        _pw_layer(d, b.cin * b.t, b.cout, -128, 127, False)) for b in s["blocks"]]
    elif k == "bottleneck":
        s["blocks"] = _bottlenecks(case)
        s["x"] = d.acts(n, s["blocks"][0][0].hw_in, s["blocks"][0][0].hw_in, s["blocks"][0][1].cin)
        s["layers"] = [(_pw_layer(d, r.cin, r.cout, 0, 127, prelu), _gconv_layer(d, g.c, g.gs, g.stride, prelu),
                        _pw_layer(d, c.cin, c.cout, -128, 127, False) if c else None,
                        _pw_layer(d, e.cin, e.cout, -128, 127, False)) for g, r, c, e in s["blocks"]]
    elif k == "dynq":
        s["x"] = d.acts(n, case["h"], case["w"], case["cin"])
        s["L"] = _pw_layer(d, case["cin"], case["cout"], 0, 127, False)
        r = lambda c, lo, hi: lo + (hi - lo) * torch.rand(c, generator=d.g, device="cuda", dtype=torch.float32)
        s["x_step"], s["w_scale"] = r(n, 0.01, 0.08), r(case["cout"], 0.02, 0.3)
        s["bias"] = r(case["cout"], -1.0, 1.0) if case["bias"] else None
    elif k == "quant":
        s["x"] = torch.randn((n, case["h"], case["w"], case["c"]), generator=d.g, device="cuda", dtype=torch.float32)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    k, n = case["kind"], case["n"]
    if k == "pw":
        s["y"] = _empty(n, case["h"], case["w"], case["cout"])
    elif k == "pw_seq":
        s["y"] = [_empty(*x.shape[:3], L["cout"]) for x, L in s["layers"]]
        s["seq"] = P.PwSequence([(x, L["packed"], L["cout"], L["rq"], None, y) for (x, L), y in zip(s["layers"], s["y"])])
    elif k in ("dw_seq", "gconv_seq"):
        s["y"] = [_empty(n, _down(x.shape[1], L["stride"]), _down(x.shape[2], L["stride"]), x.shape[3]) for x, L in s["layers"]]
        if k == "dw_seq":
            s["seq"] = P.DwSequence([(x, L["w"], L["stride"], L["rq"], y) for (x, L), y in zip(s["layers"], s["y"])])
        else:
            s["seq"] = P.GconvSequence([(x, L["w"], L["stride"], L["rq"], y, L["frag"]) for (x, L), y in zip(s["layers"], s["y"])])
    elif k == "block":
        s["y"] = _empty(n, _down(case["h"], case["stride"]), _down(case["w"], case["stride"]), case["cout"])
        size = P.prom_block_workspace_size(n, case["h"], case["w"], case["cin"], case["cin"] * case["t"], case["cout"], case["stride"])
        s["workspace"] = _empty(max(size, 256))
    elif k == "chain":
        sizes = [P.prom_block_workspace_size(n, b.hw_in, b.hw_in, b.cin, b.cin * b.t, b.cout, b.stride) for b in s["blocks"]]
        s["workspace"] = _empty(max(sizes))
        s["y"] = [_empty(n, _down(b.hw_in, b.stride), _down(b.hw_in, b.stride), b.cout) for b in s["blocks"]]
        b = s["blocks"][0]
        s["t"] = _empty(n, _down(b.hw_in, b.stride), _down(b.hw_in, b.stride), b.cin)
    elif k == "bottleneck":
        s["t"] = [(_empty(n, r.hw, r.hw, r.cout), _empty(n, e.hw, e.hw, e.cin), _empty(n, c.hw, c.hw, c.cout) if c else None)
                  for g, r, c, e in s["blocks"]]
        s["y"] = [_empty(n, e.hw, e.hw, e.cout) for g, r, c, e in s["blocks"]]
    elif k == "dynq":
        s["q"] = _empty(n, case["h"], case["w"], case["cout"])
        s["amax"], s["scale"] = (torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(2))
    elif k == "quant":
        s["q"], s["scale"] = _empty(*s["x"].shape), torch.empty(n, dtype=torch.float32, device="cuda")
    return s


# ---- a pass ---------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    k = case["kind"]
    if k == "pw":
        return P.prom_pw_conv(s["x"], s["L"]["packed"], case["cout"], s["L"]["rq"], s["res"], s["y"])
    if k in ("pw_seq", "dw_seq", "gconv_seq"):
        s["seq"].run()
        return s["y"]
    if k == "block":
        return _block(s["x"], s["B"], case["stride"], s["workspace"], s["y"])
    if k == "chain":
        x = s["x"]
        for b, (E, D, Q), y in zip(s["blocks"], s["layers"], s["y"]):
            if E is None:
                P.prom_dw_conv(x, D["w"], b.stride, D["rq"], s["t"])
                P.prom_pw_conv(s["t"], Q["packed"], b.cout, Q["rq"], None, y)
            else:
                _block(x, (E, D, Q), b.stride, s["workspace"], y)
            x = y
        return s["y"]
    if k == "bottleneck":
        x = s["x"]
        for (R, G, C, E), (t1, t2, t3), y in zip(s["layers"], s["t"], s["y"]):
            skip = x
            P.prom_pw_conv(x, R["packed"], R["cout"], R["rq"], None, t1)
            P.prom_gconv3x3(t1, G["w"], G["stride"], G["rq"], t2, None, G["frag"])
            if C is not None:  # the shortcut reads every stride-th pixel
                sub = x if G["stride"] == 1 else x[:, ::G["stride"], ::G["stride"]].contiguous()
                skip = P.prom_pw_conv(sub, C["packed"], C["cout"], C["rq"], None, t3)
            P.prom_pw_conv(t2, E["packed"], E["cout"], E["rq"], skip, y)
            x = y
        return s["y"]
    if k == "dynq":
        return P.prom_pw_conv_dynq(s["x"], s["L"]["packed"], case["cout"], s["x_step"], s["w_scale"], s["bias"], case["relu"],
                                   1e-5, s["q"], s["amax"], s["scale"])
    return P.prom_quantize_activation_absmax(s["x"], 1e-5, s["q"], s["scale"])


def _block(x, layers, stride, workspace, y):
    E, D, Q = layers
    skip = stride == 1 and x.shape[3] == Q["cout"]
    return P.prom_block(x, E["cout"], Q["cout"], stride, E["packed"], E["rq"], D["w"], D["rq"], Q["packed"], Q["rq"], skip,
                        workspace, y)


# ---- what a pass cannot do without ------------------------------------------------------------------
def _pw_work(m, cin, cout, residual=False):
    return m * (cin + cout * (2 if residual else 1)) + cout * (cin / 4 + 12), 2.0 * m * cin * cout


def _tap_work(n, h, c, gs, stride, w=None):
    m = n * _down(h, stride) * _down(w or h, stride)
    return n * h * (w or h) * c + m * c + c * (9 * gs + 12), 18.0 * m * c * gs


def _block_work(n, h, w, cin, t, cout, stride):
    """A block reads its input and writes its output; what lies between need not leave the chip."""
    chid, mo = cin * t, n * _down(h, stride) * _down(w, stride)
    flops = (2.0 * n * h * w * cin * chid if t > 1 else 0) + 18.0 * mo * chid + 2.0 * mo * chid * cout
    weights = (chid * (cin / 4 + 12) if t > 1 else 0) + chid * 21 + cout * (chid / 4 + 12)
    return n * h * w * cin + mo * cout + weights, flops


def work(case):
    k, n = case["kind"], case["n"]
    if k == "pw":
        parts = [_pw_work(n * case["h"] * case["w"], case["cin"], case["cout"], case["residual"])]
    elif k == "pw_seq":
        parts = [_pw_work(n * p.hw * p.hw, p.cin, p.cout) for p in PW_TABLES[case["net"]]()]
    elif k == "dw_seq":
        parts = [_tap_work(n, p.hw_in, p.c, 1, p.stride) for p in mobilenetv2_depthwise_layers()]
    elif k == "gconv_seq":
        parts = [_tap_work(n, p.hw_in, p.c, p.gs, p.stride) for p in GCONV_TABLES[case["net"]]()]
    elif k == "block":
        parts = [_block_work(n, case["h"], case["w"], case["cin"], case["t"], case["cout"], case["stride"])]
    elif k == "chain":
        parts = [_block_work(n, b.hw_in, b.hw_in, b.cin, b.t, b.cout, b.stride) for b in mobilenetv2_blocks(case["hw"])]
    elif k == "bottleneck":
        parts = []
        for g, r, c, e in _bottlenecks(case):
            parts += [_pw_work(n * r.hw * r.hw, r.cin, r.cout), _tap_work(n, g.hw_in, g.c, g.gs, g.stride),
                      _pw_work(n * e.hw * e.hw, e.cin, e.cout, True)]
            parts += [_pw_work(n * c.hw * c.hw, c.cin, c.cout)] if c else []
    elif k == "dynq":
        b, f = _pw_work(n * case["h"] * case["w"], case["cin"], case["cout"])
        parts = [(b + 8 * n, f)]
    else:
        e = n * case["h"] * case["w"] * case["c"]
        parts = [(5 * e + 4 * n, 2.0 * e)]
    return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}


def tolerance(case):
    return "exact"


# ---- the same in plain torch, 64 bits -----------------------------------------------------------------
def _requant(acc, rq, residual=None):
    """acc: float64 whole numbers [..., c]."""
    s = acc.to(torch.int64) + rq.bias.to(torch.int64)
    m = rq.mult.to(torch.int64)
    if rq.mult_neg is not None:
        m = torch.where(s >= 0, m, rq.mult_neg.to(torch.int64))
    sh = rq.shift.to(torch.int64)
    q = (s * m + (torch.ones_like(sh) << (30 + sh))) >> (31 + sh)
    q = q.clamp(rq.act_min, rq.act_max)
    if residual is not None:
        q = (q + residual.to(torch.int64)).clamp(-128, 127)
    return q.to(torch.int8)


def _ref_pw(x, L, residual=None):
    w = L["w"].double().t().contiguous()
    return torch.cat([_requant(x[i:i + 16].double() @ w, L["rq"], None if residual is None else residual[i:i + 16])
                      for i in range(0, x.shape[0], 16)])


def _ref_taps(x, w, stride, rq):
    """w: [3][3][c][gs]."""
    c, gs = w.shape[2], w.shape[3]
    out = []
    for i in range(0, x.shape[0], 16):
        p = torch.nn.functional.pad(x[i:i + 16].double(), (0, 0, 1, 1, 1, 1))
        n, ho, wo = p.shape[0], _down(x.shape[1], stride), _down(x.shape[2], stride)
        acc = torch.zeros((n, ho, wo, c), dtype=torch.float64, device=x.device)
        for a in range(3):
            for b in range(3):
                v = p[:, a:a + (ho - 1) * stride + 1:stride, b:b + (wo - 1) * stride + 1:stride]
                if gs == 1:
                    acc += v * w[a, b, :, 0].double()
                else:
                    v = v.reshape(-1, c // gs, gs).transpose(0, 1).contiguous()
                    u = w[a, b].double().reshape(c // gs, gs, gs).transpose(1, 2).contiguous()
                    acc += torch.bmm(v, u).transpose(0, 1).reshape(n, ho, wo, c)
        out.append(_requant(acc, rq))
    return torch.cat(out)


def _ref_block(x, layers, stride):
    E, D, Q = layers
    t = _ref_pw(x, E) if E is not None else x
    t = _ref_taps(t, D["w"].unsqueeze(3), stride, D["rq"])
    return _ref_pw(t, Q, x if E is not None and stride == 1 and x.shape[3] == Q["cout"] else None)


def exact(case, seed):
    s, k = _inputs(case, seed), case["kind"]
    if k == "pw":
        return _ref_pw(s["x"], s["L"], s["res"])
    if k == "pw_seq":
        return [_ref_pw(x, L) for x, L in s["layers"]]
    if k == "dw_seq":
        return [_ref_taps(x, L["w"].unsqueeze(3), L["stride"], L["rq"]) for x, L in s["layers"]]
    if k == "gconv_seq":
        return [_ref_taps(x, L["w"], L["stride"], L["rq"]) for x, L in s["layers"]]
    if k == "block":
        return _ref_block(s["x"], s["B"], case["stride"])
    if k == "chain":
        x, out = s["x"], []
        for b, layers in zip(s["blocks"], s["layers"]):
            x = _ref_block(x, layers, b.stride)
            out.append(x)
        return out
    if k == "bottleneck":
        x, out = s["x"], []
        for R, G, C, E in s["layers"]:
            t = _ref_taps(_ref_pw(x, R), G["w"], G["stride"], G["rq"])
            skip = x if C is None else _ref_pw(x[:, ::G["stride"], ::G["stride"]], C)
            x = _ref_pw(t, E, skip)
            out.append(x)
        return out
    if k == "dynq":  # the codes follow from float32 roundings that the interface fixes
        n = case["n"]
        z = (s["x"].double().reshape(n, -1, case["cin"]) @ s["L"]["w"].double().t()) * s["w_scale"].double()
        z = z * s["x_step"].double().reshape(n, 1, 1)
        z = z if s["bias"] is None else z + s["bias"].double()
        amax = (z.clamp(min=0) if case["relu"] else z.abs()).reshape(n, -1).max(1).values
        return None, amax, 127.0 / amax.clamp(min=1e-5)
    scale = 127.0 / s["x"].double().abs().reshape(case["n"], -1).max(1).values.clamp(min=1e-5)
    return None, scale
