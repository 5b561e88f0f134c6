"""The calls whose speed this framework is held to, with the sizes, layouts
and value distributions they meet in use.

A case is one 3x3 layer in one of the library's forms:

  op "f4", "f2"   wino_f4_conv_int8 (SPLIT) with an F(4x4,3x3) or F(2x2,3x3)
                  plan; bits 8, or 10 for the int8/10 variant
  op "direct"     direct_conv_int8
  op "calibrate"  wino_f4_calibrate_input and wino_f4_calibrate_output, the
                  two passes of post-training calibration over one batch

Everything is integer arithmetic with one correct result, so outputs are
compared exactly.  ``exact`` evaluates the same definition in float64 (every
value involved is an integer below 2^53, or a weight whose transform is
rounded far from a tie) without the library.
"""
import math

import numpy as np
import torch

import paper_2209_12982_amd as W

_LAYOUT = {"nchw": W.NCHW, "nhwc": W.NHWC}


def _case(name, op, layout, n, cin, cout, h, w, bits=8, relu=False, act="relu", outliers=0.0):
    c = dict(op=op, layout=layout, n=n, cin=cin, cout=cout, h=h, w=w, bits=bits, relu=relu, act=act,
             outliers=outliers)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest layer, in its stated layout: launches and host time
        _case("tiny_f2_nchw", "f2", "nchw", 1, 16, 16, 32, 32),
        # first and last 3x3 stages of a ResNet at batch 8; small images, F2
        _case("resnet_first_f2", "f2", "nhwc", 8, 64, 64, 56, 56, relu=True),
        _case("resnet_last_f2", "f2", "nhwc", 8, 256, 256, 14, 14, relu=True),
        # two layers of the paper's comparison table (B, H, W, Cin, Cout =
        # 8, 32, 32, 128, 128 and 8, 32, 32, 256, 512), run with F4 as there
        _case("table_128_128_f4", "f4", "nhwc", 8, 128, 128, 32, 32),
        _case("table_256_512_f4", "f4", "nhwc", 8, 256, 512, 32, 32),
        # a detection head on 300 x 300 inputs: odd image sides, NCHW
        _case("ssd_odd_f4_nchw", "f4", "nchw", 2, 256, 256, 75, 75, relu=True),
        # a UNet's first stage: few channels, large image, NCHW
        _case("unet_first_f4_nchw", "f4", "nchw", 1, 64, 64, 568, 568, relu=True),
        # segmentation backbone and detection neck at high resolution: F4's
        # own ground, the second the largest layer
        _case("segmentation_f4", "f4", "nhwc", 1, 128, 128, 256, 512),
        _case("detection_f4", "f4", "nhwc", 4, 256, 256, 160, 160, outliers=0.01),
        # the accuracy option: 10-bit Winograd domain
        _case("segmentation_f4_i10", "f4", "nhwc", 1, 128, 128, 256, 512, bits=10),
        # layers that are run without Winograd
        _case("segmentation_direct", "direct", "nhwc", 1, 128, 128, 256, 512),
        # one batch of post-training calibration
        _case("segmentation_calibrate", "calibrate", "nhwc", 1, 128, 128, 256, 512),
    ]


def draw(rng):
    """A layer of the same ranges: 1-8 images of 7 to 512 pixels a side, 16 to
    512 channels (one in four not a multiple of 16), either layout."""
    op, bits, cap = rng.choice([("f4", 8, 1.2e11)] * 6 + [("f2", 8, 1.6e10)] * 4 + [("direct", 8, 3.8e10)] * 2 +
                               [("f4", 10, 3.8e10)] * 2 + [("calibrate", 8, 3.8e10)] * 2)
    layout = rng.choice(["nhwc", "nhwc", "nchw"])

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def channels():
        c = log_int(16, 512)
        return c if rng.random() < 0.25 else max(16, (c + 8) // 16 * 16)

    while True:
        n = rng.choice([1, 1, 2, 3, 4, 8])
        h = log_int(7, 512)
        w = max(7, min(512, int(round(h * math.exp(rng.uniform(-0.7, 0.7))))))
        cin, cout = channels(), channels()
        ops = 18.0 * n * h * w * cin * cout
        # the direct convolution's general kernel is the slow one
        limit = cap / 16 if op == "direct" and (cin % 64 or layout == "nchw") else cap
        if 4e6 <= ops <= limit and n * h * w * max(cin, cout) <= 27_000_000:
            break
    return _case(None, op, layout, n, cin, cout, h, w, bits=bits, relu=rng.random() < 0.5,
                 act=rng.choice(["relu", "relu", "signed"]), outliers=rng.choice([0.0, 0.0, 0.01]))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _inputs(case, seed):
    """x int8 (in the case's layout), weights fp32 OIHW, bias int32, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n, cin, cout, h, w = (case[k] for k in ("n", "cin", "cout", "h", "w"))
    shape = (n, h, w, cin) if case["layout"] == "nhwc" else (n, cin, h, w)
    v = torch.randn(shape, device="cuda", generator=g)
    if case["act"] == "relu":
        # what a ReLU leaves: half zeros, the rest half-normal
        v = torch.where(torch.rand(shape, device="cuda", generator=g) < 0.5, torch.zeros_like(v), v.abs() * 24)
    else:
        v = v * 32
    x = v.round_().clamp_(-128, 127).to(torch.int8)
    del v
    f = torch.randn((cout, cin, 3, 3), device="cuda", generator=g) * math.sqrt(2.0 / (9 * cin))
    if case["outliers"]:
        f = torch.where(torch.rand(f.shape, device="cuda", generator=g) < case["outliers"], f * 8, f)
    b = torch.randint(-256, 257, (cout,), device="cuda", generator=g, dtype=torch.int32)
    return x, f.contiguous(), b


def _direct_weights(f):
    """int8 OHWI weights with one power-of-two scale: e is the smallest
    exponent with max |f| <= 128 * 2^e."""
    f = f.double()
    e = math.ceil(math.log2(f.abs().max().item() / 128.0))
    q = torch.floor(f / 2.0 ** e + 0.5).clamp_(-128, 127)
    return q.to(torch.int8).permute(0, 2, 3, 1).contiguous()


def _direct_shift(case):
    # the accumulators' spread is about 2^5 * 2^5 * sqrt(9 cin); keep the
    # outputs spread over the int8 range
    return max(0, int(round(math.log2(math.sqrt(9.0 * case["cin"])))) + 5)


def prepare(case, seed):
    """The tensors, plan and workspace that a program holds before the call."""
    x, f, b = _inputs(case, seed)
    n, cin, cout, h, w = (case[k] for k in ("n", "cin", "cout", "h", "w"))
    layout = _LAYOUT[case["layout"]]
    st = dict(case=case, x=x, layout=layout)
    oshape = (n, h, w, cout) if case["layout"] == "nhwc" else (n, cout, h, w)
    if case["op"] != "calibrate":
        st["y"] = torch.empty(oshape, dtype=torch.int8, device="cuda")
    if case["op"] == "direct":
        st.update(w=_direct_weights(f), b=b, shift=_direct_shift(case))
        torch.cuda.synchronize()
        return st
    bias = b.cpu().numpy()
    if case["bits"] == 10:
        fh = f.cpu().numpy()
        eb, _ = W.wino_f4_calibrate_input_i10(x, n, cin, h, w, layout)
        make = lambda s: W.wino_f4_plan_i10(fh, eb, bias=bias, out_shift=s, relu=case["relu"])
    elif case["op"] == "f2":
        eb, _ = W.wino_f2_calibrate_input(x, n, cin, h, w, layout)
        make = lambda s: W.wino_f2_plan_device(f, eb, bias=bias, out_shift=s, relu=case["relu"])
    else:
        eb, _ = W.wino_f4_calibrate_input(x, n, cin, h, w, layout)
        make = lambda s: W.wino_f4_plan_device(f, eb, bias=bias, out_shift=s, relu=case["relu"])
    plan = make(0)
    ws = torch.empty(W.wino_f4_workspace_bytes(plan, n, h, w), dtype=torch.int8, device="cuda")
    if case["op"] != "calibrate":
        shift, _ = W.wino_f4_calibrate_output(plan, x, n, h, w, layout, ws)
        plan = make(shift)
    st.update(plan=plan, ws=ws)
    torch.cuda.synchronize()
    return st


def run(st):
    """One pass through the public entry point."""
    c = st["case"]
    n, h, w = c["n"], c["h"], c["w"]
    if c["op"] == "direct":
        W.direct_conv_int8(st["x"], st["w"], st["b"], st["y"], n, c["cin"], c["cout"], h, w, st["layout"],
                           st["shift"], c["relu"])
        return st["y"]
    if c["op"] == "calibrate":
        e_b, absmax = W.wino_f4_calibrate_input(st["x"], n, c["cin"], h, w, st["layout"])
        shift, zmax = W.wino_f4_calibrate_output(st["plan"], st["x"], n, h, w, st["layout"], st["ws"])
        return np.array(list(e_b) + list(absmax) + [shift, zmax], dtype=np.int64)
    W.wino_f4_conv_int8(st["plan"], st["x"], st["y"], n, h, w, st["layout"], W.SPLIT, st["ws"])
    return st["y"]


def work(case):
    """Bytes and operations that no implementation of the call avoids: the
    input read once, the int8 output written once, the weights in the form
    that the call takes, and the multiply-adds of the algorithm it names."""
    n, cin, cout, h, w = (case[k] for k in ("n", "cin", "cout", "h", "w"))
    xb, yb = n * h * w * cin, n * h * w * cout
    if case["op"] == "direct":
        return {"bytes": xb + yb + 9 * cin * cout + 4 * cout, "flops": 18 * n * h * w * cin * cout}
    m = 2 if case["op"] == "f2" else 4
    taps = (m + 2) ** 2
    tiles = n * (-(-h // m)) * (-(-w // m))
    wb = taps * cin * cout * (2 if case["bits"] == 10 else 1) + 4 * cout
    flops = 2 * taps * tiles * cin * cout
    if case["op"] == "calibrate":
        return {"bytes": xb + wb, "flops": flops}     # x, no int8 output
    return {"bytes": xb + yb + wb, "flops": flops}


def tolerance(case):
    return "exact"


# --------------------------------------------------------------------------
# the definition in float64
# --------------------------------------------------------------------------
_F4 = dict(
    bt=[[4, 0, -5, 0, 1, 0], [0, -4, -4, 1, 1, 0], [0, 4, -4, -1, 1, 0],
        [0, -2, -1, 2, 1, 0], [0, 2, -1, -2, 1, 0], [0, 4, 0, -5, 0, 1]],
    g=[[6, 0, 0], [-4, -4, -4], [-4, 4, -4], [1, 2, 4], [1, -2, 4], [0, 0, 24]], den=24,
    at=[[1, 1, 1, 1, 1, 0], [0, 1, -1, 2, -2, 0], [0, 1, 1, 4, 4, 0], [0, 1, -1, 8, -8, 1]])
_F2 = dict(
    bt=[[1, 0, -1, 0], [0, 1, 1, 0], [0, -1, 1, 0], [0, 1, 0, -1]],
    g=[[2, 0, 0], [1, 1, 1], [1, -1, 1], [0, 0, 2]], den=2,
    at=[[1, 1, 1, 0], [0, 1, -1, -1]])


def _ceil_exp(a, rail):
    """Smallest e >= any integer with a <= rail * 2^e (0 for a = 0)."""
    if a == 0:
        return 0
    e = math.frexp(a / rail)[1]          # a / rail = m 2^e, 1/2 <= m < 1
    return e - 1 if a <= rail * 2.0 ** (e - 1) else e


def exact(case, seed):
    dev = torch.device("cuda")
    x, f, b = _inputs(case, seed)
    n, cin, cout, h, w = (case[k] for k in ("n", "cin", "cout", "h", "w"))
    nchw = x if case["layout"] == "nchw" else x.permute(0, 3, 1, 2)
    if case["op"] == "direct":
        wq = _direct_weights(f).permute(0, 3, 1, 2).double()
        xp = torch.nn.functional.pad(nchw.double(), (1, 1, 1, 1)).permute(1, 0, 2, 3).contiguous()
        z = torch.zeros((cout, n * h * w), dtype=torch.float64, device=dev)
        for r in range(3):
            for s in range(3):
                z += wq[:, :, r, s].contiguous() @ xp[:, :, r:r + h, s:s + w].reshape(cin, -1)
        z += b.double()[:, None]
        out = torch.floor((z + (2.0 ** _direct_shift(case) / 2 if _direct_shift(case) else 0.0)) /
                          2.0 ** _direct_shift(case))
        out = out.clamp_(0 if case["relu"] else -128, 127).reshape(cout, n, h, w)
        return out.permute(1, 2, 3, 0).contiguous() if case["layout"] == "nhwc" else out.permute(1, 0, 2, 3).contiguous()

    m, t = (2, _F2) if case["op"] == "f2" else (4, _F4)
    k = m + 2
    bt, g, at = (torch.tensor(t[key], dtype=torch.float64, device=dev) for key in ("bt", "g", "at"))
    rail = 512 if case["bits"] == 10 else 128
    th, tw = -(-h // m), -(-w // m)
    xp = torch.nn.functional.pad(nchw.double(), (1, m * tw + 1 - w, 1, m * th + 1 - h)).permute(1, 0, 2, 3)
    # d[a][b]: pixel (a, b) of every tile, [cin, tiles]
    d = [[xp[:, :, a:a + m * th - m + 1:m, c:c + m * tw - m + 1:m].reshape(cin, -1) for c in range(k)]
         for a in range(k)]
    rows = [[sum(bt[a, i].item() * d[i][c] for i in range(k) if t["bt"][a][i]) for c in range(k)] for a in range(k)]
    del d
    u = torch.einsum("ai,ocij,bj->aboc", g.cpu(), f.double().cpu(), g.cpu()).to(dev)     # den^2 U
    den2 = float(t["den"] ** 2)
    eb, absmax, eg, mt = [], [], [], []
    for a in range(k):
        for c in range(k):
            v = sum(bt[c, j].item() * rows[a][j] for j in range(k) if t["bt"][c][j])
            absmax.append(int(v.abs().max().item()))
            eb.append(min(15, max(0, _ceil_exp(absmax[-1], rail))))
            eg.append(_ceil_exp(u[a, c].abs().max().item() / den2, rail))
            vq = torch.floor(v / 2.0 ** eb[-1] + 0.5).clamp_(-rail, rail - 1)
            uq = torch.floor(u[a, c] / (den2 * 2.0 ** eg[-1]) + 0.5).clamp_(-rail, rail - 1)
            mt.append(uq @ vq)
    e = [p + q for p, q in zip(eb, eg)]
    mt = [v * 2.0 ** (q - min(e)) for v, q in zip(mt, e)]
    z = torch.empty((cout, n, th, m, tw, m), dtype=torch.float64, device=dev)
    for i in range(m):
        for j in range(m):
            y = sum(at[i, a].item() * at[j, c].item() * mt[k * a + c] for a in range(k) for c in range(k)
                    if t["at"][i][a] and t["at"][j][c])
            z[:, :, :, i, :, j] = y.reshape(cout, n, th, tw)
    z = z.reshape(cout, n, m * th, m * tw)[:, :, :h, :w] + b.double()[:, None, None, None]
    zmax = int(z.abs().max().item())
    shift = min(62, max(0, _ceil_exp(zmax, 128)))
    if case["op"] == "calibrate":
        return np.array(eb + absmax + [shift, zmax], dtype=np.int64)
    out = torch.floor((z + (2.0 ** (shift - 1) if shift else 0.0)) / 2.0 ** shift)
    out = out.clamp_(0 if case["relu"] else -128, 127)
    return out.permute(1, 2, 3, 0).contiguous() if case["layout"] == "nhwc" else out.permute(1, 0, 2, 3).contiguous()
