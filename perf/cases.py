"""The work a user of the library has it do, as cases that can be timed.

Each case goes through the package's public entry points on the shapes of the
networks this repository ships shapes for (ResNet-50/101 and AlexNet
convolutions and fully-connected layers, tests/ and bench.py), from single
calls at a few rows to whole residual blocks at batch 64:

  gemm       fgq_gemm on prepared weights, fp32 output
  conv       fgq_conv2d on prepared weights, fp32 output; with quant=True the
             layer's input is quantized first (fgq_quantize_act, dynamic scale)
  block      a bottleneck block with fp32 group scales: fgq_conv2d_q,
             fgq_conv2d_q, fgq_conv2d_residual_q
  block_dfp  the same block with fixed-point group scales (the paper's
             pipeline): fgq_conv2d_dfp twice, fgq_conv2d_dfp_residual
  stem       the first layer at 8-bit weights: fgq_conv2d_w8, 8-bit codes out
  fc         a fully-connected layer with fp32 group scales: fgq_gemm_ws
  fc_dfp     the same with fixed-point scales, codes out: fgq_gemm_dfp_ws
  direct     fgq_conv2d without prepared weights (the exact kernel: channel
             counts the matrix-core layouts do not take, scales that fail the
             accuracy guard)
  ternarize  fgq_ternarize of a layer's weights (model conversion)
  net        a whole ResNet-50 forward pass, the paper's pipeline with static
             scales, replayed from the graph a serving program captures once

Weights are He-Gaussian, activations ReLU-Gaussian (about half zeros), as in
fgq_inputs.py, drawn on the GPU from the seed.  Weight magnitudes have a floor
of 0.05 standard deviations, so that no group of four has a scale so far below
its channel's largest that the accuracy guard would send the layer to the
direct kernel for some seeds and not for others; the direct kernel has a case
of its own.
"""
import math

import torch
import torch.nn.functional as F

import paper_1705_01462_amd as fgq

DEV = "cuda"


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------

def listed():
    return [
        # one small fully-connected product: latency of a single call
        dict(name="gemm_small", kind="gemm", M=64, K=256, O=128, G=4, bits=8),
        # a layer between fp32 neighbours, batch 32: quantize its input, then
        # the 3x3 convolution, groups of 4 (the benchmark's step)
        dict(name="conv3x3_g4", kind="conv", B=32, H=28, W=28, C=128, O=128, R=3, stride=1, G=4, bits=8, quant=True),
        # a layer whose input is already in codes, 1x1, groups of 64, odd
        # image size: bound by the bytes of its fp32 output
        dict(name="conv1x1_g64", kind="conv", B=32, H=55, W=57, C=256, O=64, R=1, stride=1, G=64, bits=8, quant=False),
        # ResNet-101's most frequent block (third stage, batch 64), 4-bit
        # activations and groups of 64
        dict(name="block_g64_u4", kind="block", B=64, H=14, W=14, C=1024, N=256, G=64, bits=4),
        # ResNet-50's first-stage block, batch 64, 8 bits, groups of 4: the
        # largest maps
        dict(name="block_g4_u8", kind="block", B=64, H=56, W=56, C=256, N=64, G=4, bits=8),
        # last-stage block of the paper's pipeline, batch 64: few rows, long K
        dict(name="block_dfp", kind="block_dfp", B=64, H=7, W=7, C=2048, N=512, G=4, bits=8),
        # the first layer (8-bit weights) of a batch of 64 images
        dict(name="stem_w8", kind="stem", B=64, H=224, W=224, C=4, O=64, R=7, stride=2, pad=3),
        # AlexNet's fc6 at batch 64, the paper's pipeline
        dict(name="fc6_dfp_m64", kind="fc_dfp", M=64, K=9216, O=4096, G=4, bits=8),
        # AlexNet's fc7 for one image, fp32 scales: the weights' bytes
        dict(name="fc7_m1", kind="fc", M=1, K=4096, O=4096, G=4, bits=8),
        # ragged sizes and a channel count that is no multiple of 16
        dict(name="direct_c40", kind="direct", B=8, H=29, W=31, C=40, O=100, R=3, stride=1, G=4, bits=8),
        # converting one 3x3 layer of ResNet's last stage
        dict(name="ternarize_512", kind="ternarize", O=512, C=512, R=3, G=4),
        # one image through ResNet-50
        dict(name="resnet50_b1", kind="net", B=1, hw=224, G=4),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _step(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, step * max(1, round(_logint(rng, lo, hi) / step))))


def draw(rng):
    kind = rng.choice(["gemm", "conv", "conv", "block", "block_dfp", "stem", "fc", "fc_dfp", "direct", "ternarize",
                       "net"])
    G = rng.choice([4, 4, 64])
    bits = rng.choice([8, 8, 4])
    if kind == "gemm":
        return dict(kind=kind, M=_logint(rng, 16, 2048), K=_step(rng, 64, 2048, 64), O=_logint(rng, 48, 1024), G=G,
                    bits=bits)
    if kind in ("conv", "direct"):
        hw = _logint(rng, 7, 57)
        direct = kind == "direct"
        B = _logint(rng, 1, max(2, (20000 if direct else 100000) // (hw * hw)))
        B = min(B, 16 if direct else 64)
        if direct:
            C, G = 4 * _logint(rng, 5, 24), 4
        else:
            C = _step(rng, 64, 512, 64 if G == 64 else 16)
        c = dict(kind=kind, B=B, H=hw, W=hw + rng.randrange(3), C=C, O=_logint(rng, 30, 128 if direct else 512),
                 R=rng.choice([1, 3]), stride=rng.choice([1, 1, 2]), G=G, bits=bits,
                 **({} if direct else {"quant": rng.random() < 0.5}))
        while c["B"] > 1 and work(c)["flops"] > 2e10:
            c["B"] //= 2
        return c
    if kind in ("block", "block_dfp"):
        N = rng.choice([64, 128, 256, 512])
        hw = 56 * 64 // N + rng.randrange(-1, 2)
        return dict(kind=kind, B=_logint(rng, 1, 48), H=hw, W=hw, C=4 * N, N=N, G=G, bits=bits)
    if kind == "stem":
        hw = rng.randrange(160, 230)
        R, stride, pad, O = rng.choice([(7, 2, 3, 64), (11, 4, 0, 96)])
        return dict(kind=kind, B=_logint(rng, 1, 64), H=hw, W=hw, C=4, O=O, R=R, stride=stride, pad=pad)
    if kind in ("fc", "fc_dfp"):
        return dict(kind=kind, M=_logint(rng, 1, 64), K=_step(rng, 1024, 9216, 64), O=4 * _logint(rng, 250, 1024), G=4,
                    bits=bits)
    if kind == "ternarize":
        g = rng.choice([4, 8, 64])
        return dict(kind=kind, O=_logint(rng, 64, 512), C=_step(rng, 64, 512, 64), R=rng.choice([1, 3]), G=g)
    return dict(kind=kind, B=rng.randrange(1, 4), hw=rng.randrange(150, 224), G=4)


# --------------------------------------------------------------------------
# inputs (plain torch, from the seed alone)
# --------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _weights(O, C, R, g):
    z = torch.randn((O, C, R, R), generator=g, device=DEV)
    z = torch.where(z.abs() < 0.05, torch.copysign(torch.full_like(z, 0.05), z), z)
    return z * math.sqrt(2.0 / (C * R * R))


def _ternary(w, G):
    """Codes t in {-1, 0, 1} [O][K] (int8), group scales fp32 [O][K/G] and
    thresholds, k = (r*S + s)*C + c: per group the kept count J maximises
    (sum of the J largest magnitudes)^2 / J."""
    O = w.shape[0]
    v = w.permute(0, 2, 3, 1).reshape(O, -1, G)
    mag, order = v.abs().sort(dim=-1, descending=True, stable=True)
    S = mag.double().cumsum(-1)
    j = torch.arange(1, G + 1, device=DEV, dtype=torch.float64)
    J = (S * S / j).argmax(-1, keepdim=True)
    alpha = (S.gather(-1, J) / (J + 1)).float().squeeze(-1)
    mag0 = F.pad(mag, (0, 1))
    delta = mag0.gather(-1, J + 1).squeeze(-1)
    rank = torch.empty_like(order)
    rank.scatter_(-1, order, torch.arange(G, device=DEV).expand_as(order).contiguous())
    t = torch.where(rank <= J, torch.sign(v), torch.zeros_like(v)).to(torch.int8).reshape(O, -1)
    return t, alpha.contiguous(), delta.contiguous()


def _pack_codes(t):
    c = F.pad((t & 3).to(torch.uint8), (0, -t.shape[1] % 4)).view(t.shape[0], -1, 4)
    return (c[..., 0] | (c[..., 1] << 2) | (c[..., 2] << 4) | (c[..., 3] << 6)).contiguous()


def _qmax(bits):
    return 255.0 if bits == 8 else 15.0


def _codes_of(y, s, bits):
    """Codes of the fp32 values y at the fp32 scale s, one per element: the
    quotient rounded to fp32, then to a whole number, halves to even."""
    return torch.round((y.double() / s.double()).float()).clamp_(0, _qmax(bits)).to(torch.uint8)


def _dynamic_scale(y, bits):
    return (y.max().clamp(min=1e-30).double() / _qmax(bits)).float().reshape(1)


def _pack_acts(q, bits):
    if bits == 8:
        return q.reshape(-1).contiguous()
    f = q.reshape(-1, 2)
    return (f[:, 0] | (f[:, 1] << 4)).contiguous()


def _relu_gauss(shape, g):
    return torch.randn(shape, generator=g, device=DEV).clamp_(min=0)


def _scale(v):
    return torch.full((1,), v, dtype=torch.float32, device=DEV)


def _acts(shape, bits, g):
    """Unpacked codes of a ReLU-Gaussian map and their scale."""
    s = _scale(4.5 / _qmax(bits))
    return _codes_of(_relu_gauss(shape, g), s, bits), s


def _geom(case):
    if case["kind"] in ("gemm", "fc", "fc_dfp"):
        return 1, case["M"], 1, case["K"], case["O"], 1, 1, 0
    R = case["R"]
    return case["B"], case["H"], case["W"], case["C"], case["O"], R, case["stride"], case.get("pad", R // 2)


def _block_layers(case):
    """(C, O, R) of a bottleneck's three convolutions."""
    C, N = case["C"], case["N"]
    return [(C, N, 1), (N, N, 3), (N, C, 1)]


def _net_layers(hw):
    """ResNet-50 after its stem: (name, H, C, O, R, stride)."""
    H = ((hw - 1) // 2 + 1 - 1) // 2 + 1
    cin, out = 64, []
    for stage, (n, width) in enumerate(zip((3, 4, 6, 3), (64, 128, 256, 512))):
        for i in range(n):
            st = 2 if i == 0 and stage > 0 else 1
            p, Ho = "%d.%d" % (stage, i), (H - 1) // st + 1
            out += [(p + ".c1", H, cin, width, 1, 1), (p + ".c2", H, width, width, 3, st),
                    (p + ".c3", Ho, width, 4 * width, 1, 1)]
            if i == 0:
                out.append((p + ".ds", H, cin, 4 * width, 1, st))
            cin, H = 4 * width, Ho
    return out


def _pixels(B, H, W, g):
    x = torch.round(128.0 + 32.0 * torch.randn((B, H, W, 4), generator=g, device=DEV)).clamp_(0, 255)
    x[..., 3] = 0  # three image channels, padded to four
    return x.to(torch.uint8)


def _make(case, seed):
    """Everything a case starts from, in plain torch."""
    g, kind, d = _gen(seed), case["kind"], {}
    if kind == "ternarize":
        d["w"] = _weights(case["O"], case["C"], case["R"], g)
    elif kind == "stem":
        d["w"] = _weights(case["O"], 4, case["R"], g)
        d["w"][:, 3:] = 0
        d["q"], d["sx"] = _pixels(case["B"], case["H"], case["W"], g), _scale(1 / 255.0)
        d["so"] = _scale(0.02)
    elif kind in ("block", "block_dfp"):
        bits, shape = case["bits"], (case["B"], case["H"], case["W"], case["C"])
        d["q"], d["sx"] = _acts(shape, bits, g)
        d["res"] = _relu_gauss(shape, g)
        d["scales"] = [_scale(v / _qmax(bits)) for v in (3.9, 4.1, 6.1)]
        d["layers"] = [_ternary(_weights(O, C, R, g), case["G"]) for C, O, R in _block_layers(case)]
    elif kind == "net":
        d["q"], d["sx"] = _pixels(case["B"], case["hw"], case["hw"], g), _scale(1 / 255.0)
        d["w"] = _weights(64, 4, 7, g)
        d["w"][:, 3:] = 0
        d["layers"] = {n: _ternary(_weights(O, C, R, g), case["G"]) for n, _, C, O, R, _ in _net_layers(case["hw"])}
        d["fc"] = _ternary(_weights(1000, 2048, 1, g), case["G"])
    else:
        B, H, W, C, O, R, _, _ = _geom(case)
        if case.get("quant"):
            d["x"] = _relu_gauss((B, H, W, C), g)
        else:
            d["q"], d["sx"] = _acts((B, H, W, C), case["bits"], g)
        d["layer"] = _ternary(_weights(O, C, R, g), case["G"])
        d["so"] = _scale(4.0 / _qmax(case["bits"]))
    return d


# --------------------------------------------------------------------------
# the path
# --------------------------------------------------------------------------

def _out_hw(H, W, R, stride, pad):
    return (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1


def _empty(shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _bytes(n):
    return _empty((max(int(n), 4),), torch.uint8)


def _fold(layer, O, K, G):
    t, alpha, _ = layer
    codes = _pack_codes(t)
    return dict(codes=codes, alpha=alpha, prep=fgq.fgq_prepare_weights(codes, alpha, O, K, G, fallback=True))


def _dfp(layer, O, K, G):
    t, alpha, _ = layer
    codes = _pack_codes(t)
    return dict(codes=codes, prep=fgq.fgq_prepare_weights_dfp(codes, alpha, O, K, G, 8))


def prepare(case, seed):
    d, kind = _make(case, seed), case["kind"]
    s = dict(case=case)
    if kind == "ternarize":
        s["w"] = d["w"]
    elif kind == "stem":
        Ho, Wo = _out_hw(case["H"], case["W"], case["R"], case["stride"], case["pad"])
        s.update(q=_pack_acts(d["q"], 8), sx=d["sx"], so=d["so"], prep=fgq.fgq_prepare_weights_w8(d["w"]),
                 out=_empty((case["B"], Ho, Wo, case["O"]), torch.uint8))
    elif kind in ("block", "block_dfp"):
        bits, B, H, W, C, N = (case[k] for k in ("bits", "B", "H", "W", "C", "N"))
        make = _fold if kind == "block" else _dfp
        s.update(q=_pack_acts(d["q"], bits), sx=d["sx"], res=d["res"], scales=d["scales"],
                 layers=[make(l, O, R * R * Ci, case["G"]) for l, (Ci, O, R) in zip(d["layers"], _block_layers(case))],
                 q1=_empty((B, H, W, N * bits // 8), torch.uint8), q2=_empty((B, H, W, N * bits // 8), torch.uint8),
                 y=_empty((B, H, W, C)), qo=_empty((B, H, W, C * bits // 8), torch.uint8))
    elif kind == "net":
        _net_prepare(s, d, case, seed)
    else:
        B, H, W, C, O, R, stride, pad = _geom(case)
        K, G, bits = R * R * C, case["G"], case["bits"]
        Ho, Wo = _out_hw(H, W, R, stride, pad)
        if kind == "direct":
            s["layer"] = dict(codes=_pack_codes(d["layer"][0]), alpha=d["layer"][1], prep=None)
        else:
            s["layer"] = (_dfp if kind == "fc_dfp" else _fold)(d["layer"], O, K, G)
        if case.get("quant"):
            n = B * H * W * C
            s.update(x=d["x"], q=_bytes(n * bits // 8), sx=_empty((1,)), ws=_bytes(fgq.fgq_quantize_ws_bytes(n)))
        else:
            s.update(q=_pack_acts(d["q"], bits), sx=d["sx"])
        if kind in ("fc", "fc_dfp"):
            s["ws"] = _bytes(fgq.fgq_gemm_ws_bytes(case["M"], K, O, G, kind == "fc_dfp"))
        if kind == "fc_dfp":
            s.update(so=d["so"], out=_empty((case["M"], O * bits // 8), torch.uint8))
        else:
            s["out"] = _empty((case["M"], O) if kind in ("gemm", "fc") else (B, Ho, Wo, O))
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "ternarize":
        return list(fgq.fgq_ternarize(s["w"], case["G"]))
    if kind == "stem":
        return fgq.fgq_conv2d_w8(s["q"], 8, s["sx"], (case["B"], case["H"], case["W"], 4), s["prep"], case["O"],
                                 case["R"], case["R"], case["stride"], case["pad"], 8, s["so"], out=s["out"])
    if kind == "net":
        s["graph"].replay()
        return [s["feat"], s["logits"]]
    if kind in ("block", "block_dfp"):
        return _run_block(s, case)
    l, bits, G = s["layer"], case["bits"], case["G"]
    if kind == "gemm":
        return fgq.fgq_gemm(s["q"], bits, s["sx"], case["M"], case["K"], l["codes"], l["alpha"], case["O"], G,
                            prepared=l["prep"], y=s["out"])
    if kind == "fc":
        return fgq.fgq_gemm_ws(s["q"], bits, s["sx"], case["M"], case["K"], l["codes"], l["alpha"], case["O"], G,
                               prepared=l["prep"], out=s["out"], ws=s["ws"])
    if kind == "fc_dfp":
        return fgq.fgq_gemm_dfp_ws(s["q"], bits, s["sx"], case["M"], case["K"], l["codes"], l["prep"], case["O"], G,
                                   bits, s["so"], out=s["out"], ws=s["ws"])
    B, H, W, C, O, R, stride, pad = _geom(case)
    if case.get("quant"):
        fgq.fgq_quantize_act(s["x"], bits, q=s["q"], scale_out=s["sx"], ws=s["ws"])
    y = fgq.fgq_conv2d(s["q"], bits, s["sx"], (B, H, W, C), l["codes"], l["alpha"], O, R, R, stride, pad, G,
                       prepared=l["prep"], y=s["out"])
    return [s["sx"], y] if case.get("quant") else y


def _run_block(s, case):
    bits, G, B, H, W, C, N = (case[k] for k in ("bits", "G", "B", "H", "W", "C", "N"))
    a, b, c = s["layers"]
    s1, s2, s3 = s["scales"]
    if case["kind"] == "block":
        fgq.fgq_conv2d_q(s["q"], bits, s["sx"], (B, H, W, C), a["codes"], a["alpha"], N, 1, 1, 1, 0, G, bits, s1,
                         prepared=a["prep"], q_out=s["q1"])
        fgq.fgq_conv2d_q(s["q1"], bits, s1, (B, H, W, N), b["codes"], b["alpha"], N, 3, 3, 1, 1, G, bits, s2,
                         prepared=b["prep"], q_out=s["q2"])
        y, q = fgq.fgq_conv2d_residual_q(s["q2"], bits, s2, (B, H, W, N), c["codes"], c["alpha"], C, 1, 1, 1, 0, G,
                                         s["res"], bits, s3, prepared=c["prep"], y=s["y"], q_out=s["qo"])
    else:
        fgq.fgq_conv2d_dfp(s["q"], bits, s["sx"], (B, H, W, C), a["codes"], a["prep"], N, 1, 1, 1, 0, G, bits, s1,
                           out=s["q1"])
        fgq.fgq_conv2d_dfp(s["q1"], bits, s1, (B, H, W, N), b["codes"], b["prep"], N, 3, 3, 1, 1, G, bits, s2,
                           out=s["q2"])
        y, q = fgq.fgq_conv2d_dfp_residual(s["q2"], bits, s2, (B, H, W, N), c["codes"], c["prep"], C, 1, 1, 1, 0, G,
                                           s["res"], bits, s3, y=s["y"], q_out=s["qo"])
    return [y, q]


def _net_prepare(s, d, case, seed):
    """The network's buffers, its static scales (one pass in plain torch over
    the same images) and the captured forward pass."""
    B, hw, G = case["B"], case["hw"], case["G"]
    scales = _net_plain(d, case)[2]
    L = {n: dict(_dfp(d["layers"][n], O, R * R * C, G), H=H, C=C, O=O, R=R, st=st, sx=scales.get(n))
         for n, H, C, O, R, st in _net_layers(hw)}
    fc = _dfp(d["fc"], 1000, 2048, G)
    q0, sx0, w0 = _pack_acts(d["q"], 8), d["sx"], fgq.fgq_prepare_weights_w8(d["w"])
    H1 = (hw - 1) // 2 + 1
    H2 = (H1 - 1) // 2 + 1
    y0, stem = _empty((B, H1, H1, 64)), _empty((B, H2, H2, 64))
    n = stem.numel()
    qin, qws = _bytes(n), _bytes(fgq.fgq_quantize_ws_bytes(n))
    for l in L.values():
        Ho = (l["H"] - 1) // l["st"] + 1
        l["y"] = _empty((B, Ho, Ho, l["O"]))
        l["q"] = _empty((B, Ho, Ho, l["O"]), torch.uint8)
    pooled, qfc, sfc = _empty((B, 2048)), _bytes(B * 2048), _empty((1,))
    wsq, logits = _bytes(fgq.fgq_quantize_ws_bytes(B * 2048)), _empty((B, 1000))
    wsfc = _bytes(fgq.fgq_gemm_ws_bytes(B, 2048, 1000, G, True))
    scratch = _empty((1,))
    blocks = [n[:-3] for n in L if n.endswith(".c1")]
    buffers = [q0, sx0, w0, L, fc, y0, stem, qin, qws, pooled, qfc, sfc, wsq, wsfc, scratch]

    def conv(l, q, nxt):
        fgq.fgq_conv2d_dfp(q, 8, l["sx"], (B, l["H"], l["H"], l["C"]), l["codes"], l["prep"], l["O"], l["R"], l["R"],
                           l["st"], l["R"] // 2, G, 8, nxt, out=l["q"])
        return l["q"]

    def forward():
        fgq.fgq_conv2d_w8(q0, 8, sx0, (B, hw, hw, 4), w0, 64, 7, 7, 2, 3, out=y0)
        stem.copy_(F.max_pool2d(y0.permute(0, 3, 1, 2), 3, 2, 1).permute(0, 2, 3, 1))
        fgq.fgq_quantize_act(stem, 8, scale_in=L["0.0.c1"]["sx"], q=qin, scale_out=scratch, ws=qws)
        q, h = qin, stem
        for i, p in enumerate(blocks):
            a, b, c, ds = L[p + ".c1"], L[p + ".c2"], L[p + ".c3"], L.get(p + ".ds")
            short = h
            if ds is not None:
                short = fgq.fgq_conv2d_dfp(q, 8, a["sx"], (B, ds["H"], ds["H"], ds["C"]), ds["codes"], ds["prep"],
                                           ds["O"], 1, 1, ds["st"], 0, G, out=ds["y"])
            q = conv(b, conv(a, q, b["sx"]), c["sx"])
            last = i + 1 == len(blocks)
            r = fgq.fgq_conv2d_dfp_residual(q, 8, c["sx"], (B, c["H"], c["H"], c["C"]), c["codes"], c["prep"], c["O"],
                                            1, 1, 1, 0, G, short, 0 if last else 8,
                                            None if last else L[blocks[i + 1] + ".c1"]["sx"], y=c["y"],
                                            q_out=None if last else c["q"])
            h, q = (r, None) if last else r
        torch.mean(h, dim=(1, 2), out=pooled)
        fgq.fgq_quantize_act(pooled, 8, q=qfc, scale_out=sfc, ws=wsq)
        fgq.fgq_gemm_dfp_ws(qfc, 8, sfc, B, 2048, fc["codes"], fc["prep"], 1000, G, out=logits, ws=wsfc)
        return h

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        forward()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        feat = forward()
    s.update(graph=graph, feat=feat, logits=logits, buffers=buffers)


# --------------------------------------------------------------------------
# what it costs, and what it should give
# --------------------------------------------------------------------------

def _weight_bytes(O, K, G, fixed):
    return O * K / 4 + O * (K / G) * (1 if fixed else 4)


def work(case):
    kind = case["kind"]
    if kind == "ternarize":
        n = case["O"] * case["C"] * case["R"] ** 2
        return dict(bytes=4 * n + n / 4 + 8 * n / case["G"], flops=4.0 * n)
    if kind in ("block", "block_dfp"):
        M, bits, C = case["B"] * case["H"] * case["W"], case["bits"], case["C"]
        dims = [(O, R * R * Ci) for Ci, O, R in _block_layers(case)]
        return dict(bytes=M * C * (2 * bits / 8 + 8) + sum(_weight_bytes(O, K, case["G"], kind != "block")
                                                           for O, K in dims),
                    flops=sum(2.0 * M * O * K for O, K in dims))
    if kind == "net":
        B, hw, by, fl = case["B"], case["hw"], 0.0, 0.0
        H1 = (hw - 1) // 2 + 1
        for _, H, C, O, R, st in _net_layers(hw):
            Ho = (H - 1) // st + 1
            fl += 2.0 * B * Ho * Ho * O * R * R * C
            by += _weight_bytes(O, R * R * C, case["G"], True)
        by += B * hw * hw * 4 + 64 * 196 + _weight_bytes(1000, 2048, case["G"], True) + B * 4000
        Hf = _net_layers(hw)[-1][1]
        by += 4.0 * B * Hf * Hf * 2048
        return dict(bytes=by, flops=fl + 2.0 * B * H1 * H1 * 64 * 147 + 2.0 * B * 1000 * 2048)
    B, H, W, C, O, R, stride, pad = _geom(case)
    Ho, Wo = _out_hw(H, W, R, stride, pad)
    M, K = B * Ho * Wo, R * R * C
    n = B * H * W * C
    if kind == "stem":
        return dict(bytes=n + O * K + M * O, flops=2.0 * M * O * R * R * 3)
    bits = case["bits"]
    return dict(bytes=n * (4 if case.get("quant") else bits / 8) + _weight_bytes(O, K, case["G"], kind == "fc_dfp") +
                M * O * (bits / 8 if kind == "fc_dfp" else 4),
                flops=2.0 * M * O * K)


def tolerance(case):
    kind = case["kind"]
    if kind in ("ternarize", "stem", "fc_dfp", "block_dfp"):
        return "exact"  # integers, or fp32 values rounded once from an exact integer sum
    if kind == "net":
        return {"rel": 1e-3}  # fixed-point layers; the mean of the last map is a 32-bit sum ahead of a rounding to codes
    if kind == "block":
        # 32-bit sums: a code next to a rounding boundary may move by one
        return {"rel": 4e-4 if case["bits"] == 8 else 4e-3, "max": 0.1, "differ": 1e-3}
    return {"rel": 1e-6, "max": 1e-5}


def _conv64(q, t_alpha, C, O, R, stride, pad):
    """sum_k alpha t q in 64 bits: q [B][H][W][C] codes, weights [O][R*R*C]."""
    x = F.pad(q.double(), (0, 0, pad, pad, pad, pad))
    B, Hp, Wp, _ = x.shape
    Ho, Wo = (Hp - R) // stride + 1, (Wp - R) // stride + 1
    w = t_alpha.view(O, R, R, C)
    y = torch.zeros((B * Ho * Wo, O), dtype=torch.float64, device=DEV)
    for r in range(R):
        for s in range(R):
            xs = x[:, r:r + (Ho - 1) * stride + 1:stride, s:s + (Wo - 1) * stride + 1:stride]
            y += xs.reshape(-1, C) @ w[:, r, s].t().contiguous()
    return y.view(B, Ho, Wo, O)


def _w64(layer, G):
    t, alpha, _ = layer
    return t.double() * alpha.double().repeat_interleave(G, dim=1)


def _fixed(v, bits=8):
    """v as a `bits`-bit dynamic fixed point with one exponent: (codes, 2^-fl)."""
    top = v.abs().max().double()
    fl = bits - (torch.ceil(torch.log2(top)) + 1)
    lim = 2 ** (bits - 1)
    return torch.round(v.double() * 2 ** fl).clamp_(-lim, lim - 1), 2 ** -fl


def _wdfp(layer, G):
    t, alpha, _ = layer
    A, unit = _fixed(alpha)
    return t.double() * A.repeat_interleave(G, dim=1), unit


def _w8(w):
    W8, unit = _fixed(w)
    return W8.permute(0, 2, 3, 1).reshape(w.shape[0], -1), unit


def _net_plain(d, case):
    """The network in plain torch, every layer's input scale from that input's
    largest value: (last map, logits, scales by layer)."""
    G, scales = case["G"], {}

    def layer(q, sx, n, C, O, R, st):
        w, unit = _wdfp(d["layers"][n], G)
        return (_conv64(q, w, C, O, R, st, R // 2) * (sx.double() * unit)).float()

    def scale_of(y, n):
        scales[n] = _dynamic_scale(y, 8)
        return _codes_of(y, scales[n], 8)

    w, unit = _w8(d["w"])
    y = (_conv64(d["q"], w, 4, 64, 7, 2, 3) * (d["sx"].double() * unit)).float()
    h = F.max_pool2d(y.permute(0, 3, 1, 2), 3, 2, 1).permute(0, 2, 3, 1).contiguous()
    dims = {n: (C, O, R, st) for n, _, C, O, R, st in _net_layers(case["hw"])}
    for p in [n[:-3] for n in dims if n.endswith(".c1")]:
        a, b, c = p + ".c1", p + ".c2", p + ".c3"
        q = scale_of(h, a)
        short = layer(q, scales[a], p + ".ds", *dims[p + ".ds"]) if p + ".ds" in dims else h
        q = scale_of(layer(q, scales[a], a, *dims[a]), b)
        q = scale_of(layer(q, scales[b], b, *dims[b]), c)
        h = (layer(q, scales[c], c, *dims[c]) + short).clamp_(min=0)
    pooled = h.double().mean(dim=(1, 2)).float()
    sfc = _dynamic_scale(pooled, 8)
    w, unit = _wdfp(d["fc"], G)
    logits = (_codes_of(pooled, sfc, 8).double() @ w.t().contiguous()) * (sfc.double() * unit)
    return h.double(), logits, scales


def exact(case, seed):
    d, kind = _make(case, seed), case["kind"]
    if kind == "ternarize":
        _, alpha, delta = _ternary(d["w"], case["G"])
        return [None, alpha.double(), delta.double()]
    if kind == "net":
        h, logits, _ = _net_plain(d, case)
        return [h, logits]
    if kind in ("stem", "fc_dfp"):
        return None  # codes only
    if kind in ("block", "block_dfp"):
        q, sx, G = d["q"], d["sx"], case["G"]
        for i, (l, (C, O, R)) in enumerate(zip(d["layers"], _block_layers(case))):
            w, unit = (_w64(l, G), 1.0) if kind == "block" else _wdfp(l, G)
            y = _conv64(q, w, C, O, R, 1, R // 2) * (sx.double() * unit)
            if i < 2:
                sx = d["scales"][i]
                q = _codes_of(y.float(), sx, case["bits"])
        return [(y + d["res"].double()).clamp_(min=0), None]
    B, H, W, C, O, R, stride, pad = _geom(case)
    if case.get("quant"):
        sx = _dynamic_scale(d["x"], case["bits"])
        q = _codes_of(d["x"], sx, case["bits"])
    else:
        q, sx = d["q"], d["sx"]
    y = _conv64(q, _w64(d["layer"], case["G"]), C, O, R, stride, pad) * sx.double()
    if kind in ("gemm", "fc"):
        return y.view(case["M"], O)
    return [sx.double(), y] if case.get("quant") else y
