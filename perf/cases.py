"""The work that users of this library have it do, as measurable cases.

A case is one of four kinds:

  conv   one binary convolution through one entry point: "mfma"
         (bconv2d_mfma), "quant" (quantize_bconv2d_mfma, float input; where
         the library refuses the shape the program runs bitpack and
         bconv2d_mfma, as the header tells it to) or "xor" (bconv2d, with
         the correction table where zero padding needs it)
  net    a chain of binary convolutions, marshalled once (Prepared* calls):
         the 12-layer QuickNet-like stack, or the four batch-64 layers; with
         "graph" the calls are captured once and a pass replays them
  codec  bitpack and dequantize, the two ends of the binary section
  pool   binary max pooling

Sizes are those of workloads/configs.py (the ResNet18 and QuickNet layers, the
stack, the convolution sweep), or generic ones around them.
"""
import math

import torch

import paper_2011_09398_amd as lce

DEVICE = "cuda"


def listed():
    return [
        # one image, one layer, the plain function: an interactive call or a
        # short script, bound by latency
        dict(name="call_b1", kind="conv", entry="quant", n=1, h=56, w=56, c_in=64, c_out=64,
             kh=3, kw=3, sh=1, sw=1, padding="same", pad_value="one", out="float", clamp=True),
        # single-image inference through the whole binary section, captured
        # in a graph because every layer is shorter than its launch
        dict(name="stack_b1", kind="net", net="stack", n=1, hw=56, width=64, graph=True),
        # the stack at an ordinary serving batch
        dict(name="stack_b16", kind="net", net="stack", n=16, hw=56, width=64, graph=False),
        # the benchmark's step: four layers at batch 64, bits in and out
        dict(name="layers_b64", kind="net", net="layers", n=64, hw=56, width=64, graph=False),
        # offline throughput: the stack over a large batch
        dict(name="stack_b256", kind="net", net="stack", n=256, hw=56, width=64, graph=False),
        # a residual block's convolution: floats in from the shortcut, floats
        # out to it, clamped
        dict(name="residual_b128", kind="conv", entry="quant", n=128, h=28, w=28, c_in=128,
             c_out=128, kh=3, kw=3, sh=1, sw=1, padding="same", pad_value="one", out="float",
             clamp=True),
        # dense prediction: two large images, TensorFlow's zero padding
        dict(name="image_zero", kind="conv", entry="mfma", n=2, h=360, w=640, c_in=64, c_out=64,
             kh=3, kw=3, sh=1, sw=1, padding="same", pad_value="zero", out="float", clamp=False),
        # the widest layer of the convolution sweep, over a batch: long K
        dict(name="sweep_5x5", kind="conv", entry="mfma", n=32, h=64, w=64, c_in=256, c_out=256,
             kh=5, kw=5, sh=1, sw=1, padding="same", pad_value="one", out="float", clamp=False),
        # a pointwise layer: short K, bits out to the next binary layer
        dict(name="pointwise", kind="conv", entry="mfma", n=256, h=28, w=28, c_in=256, c_out=512,
             kh=1, kw=1, sh=1, sw=1, padding="same", pad_value="one", out="bitpacked",
             clamp=False),
        # packed filters used as they are stored (no widened copy), with
        # channel counts and a size that divide by nothing, stride 2
        dict(name="xor_ragged", kind="conv", entry="xor", n=64, h=45, w=61, c_in=200, c_out=136,
             kh=3, kw=3, sh=2, sw=2, padding="same", pad_value="zero", out="float", clamp=False),
        # quantize and dequantize activations whose channels fill no word
        dict(name="codec_ragged", kind="codec", n=64, h=56, w=56, c=72),
        # pooling between binary sections, on packed words
        dict(name="pool", kind="pool", n=512, h=56, w=56, c=256, k=3, s=2, padding="same"),
    ]


# ---- drawn cases

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Half of the layers have whole words of channels, as networks do."""
    c = _log(rng, lo, hi)
    return max(32, (c + 16) // 32 * 32) if rng.random() < 0.5 else c


# What one drawn case may cost: no more than the largest listed one.
MOST_FLOPS = 4.0e11
MOST_BYTES = 4.0e8


def _fits(case):
    w = work(case)
    return w["bytes"] <= MOST_BYTES and w["flops"] <= MOST_FLOPS


def draw(rng):
    kind = rng.choice(("quant", "mfma", "mfma", "pointwise", "xor", "net", "codec", "pool"))
    if kind == "net":
        n = _log(rng, 1, 256)
        case = dict(kind="net", net=rng.choice(("stack", "stack", "layers")), n=n,
                    hw=rng.randint(24, 64), width=64, graph=n <= 4)
        while not _fits(case):
            case["n"] = max(1, case["n"] // 2)
        return case
    if kind == "codec":
        case = dict(kind="codec", n=_log(rng, 1, 128), h=_log(rng, 7, 112), w=_log(rng, 7, 112),
                    c=_channels(rng, 8, 512))
    elif kind == "pool":
        k = rng.choice((2, 3))
        case = dict(kind="pool", n=_log(rng, 1, 1024), h=_log(rng, 7, 112), w=_log(rng, 7, 112),
                    c=_channels(rng, 16, 512), k=k, s=rng.choice((2, 2, k)),
                    padding=rng.choice(("same", "valid")))
    else:
        k = 1 if kind == "pointwise" else rng.choice((3, 3, 3, 5))
        s = 1 if kind == "pointwise" else rng.choice((1, 1, 2))
        case = dict(kind="conv", entry="mfma" if kind == "pointwise" else kind,
                    n=_log(rng, 1, 512), h=_log(rng, 7, 128), w=_log(rng, 7, 128),
                    c_in=_channels(rng, 32, 512), c_out=_channels(rng, 24, 512), kh=k, kw=k,
                    sh=s, sw=s, padding=rng.choice(("same", "same", "same", "valid")),
                    pad_value=rng.choice(("one", "one", "zero")),
                    out=rng.choice(("float", "bitpacked", "bitpacked", "int32")),
                    clamp=rng.random() < 0.3)
        if kind == "quant":
            case["c_in"] = max(32, case["c_in"] // 32 * 32)
            case["pad_value"] = "one"
    while not _fits(case):
        if case["n"] > 1:
            case["n"] = max(1, case["n"] // 2)
        else:
            case["h"] = max(7, case["h"] // 2)
    return case


# ---- layers

def _words(c):
    return (c + 31) // 32


def _out_hw(c):
    if c["padding"] == "same":
        return -(-c["h"] // c["sh"]), -(-c["w"] // c["sw"])
    return (c["h"] - c["kh"]) // c["sh"] + 1, (c["w"] - c["kw"]) // c["sw"] + 1


def _layers(case):
    """The convolutions of a case, in order; "src" is the index of the layer
    that feeds one (None: an input of its own)."""
    if case["kind"] == "conv":
        return [dict(case, src=None)]
    n, hw, c = case["n"], case["hw"], case["width"]

    def conv(h, ci, co, s=1, out="bitpacked", src=None, entry="mfma"):
        return dict(entry=entry, n=n, h=h, w=h, c_in=ci, c_out=co, kh=3, kw=3, sh=s, sw=s,
                    padding="same", pad_value="one", out=out, clamp=False, src=src)

    half = lambda v: -(-v // 2)  # noqa: E731
    h2, h4, h8 = half(hw), half(half(hw)), half(half(half(hw)))
    if case["net"] == "layers":
        return [conv(hw, c, 2 * c, 2), conv(h2, 2 * c, 2 * c, src=0), conv(h4, 4 * c, 4 * c),
                conv(h8, 8 * c, 8 * c)]
    made = [conv(hw, c, c, entry="quant")] + [conv(hw, c, c, src=i) for i in range(3)]
    made.append(conv(hw, c, 2 * c, 2, src=3))
    made += [conv(h2, 2 * c, 2 * c, src=i) for i in range(4, 7)]
    made.append(conv(h2, 2 * c, 4 * c, 2, src=7))
    made += [conv(h4, 4 * c, 4 * c, src=i) for i in range(8, 11)]
    made[-1]["out"] = "float"
    return made


def _layer_work(c):
    oh, ow = _out_hw(c)
    m = c["n"] * oh * ow
    in_bytes = c["n"] * c["h"] * c["w"] * (4 * c["c_in"] if c["entry"] == "quant"
                                           else 4 * _words(c["c_in"]))
    w_bytes = 4 * c["c_out"] * c["kh"] * c["kw"] * _words(c["c_in"])
    out_bytes = 4 * m * (_words(c["c_out"]) if c["out"] == "bitpacked" else c["c_out"])
    return in_bytes + w_bytes + out_bytes, 2 * m * c["c_out"] * c["kh"] * c["kw"] * c["c_in"]


def work(case):
    """Bytes: every call's input, filters and output once.  Operations: one
    multiply and one add per +-1 product."""
    if case["kind"] == "codec":
        pixels = case["n"] * case["h"] * case["w"]
        return {"bytes": pixels * (8 * case["c"] + 8 * _words(case["c"])), "flops": 0}
    if case["kind"] == "pool":
        oh, ow = _pool_hw(case)
        return {"bytes": 4 * _words(case["c"]) * case["n"] * (case["h"] * case["w"] + oh * ow),
                "flops": 0}
    each = [_layer_work(c) for c in _layers(case)]
    return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}


def _pool_hw(c):
    if c["padding"] == "same":
        return -(-c["h"] // c["s"]), -(-c["w"] // c["s"])
    return (c["h"] - c["k"]) // c["s"] + 1, (c["w"] - c["k"]) // c["s"] + 1


# ---- inputs

def _activations(gen, *shape):
    return torch.randn(*shape, device=DEVICE, generator=gen)


def _make(case, seed):
    """Float activations (normal, as after a batch normalization), filter
    signs, and per layer the folded batch normalization: a multiplier about
    1/sqrt(K), one in eight negative, and a bias."""
    gen = torch.Generator(DEVICE).manual_seed(seed)
    made = []
    for c in _layers(case):
        x = None if c["src"] is not None else _activations(gen, c["n"], c["h"], c["w"], c["c_in"])
        w = torch.randint(0, 2, (c["c_out"], c["kh"], c["kw"], c["c_in"]), device=DEVICE,
                          generator=gen).float() * 2 - 1
        k = c["kh"] * c["kw"] * c["c_in"]
        m = (1 + 0.1 * torch.randn(c["c_out"], device=DEVICE, generator=gen)) / math.sqrt(k)
        m = torch.where(torch.rand(c["c_out"], device=DEVICE, generator=gen) < 0.125, -m, m)
        b = 0.3 * torch.randn(c["c_out"], device=DEVICE, generator=gen)
        made.append((c, x, w, m, b))
    return made


def _clamp(c):
    """A ReLU-like activation on the accumulator, or none."""
    k = c["kh"] * c["kw"] * c["c_in"]
    return (0, k) if c["clamp"] else None


def _conv_kw(c, m, b):
    kw = dict(stride=(c["sh"], c["sw"]), padding=c["padding"], clamp=_clamp(c), out_type=c["out"])
    if c["out"] == "float":
        kw.update(multiplier=m, bias=b)
    elif c["out"] == "bitpacked":
        thr, flip = lce.fold_thresholds(m.cpu().numpy(), b.cpu().numpy(), c["c_out"],
                                        c["kh"] * c["kw"] * c["c_in"], _clamp(c))
        kw.update(thresholds=torch.from_numpy(thr).to(DEVICE),
                  flip=torch.from_numpy(flip).to(DEVICE))
    return kw


def _conv_out(c):
    oh, ow = _out_hw(c)
    oc = _words(c["c_out"]) if c["out"] == "bitpacked" else c["c_out"]
    return torch.empty((c["n"], oh, ow, oc), device=DEVICE,
                       dtype=torch.float32 if c["out"] == "float" else torch.int32)


def _prepare_conv(case, seed):
    (c, x, w, m, b), = _make(case, seed)
    kw = _conv_kw(c, m, b)
    kernel = (c["kh"], c["kw"])
    wp = lce.bitpack(w)
    if c["entry"] == "xor":
        table = lce.pad_correction(wp, c["c_in"]) if c["pad_value"] == "zero" else None
        kw.update(pad_value=c["pad_value"], pad_correction=table)
        xp = lce.bitpack(x)
        return lambda: lce.bconv2d(xp, wp, c["c_in"], **kw)
    wf = lce.mfma_weights(wp, c["c_in"])
    kw.update(pad_value=c["pad_value"])
    if c["entry"] == "mfma":
        xp = lce.bitpack(x)
        return lambda: lce.bconv2d_mfma(xp, wf, c["c_in"], c["c_out"], kernel, **kw)
    try:
        lce.quantize_bconv2d_mfma(x, wf, c["c_out"], kernel, **kw)
    except lce.LceError as e:
        if e.status != lce.LCE_EUNSUPPORTED:
            raise
        return lambda: lce.bconv2d_mfma(lce.bitpack(x), wf, c["c_in"], c["c_out"], kernel, **kw)
    return lambda: lce.quantize_bconv2d_mfma(x, wf, c["c_out"], kernel, **kw)


def _prepare_net(case, seed):
    calls, outs = [], []
    for c, x, w, m, b in _make(case, seed):
        kw = _conv_kw(c, m, b)
        wf = lce.mfma_weights(lce.bitpack(w), c["c_in"])
        out = _conv_out(c)
        if c["entry"] == "quant":
            try:
                calls.append(lce.PreparedQuantBConv2dMfma(x, wf, c["c_out"], (3, 3), out, **kw))
                outs.append(out)
                continue
            except lce.LceError as e:
                if e.status != lce.LCE_EUNSUPPORTED:
                    raise
        if c["src"] is not None:
            xp = outs[c["src"]]
        else:
            xp = lce.bitpack(x)
            if c["entry"] == "quant":
                calls.append(lce.PreparedBitpack(x, xp))
        calls.append(lce.PreparedBConv2dMfma(xp, wf, c["c_in"], c["c_out"], (3, 3), out, **kw))
        outs.append(out)

    def through():
        for call in calls:
            call()
        return outs

    if not case["graph"]:
        return through
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        through()

    def replay():
        graph.replay()
        return outs

    return replay


def prepare(case, seed):
    if case["kind"] == "conv":
        return _prepare_conv(case, seed)
    if case["kind"] == "net":
        return _prepare_net(case, seed)
    gen = torch.Generator(DEVICE).manual_seed(seed)
    x = _activations(gen, case["n"], case["h"], case["w"], case["c"])
    if case["kind"] == "codec":
        return lambda: _codec(x, case["c"])
    xp = lce.bitpack(x)
    return lambda: lce.bmaxpool2d(xp, case["c"], case["k"], case["s"], case["padding"])


def _codec(x, c):
    packed = lce.bitpack(x)
    return [packed, lce.dequantize(packed, c)]


def run(state):
    return state()


def tolerance(case):
    """Bits and accumulators are whole numbers.  A float output is an exact
    integer through one fused multiply-add: half a unit in the last place
    (3e-8 on average; 6e-8 at most, of the value)."""
    if case["kind"] == "conv" and case["out"] == "float" or \
            case["kind"] == "net" and case["net"] == "stack":
        return {"rel": 1.2e-7, "max": 1e-6}
    return "exact"


# ---- the same in 64 bits, in plain torch

def _pack64(neg):
    """bool [..., C] -> int32 words, bit c%32 of word c/32."""
    c = neg.shape[-1]
    bits = torch.zeros(neg.shape[:-1] + (_words(c) * 32,), dtype=torch.int64, device=neg.device)
    bits[..., :c] = neg
    bits = bits.view(neg.shape[:-1] + (_words(c), 32))
    words = (bits << torch.arange(32, device=neg.device)).sum(-1)
    return torch.where(words >= 2 ** 31, words - 2 ** 32, words).to(torch.int32)


def _conv64(c, sign, w):
    """The +-1 cross-correlation, tap by tap, as float64 matrix products."""
    oh, ow = _out_hw(c)
    if c["padding"] == "same":
        ph = max(0, (oh - 1) * c["sh"] + c["kh"] - c["h"])
        pw = max(0, (ow - 1) * c["sw"] + c["kw"] - c["w"])
        sign = torch.nn.functional.pad(
            sign, (0, 0, pw // 2, pw - pw // 2, ph // 2, ph - ph // 2),
            value=1.0 if c["pad_value"] == "one" else 0.0)
    acc = torch.zeros(c["n"] * oh * ow, c["c_out"], dtype=torch.float64, device=sign.device)
    for ky in range(c["kh"]):
        for kx in range(c["kw"]):
            tap = sign[:, ky:ky + (oh - 1) * c["sh"] + 1:c["sh"],
                       kx:kx + (ow - 1) * c["sw"] + 1:c["sw"]].reshape(-1, c["c_in"])
            acc += tap @ w[:, ky, kx].double().t().contiguous()
    acc = acc.view(c["n"], oh, ow, c["c_out"])
    return acc if _clamp(c) is None else acc.clamp(*map(float, _clamp(c)))


def exact(case, seed):
    if case["kind"] in ("codec", "pool"):
        gen = torch.Generator(DEVICE).manual_seed(seed)
        neg = _activations(gen, case["n"], case["h"], case["w"], case["c"]) < 0
        if case["kind"] == "codec":
            return [_pack64(neg), 1.0 - 2.0 * neg.double()]
        k, s = case["k"], case["s"]
        oh, ow = _pool_hw(case)
        if case["padding"] == "same":
            ph = max(0, (oh - 1) * s + k - case["h"])
            pw = max(0, (ow - 1) * s + k - case["w"])
            neg = torch.nn.functional.pad(
                neg, (0, 0, pw // 2, pw - pw // 2, ph // 2, ph - ph // 2), value=True)
        got = torch.ones(case["n"], oh, ow, case["c"], dtype=torch.bool, device=neg.device)
        for y in range(k):
            for x in range(k):
                got &= neg[:, y:y + (oh - 1) * s + 1:s, x:x + (ow - 1) * s + 1:s]
        return _pack64(got)
    outs, signs = [], []
    for c, x, w, m, b in _make(case, seed):
        sign = signs[c["src"]] if x is None else torch.where(x < 0, -1.0, 1.0).double()
        acc = _conv64(c, sign, w)
        y = acc * m.double() + b.double()
        signs.append(torch.where(y < 0, -1.0, 1.0).double() if c["out"] == "bitpacked" else None)
        outs.append(y if c["out"] == "float" else _pack64(y < 0) if c["out"] == "bitpacked"
                    else acc.to(torch.int32))
    return outs if case["kind"] == "net" else outs[0]
