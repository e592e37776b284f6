"""The work a user of this library has it do, as cases to measure.

A case is a dict of plain values; its "kind" is one of the library's entry
points (paper_1908_11263_amd):

  conv       conv2d: one quantized convolution layer
  conv_pool  conv2d_maxpool: the layer fused with its 2x2 max-pooling
  linear     linear: a fully connected layer over whole images
  net        network.cifar_forward: the CIFAR-10-shaped network
  relu_pool  relu_s8, then maxpool2d on its output (unfused helpers)

Sizes: the single-layer workloads and networks of bench.py (16x16x32 INT-8,
32x32x64 INT-4, 16x16x128 INT-2, 8x8x256 INT-1, the networks) and generic
layers around them: other strides, filter sizes, channel counts that fill no
tile, odd image sizes, other epilogues.

Inputs are uniform codes (packed uniform bytes are uniform codes at every
bit-width), as the workloads define them.  Layer parameters place the
accumulator's distribution over the whole output range, so that every output
code occurs; the networks take the workloads' own parameters.
"""
import math

import torch

import paper_1908_11263_amd as qnn
from paper_1908_11263_amd import network


def _conv(name, bits, n, h, w, c, m, k, stride, pad, epi, kind="conv"):
    return dict(name=name, kind=kind, bits=bits, n=n, h=h, w=w, c=c, m=m, k=k, stride=stride,
                pad=pad, epi=epi)


def listed():
    return [
        # one image through one small layer: a device that answers one request
        # at a time, where latency and the launch are what counts
        _conv("layer8_b1", 8, 1, 16, 16, 32, 32, 3, 1, 1, "requant"),
        # the benchmark layers at their batches, one per bit-width
        _conv("layer4_b64", 4, 64, 32, 32, 64, 64, 3, 1, 1, "requant"),
        _conv("layer2_b256", 2, 256, 16, 16, 128, 128, 3, 1, 1, "requant"),
        _conv("layer1_b1024", 1, 1024, 8, 8, 256, 256, 3, 1, 1, "thresh1"),
        # a late, wide layer of a larger network: most of its arithmetic
        _conv("wide8_b256", 8, 256, 14, 14, 256, 256, 3, 1, 1, "requant"),
        # a strided layer that halves the image, with the paper's staircase
        _conv("down4_b256", 4, 256, 56, 56, 64, 128, 3, 2, 1, "stair"),
        # a pointwise (1x1) layer: as much memory traffic as arithmetic
        _conv("point8_b256", 8, 256, 28, 28, 128, 256, 1, 1, 0, "requant"),
        # sizes that fill no tile: odd image, channels that are no power of two
        _conv("odd4_pool_b129", 4, 129, 45, 37, 48, 72, 3, 1, 1, "requant", kind="conv_pool"),
        # a fully connected layer with many outputs and raw logits
        dict(name="linear8_n1000", kind="linear", bits=8, n=1000, h=8, w=8, c=64, m=1000, epi="raw32"),
        # the end-to-end networks: a large batch, and one that is no round number
        dict(name="net8_b4096", kind="net", bits=8, n=4096),
        dict(name="net4_b1000", kind="net", bits=4, n=1000),
        # activations whose ReLU and pooling are not fused into a convolution
        dict(name="relu_pool8", kind="relu_pool", bits=8, n=128, h=112, w=112, c=64, k=3, stride=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _epi_of(rng, bits, pool=False):
    if bits == 1:
        return rng.choice(["thresh1", "thresh1", "raw32"])
    kinds = ["requant", "requant", "requant"] + ([] if pool else ["raw32"])
    return rng.choice(kinds + (["stair"] if bits != 8 else []))


def draw(rng):
    kind = rng.choice(["conv"] * 6 + ["conv_pool"] * 2 + ["linear"] * 2 + ["net", "relu_pool"])
    if kind == "net":
        return dict(kind=kind, bits=rng.choice([8, 4]), n=_log_int(rng, 1, 4096))
    if kind == "linear":
        bits = rng.choice([8, 8, 4, 2, 1])
        epi = rng.choice(["raw32", "thresh1" if bits == 1 else "requant"])
        side = rng.choice([1, 2, 4, 7, 8])
        unit = 32 // bits
        most = 4096 if epi == "raw32" else 1024
        c = unit * max(1, _log_int(rng, 64, most) // (side * side * unit))
        if side * side * c > most:
            side = 1
        if side * side * c > 1024 and side * side * c % 64:
            # longer reductions are refused unless they are whole 64s
            c = c // 64 * 64 or 1024 // (side * side) // unit * unit or unit
        return dict(kind=kind, bits=bits, n=_log_int(rng, 1, 4096), h=side, w=side, c=c,
                    m=_log_int(rng, 10, 1024), epi=epi)
    if kind == "relu_pool":
        h, w, c = _log_int(rng, 8, 128), _log_int(rng, 8, 128), 4 * _log_int(rng, 1, 64)
        k = rng.choice([2, 3])
        n = max(1, _log_int(rng, 1 << 14, 64 << 20) // (h * w * c))
        return dict(kind=kind, bits=8, n=n, h=h, w=w, c=c, k=k, stride=2)
    bits = rng.choice([8, 4, 2, 1]) if kind == "conv" else rng.choice([8, 4, 2])
    k = rng.choice([1, 3, 3, 3, 5])
    stride = rng.choice([1, 1, 2])
    unit = 32 // bits
    # pooled layers are the early, narrower ones
    most = 64 if k == 5 else 128 if kind == "conv_pool" else 256
    c = unit * max(1, _log_int(rng, 16, most) // unit)
    m = _log_int(rng, 8, 256)
    if rng.random() < 0.5:
        m = max(32, m // 32 * 32)
    h, w = _log_int(rng, 7, 64), _log_int(rng, 7, 64)
    per = (h // stride) * (w // stride) * m * k * k * c
    # the image count gives 2 M to 30 G multiply-adds, within 128 MB of traffic
    n = max(1, int(_log_int(rng, 2_000_000, 30_000_000_000) / per))
    epi = _epi_of(rng, bits, kind == "conv_pool")
    out = (h // stride) * (w // stride) * m * (32 if epi == "raw32" else bits) // 8
    n = max(1, min(n, (128 << 20) // (h * w * c * bits // 8 + out)))
    return dict(kind=kind, bits=bits, n=n, h=h, w=w, c=c, m=m, k=k, stride=stride, pad=k // 2, epi=epi)


# --- shapes -----------------------------------------------------------------

def _pix(c, bits):
    return 4 * c if bits == 32 else (c * bits + 7) // 8


def _out_hw(c):
    return ((c["h"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1,
            (c["w"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1)


def _out_bits(c):
    return {"requant": c["bits"], "stair": c["bits"], "thresh1": 1, "raw32": 32}[c["epi"]]


# channels (in, out) and image side of the network's three 5x5 layers
_NET = ((3, 32, 32), (32, 32, 16), (32, 64, 8))


def work(case):
    """Dense multiply-adds (two operations each; padding taps counted, padding
    channels not) and the bytes of one pass: inputs, weights, parameters and
    outputs once each."""
    kind, bits, n = case["kind"], case["bits"], case["n"]
    if kind == "net":
        macs = sum(n * s * s * m * 25 * c for c, m, s in _NET) + n * 10240
        # the image's 4th channel is alignment only, but it is in the input
        byts = n * 32 * 32 * _pix(4, bits) + n * 40
        byts += sum(m * 25 * max(4, c) * bits // 8 + 9 * m for c, m, s in _NET) + 10240 * bits // 8 + 40
        return {"bytes": byts, "flops": 2 * macs}
    if kind == "relu_pool":
        ho, wo = (case["h"] - case["k"]) // case["stride"] + 1, (case["w"] - case["k"]) // case["stride"] + 1
        # both results are returned: the input read, the ReLU written, the pooled pixels written
        byts = n * case["c"] * (2 * case["h"] * case["w"] + ho * wo)
        return {"bytes": byts, "flops": n * case["c"] * (case["h"] * case["w"] + ho * wo * case["k"] ** 2)}
    m = case["m"]
    params = m * (4 * ((1 << bits) - 1) if case["epi"] == "stair" else 9) + 4 * m
    xin = n * case["h"] * case["w"] * _pix(case["c"], bits)
    if kind == "linear":
        K = case["h"] * case["w"] * case["c"]
        return {"bytes": xin + m * K * bits // 8 + params + n * _pix(m, _out_bits(case)), "flops": 2 * n * m * K}
    ho, wo = _out_hw(case)
    K = case["k"] ** 2 * case["c"]
    px = n * (ho // 2) * (wo // 2) if kind == "conv_pool" else n * ho * wo
    return {"bytes": xin + m * K * bits // 8 + params + px * _pix(m, _out_bits(case)),
            "flops": 2 * n * ho * wo * m * K}


def tolerance(case):
    """Every output is a whole number that the layer defines uniquely."""
    return "exact"


# --- inputs -----------------------------------------------------------------

def _bytes(g, *shape):
    return torch.randint(0, 256, shape, generator=g, device="cuda", dtype=torch.uint8)


def _ints(g, lo, hi, *shape):
    return torch.randint(lo, hi + 1, shape, generator=g, device="cuda", dtype=torch.int32)


def _codes(packed, bits):
    """Unsigned codes of the last axis, lowest channel in the lowest bits."""
    sh = torch.arange(0, 8, bits, device=packed.device)
    v = (packed.long().unsqueeze(-1) >> sh) & ((1 << bits) - 1)
    return v.reshape(*packed.shape[:-1], -1)


def _act_values(packed, bits):
    v = _codes(packed, bits)
    return 2 * v - 1 if bits == 1 else v


def _weight_values(packed, bits):
    v = _codes(packed, bits)
    if bits == 1:
        return 2 * v - 1
    return v - ((v >> (bits - 1)) << bits)


def _params(g, case, w, K):
    """Epilogue parameters: the accumulator of uniform inputs has the mean
    E[x] sum(w) and about the deviation sqrt(K) dev(x) rms(w) per channel; the
    output range covers 1.5 deviations on each side of the mean."""
    bits, m, epi = case["bits"], case["m"], case["epi"]
    if bits == 1:
        p = dict(bias=None, mult=None, shift=None, thresh=None, clip=(0, 0))
        if epi == "thresh1":
            s = max(1, int(1.5 * math.sqrt(K)))
            p["thresh"] = _ints(g, -s, s, m)
        return p
    hi = (1 << bits) - 1
    wsum = _weight_values(w, bits).sum(-1)
    centre = wsum * hi // 2
    dev = math.sqrt(K) * math.sqrt((hi * (hi + 2)) / 12.0) * (1 << bits) / math.sqrt(12.0)
    p = dict(bias=None, mult=None, shift=None, thresh=None, clip=(0, hi))
    if epi == "raw32":
        p["bias"] = _ints(g, -16 * hi, 16 * hi, m)
    elif epi == "requant":
        # hi codes over 3 deviations: (acc - centre + 1.5 dev) * hi / (3 dev)
        p["mult"] = _ints(g, 1 << 14, 1 << 15, m)
        p["shift"] = torch.full((m,), max(0, round(math.log2(24576 * 3 * dev / hi))), dtype=torch.int8,
                                device="cuda")
        p["bias"] = (_ints(g, int(dev), int(2 * dev) + 1, m).long() - centre).int()
    else:
        # thresholds compare with acc + bias; the bias is centred the same way
        p["bias"] = (-centre).int()
        r = max(2, int(2 * dev))
        p["thresh"] = _ints(g, -r, r, m, hi).sort(dim=1).values.contiguous()
    return p


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 7919 + 17)
    kind, bits, n = case["kind"], case["bits"], case["n"]
    if kind == "net":
        hi = (1 << bits) - 1
        x = _bytes(g, n, 32, 32, _pix(4, bits))
        # three image channels and a zero channel that fills the pixel
        keep = torch.tensor([255, 255, 255, 0] if bits == 8 else [255, 15], dtype=torch.uint8, device="cuda")
        x &= keep
        convs, cin = [], 4
        for c, m, _ in _NET:
            w = _bytes(g, m, 25, _pix(cin, bits))
            if c == 3:
                w &= keep
            convs.append(dict(w=w.reshape(m, -1).contiguous(), m=m, k=5, pad=2,
                              bias=_ints(g, -16 * hi - 16, 16 * hi + 16, m), mult=_ints(g, 1 << 14, 1 << 15, m),
                              shift=torch.full((m,), 25 if bits == 8 else 21, dtype=torch.int8, device="cuda")))
            cin = m
        fc = dict(w=_bytes(g, 10, 1024 * bits // 8), bias=_ints(g, -16 * hi, 16 * hi, 10), m=10)
        return dict(case=case, x=x, convs=convs, fc=fc, clip=(0, hi))
    x = _bytes(g, n, case["h"], case["w"], _pix(case["c"], bits))
    if kind == "relu_pool":
        return dict(case=case, x=x)
    K = case["h"] * case["w"] * case["c"] if kind == "linear" else case["k"] ** 2 * case["c"]
    w = _bytes(g, case["m"], K * bits // 8)
    return dict(case=case, x=x, w=w, p=_params(g, case, w, K))


def run(state):
    c = state["case"]
    kind, bits, n = c["kind"], c["bits"], c["n"]
    if kind == "net":
        # the logits and every layer's activations
        return network.cifar_forward(state["x"], n, bits, 4, state["convs"], state["fc"], state["clip"], keep=True)
    shape = (n, c["h"], c["w"], c["c"])
    if kind == "relu_pool":
        y = qnn.relu_s8(state["x"])
        return y, qnn.maxpool2d(y, shape, bits, c["k"], c["k"], c["stride"], c["stride"])
    p = state["p"]
    if kind == "linear":
        return qnn.linear(state["x"], shape, bits, state["w"], c["m"], c["epi"], bias=p["bias"],
                          mult=p["mult"], shift=p["shift"], thresh=p["thresh"], clip=p["clip"])
    fn = qnn.conv2d_maxpool if kind == "conv_pool" else qnn.conv2d
    return fn(state["x"], shape, bits, state["w"], c["m"], c["k"], c["k"], (c["stride"], c["stride"]),
              (c["pad"], c["pad"]), c["epi"], bias=p["bias"], mult=p["mult"], shift=p["shift"],
              thresh=p["thresh"], clip=p["clip"])


# --- the same in plain torch, 64 bits ---------------------------------------

def _pack(codes, bits):
    per = 8 // bits
    c = codes.shape[-1]
    codes = torch.nn.functional.pad(codes, (0, -c % per)).reshape(*codes.shape[:-1], -1, per)
    sh = torch.arange(0, 8, bits, device=codes.device)
    return (codes << sh).sum(-1).to(torch.uint8)


def _level(acc, p, epi, bits):
    """Epilogue of int64 sums acc [..., m]: codes, or int32 sums."""
    t = acc if p["bias"] is None else acc + p["bias"].long()
    if epi == "raw32":
        return t.int()
    if epi == "thresh1":
        return _pack((t >= p["thresh"].long()).long(), 1)
    if epi == "stair":
        y = torch.zeros_like(t)
        for i in range((1 << bits) - 1):
            y += t >= p["thresh"][:, i].long()
        return _pack(y, bits)
    s = p["shift"].long()
    t = t * p["mult"].long()
    t = (t + torch.where(s > 0, 1 << (s - 1).clamp(min=0), 0)) >> s
    return _pack(t.clamp(p["clip"][0], p["clip"][1]), bits)


def _exact_conv(x, bits, w, m, k, stride, pad, p, epi, pool):
    """x packed [n, h, w, bytes] -> the layer's output, a group of images at a time."""
    c = w.shape[1] * 8 // bits // (k * k)
    wv = _weight_values(w, bits).reshape(m, k, k, c).double()
    ho = (x.shape[1] + 2 * pad - k) // stride + 1
    wo = (x.shape[2] + 2 * pad - k) // stride + 1
    step = max(1, (1 << 26) // (ho * wo * m + (x.shape[1] + 2 * pad) * (x.shape[2] + 2 * pad) * c))
    out = []
    for b in range(0, x.shape[0], step):
        v = _act_values(x[b:b + step], bits)[..., :c].double()
        v = torch.nn.functional.pad(v, (0, 0, pad, pad, pad, pad), value=-1.0 if bits == 1 else 0.0)
        acc = torch.zeros(v.shape[0] * ho * wo, m, dtype=torch.float64, device=x.device)
        for ky in range(k):
            for kx in range(k):
                t = v[:, ky:ky + (ho - 1) * stride + 1:stride, kx:kx + (wo - 1) * stride + 1:stride]
                acc += t.reshape(-1, c) @ wv[:, ky, kx].t().contiguous()
        y = _level(acc.long().reshape(-1, ho, wo, m), p, epi, bits)
        if pool:
            y = _codes(y, bits)[:, :ho // 2 * 2, :wo // 2 * 2]
            y = y.reshape(y.shape[0], ho // 2, 2, wo // 2, 2, -1).amax((2, 4))[..., :m]
            y = _pack(y, bits)
        out.append(y)
    return torch.cat(out)


def exact(case, seed):
    s = prepare(case, seed)
    kind, bits, n = case["kind"], case["bits"], case["n"]
    if kind == "net":
        x, acts = s["x"], []
        for cv in s["convs"]:
            p = dict(bias=cv["bias"], mult=cv["mult"], shift=cv["shift"], clip=s["clip"])
            x = _exact_conv(x, bits, cv["w"], cv["m"], 5, 1, 2, p, "requant", True)
            acts.append(x)
        acc = _act_values(x.reshape(n, -1), bits).double() @ _weight_values(s["fc"]["w"], bits).double().t().contiguous()
        return (acc.long() + s["fc"]["bias"].long()).int().reshape(n, 1, 1, 10), acts
    if kind == "relu_pool":
        v = s["x"].long()
        v = torch.where(v >= 128, 0, v)
        k, st = case["k"], case["stride"]
        pooled = v.unfold(1, k, st).unfold(2, k, st).amax((-1, -2))
        return v.to(torch.uint8), pooled.to(torch.uint8)
    if kind == "linear":
        acc = (_act_values(s["x"].reshape(n, -1), bits).double()
               @ _weight_values(s["w"], bits).double().t().contiguous())
        return _level(acc.long().reshape(n, 1, 1, case["m"]), s["p"], case["epi"], bits)
    return _exact_conv(s["x"], bits, s["w"], case["m"], case["k"], case["stride"], case["pad"], s["p"],
                       case["epi"], kind == "conv_pool")
