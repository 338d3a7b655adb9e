"""The work whose speed is measured: what a program that uses this library has it do.

``listed()`` are the fixed cases, ``draw(rng)`` gives more of the same ranges.  A case is a plain dict; ``kind`` says which
entry points it goes through:

  fc          bmm_thr / bmm: one binarized fully-connected layer or bit matrix product (packed bits in, bits or int32 out)
  fc_general  bmm_general_f32: real-valued operands in, real-valued sums out
  conv        bconv_thr: one binarized convolution + threshold, optionally with the int32 residual in and the sum out; bconv
  thrd_pool   threshold_pack, then maxpool_or: threshold and pooling of a layer whose int32 sums are in memory
  first       bwn_conv_thr / conv_f32_split_thr: the first layer of a network (real-valued image in, bits out)
  net         Net.forward: a whole network (the shapes of the paper's Table 5 and the MLP)

Everything binarized is exact.  So are the networks here: their images are 8-bit pixels scaled by a power of two, the first
layer's weights are bits or 8-bit fixed-point numbers, and such a layer's sums are exact in fp32 in any order, so no bit behind
them depends on rounding; only the fp32 logits of a pooled head do.  The stand-alone first layers get images normalised the
usual way (mean and deviation), whose sums do round: a bit whose sum is that close to its threshold may differ.
"""
from __future__ import annotations

import torch

import paper_2006_16578_amd as bnn

MINUS_ONE, EXCLUDE = bnn.PAD_MINUS_ONE, bnn.PAD_EXCLUDE


def listed():
    return [
        # one request batch of a fully-connected layer while serving: latency, weights streamed once
        {"name": "fc_batch8", "kind": "fc", "M": 8, "N": 4096, "K": 4096, "out": "bits"},
        # a product of ordinary size whose integer sums are wanted, no dimension a multiple of a tile
        {"name": "bmm_ragged_int32", "kind": "fc", "M": 3001, "N": 2047, "K": 3500, "out": "int32"},
        # the large end of the bit matrix product sweep
        {"name": "bmm_16384", "kind": "fc", "M": 16384, "N": 16384, "K": 16384, "out": "bits"},
        # real-valued operands binarized on the way, real-valued result: a layer inside an otherwise real-valued program
        {"name": "general_4096", "kind": "fc_general", "M": 4096, "N": 4096, "K": 4096},
        # the 3x3 convolution of a network's middle, batch 128
        {"name": "conv3x3_128_56", "kind": "conv", "B": 128, "H": 56, "W": 56, "C": 128, "O": 128, "k": 3, "stride": 1, "pad": 1,
         "mode": MINUS_ONE, "out": "bits"},
        # the second convolution of a residual block run layer by layer: int32 residual in, sum and bits out
        {"name": "conv3x3_residual", "kind": "conv", "B": 256, "H": 28, "W": 28, "C": 128, "O": 128, "k": 3, "stride": 1, "pad": 1,
         "mode": MINUS_ONE, "out": "residual"},
        # channel counts that fill no tile and no 128-bit unit, a 5x5 window, the paper's own padding rule
        {"name": "conv5x5_odd_exclude", "kind": "conv", "B": 64, "H": 27, "W": 27, "C": 96, "O": 200, "k": 5, "stride": 1, "pad": 2,
         "mode": EXCLUDE, "out": "bits"},
        # threshold and 2x2 pooling behind a convolution whose sums were kept
        {"name": "threshold_pool", "kind": "thrd_pool", "B": 32, "H": 112, "W": 112, "C": 128, "win": 2},
        # first layer with binarized weights on 224x224 images (VGG-16's)
        {"name": "first_bwn_224", "kind": "first", "weights": "bits", "B": 128, "HW": 224, "O": 64, "k": 3, "stride": 1, "pad": 1},
        # the benchmark network at its throughput batch
        {"name": "resnet18_batch256", "kind": "net", "net": "resnet18", "batch": 256},
        # a small network at the paper's latency batch: launches and short kernels
        {"name": "cifar_vgg_batch8", "kind": "net", "net": "cifar_vgg", "batch": 8},
        # the MLP at its throughput batch
        {"name": "mlp_batch1024", "kind": "net", "net": "mlp", "batch": 1024},
    ]


# bytes and operations no drawn case goes over
MAX_BYTES, MAX_FLOPS = 200e6, 1.2e12


def _log(rng, lo, hi):
    """A whole number spread over [lo, hi] by its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    while True:
        kind = rng.choice(["fc", "fc", "fc_general", "conv", "conv", "conv", "thrd_pool", "first", "net", "net"])
        if kind == "fc":
            c = {"M": _log(rng, 1, 16384), "N": _log(rng, 10, 16384), "K": _log(rng, 64, 16384),
                 "out": rng.choice(["bits", "bits", "int32"])}
        elif kind == "fc_general":
            c = {"M": _log(rng, 64, 8192), "N": _log(rng, 64, 8192), "K": _log(rng, 64, 8192)}
        elif kind == "conv":
            k = rng.choice([1, 3, 3, 3, 5])
            hw = _log(rng, 7, 112)
            c = {"B": _log(rng, 1, 256), "H": hw, "W": max(5, hw + rng.choice([0, 0, 0, -1, 3])),
                 "C": rng.choice([64, 128, 256, 512, _log(rng, 32, 512)]), "O": rng.choice([64, 128, 256, 512, _log(rng, 32, 512)]),
                 "k": k, "stride": rng.choice([1, 1, 1, 2]), "pad": k // 2, "mode": rng.choice([MINUS_ONE, EXCLUDE]),
                 "out": rng.choice(["bits", "bits", "residual", "int32"])}
        elif kind == "thrd_pool":
            hw = _log(rng, 8, 224)
            c = {"B": _log(rng, 1, 256), "H": hw, "W": hw + rng.choice([0, 0, 1]), "C": rng.choice([64, 128, 256, _log(rng, 32, 512)]),
                 "win": 2}
        elif kind == "first":
            k, stride, pad = rng.choice([(3, 1, 1), (3, 2, 1), (5, 1, 2), (7, 2, 3), (7, 4, 3), (11, 4, 2)])
            c = {"weights": rng.choice(["bits", "bits", "f32"]), "B": _log(rng, 1, 128), "HW": rng.choice([32, 224, _log(rng, 32, 224)]),
                 "O": rng.choice([64, 128, _log(rng, 32, 128)]), "k": k, "stride": stride, "pad": pad}
            if c["weights"] == "f32" and k == 11:
                continue
        else:
            net = rng.choice(["resnet18", "mlp", "cifar_vgg", "cifar_resnet14", "alexnet", "vgg16"])
            c = {"net": net, "batch": _log(rng, 1, {"mlp": 32768, "cifar_vgg": 512, "cifar_resnet14": 512, "vgg16": 16}.get(net, 192))}
        c["kind"] = kind
        w = work(c)
        if w["bytes"] <= MAX_BYTES and w["flops"] <= MAX_FLOPS:
            return c


# ------------------------------------------------------------------------------------------ networks
def _layers(net):
    """[(op, ...)] of a network: first(O, k, stride, pad, weights) | conv(C, O, k, pad) | pool | block(cin, cout, stride) |
    fc(K, N) | head(C, J); and the image size."""
    def convs(*co):
        return [("conv", c, o, 3, 1) for c, o in co]

    def fcs(*dims):
        return [("fc", a, b) for a, b in zip(dims, dims[1:])]

    if net == "mlp":
        return fcs(784, 1024, 1024, 1024, 10), 0
    if net == "resnet18":
        return [("first", 64, 7, 4, 3, "f32")] + [("block", a, b, s) for a, b, s in (
            (64, 64, 1), (64, 64, 1), (64, 128, 2), (128, 128, 1), (128, 256, 2), (256, 256, 1), (256, 512, 2),
            (512, 512, 1))] + [("head", 512, 1000)], 224
    if net == "cifar_vgg":
        return ([("first", 128, 3, 1, 1, "bits")] + convs((128, 128)) + [("pool",)] + convs((128, 256), (256, 256)) + [("pool",)]
                + convs((256, 512), (512, 512)) + [("pool",)] + fcs(8192, 1024, 1024, 10)), 32
    if net == "cifar_resnet14":
        return [("first", 128, 3, 2, 1, "bits")] + [("block", a, b, s) for a, b, s in (
            (128, 128, 1), (128, 128, 1), (128, 256, 2), (256, 256, 1), (256, 512, 2), (512, 512, 1))] + fcs(8192, 512, 10), 32
    if net == "alexnet":
        return ([("first", 128, 11, 4, 2, "bits"), ("pool",), ("conv", 128, 256, 5, 2), ("pool",)]
                + convs((256, 256), (256, 256), (256, 256)) + [("pool",)] + fcs(9216, 4096, 4096, 1000)), 224
    if net == "vgg16":
        return ([("first", 64, 3, 1, 1, "bits")] + convs((64, 64)) + [("pool",)] + convs((64, 128), (128, 128)) + [("pool",)]
                + convs((128, 256), (256, 256), (256, 256)) + [("pool",)] + convs((256, 512), (512, 512), (512, 512)) + [("pool",)]
                + convs((512, 512), (512, 512), (512, 512)) + [("pool",)] + fcs(25088, 4096, 4096, 1000)), 224
    raise KeyError(net)


def _out_hw(hw, k, stride, pad):
    return (hw + 2 * pad - k) // stride + 1


def _net_work(net, batch):
    layers, hw = _layers(net)
    flops = weight_bytes = 0
    in_bytes = batch * (784 if net == "mlp" else hw * hw * 3 * 4)
    for L in layers:
        if L[0] == "first":
            _, O, k, s, p, weights = L
            hw = _out_hw(hw, k, s, p)
            flops += 2 * hw * hw * O * k * k * 3
            weight_bytes += O * k * k * (12 if weights == "f32" else 4) + 4 * O
        elif L[0] == "conv":
            _, C, O, k, p = L
            flops += 2 * hw * hw * O * k * k * C
            weight_bytes += O * k * k * C // 8 + 4 * O
        elif L[0] == "pool":
            hw //= 2
        elif L[0] == "block":
            _, a, b, s = L
            hw = _out_hw(hw, 3, s, 1)
            flops += 2 * hw * hw * b * (9 * a + 9 * b + (a if (s != 1 or a != b) else 0))
            weight_bytes += b * (9 * a + 9 * b) // 8 + 8 * b + (a * b // 8 if (s != 1 or a != b) else 0)
        elif L[0] == "fc":
            flops += 2 * L[1] * L[2]
            weight_bytes += L[1] * L[2] // 8 + 4 * L[2]
        else:
            flops += 2 * L[1] * L[2]
            weight_bytes += 4 * L[1] * L[2]
    return {"bytes": in_bytes + weight_bytes + batch * layers[-1][2] * 4, "flops": batch * flops}


def work(case):
    """What a pass cannot do without: inputs read once, outputs written once, two operations for each product."""
    kind = case["kind"]
    if kind in ("fc", "fc_general"):
        M, N, K = case["M"], case["N"], case["K"]
        if kind == "fc_general":
            return {"bytes": 4 * (M * K + N * K + M * N), "flops": 2 * M * N * K}
        out = 4 * M * N if case["out"] == "int32" else M * N / 8 + 4 * N
        return {"bytes": (M + N) * K / 8 + out, "flops": 2 * M * N * K}
    if kind == "conv":
        P, Q = (_out_hw(case[d], case["k"], case["stride"], case["pad"]) for d in "HW")
        pix, O, C, kk = case["B"] * P * Q, case["O"], case["C"], case["k"] ** 2
        out = {"bits": pix * O / 8 + 4 * O, "int32": 4 * pix * O, "residual": pix * O * (8 + 1 / 8) + 4 * O}[case["out"]]
        return {"bytes": (case["B"] * case["H"] * case["W"] + O * kk) * C / 8 + out, "flops": 2 * pix * O * kk * C}
    if kind == "thrd_pool":
        n = case["B"] * case["H"] * case["W"] * case["C"]
        return {"bytes": 4 * n + 4 * case["C"] + n / 8 + n / 32, "flops": 0}
    if kind == "first":
        P = _out_hw(case["HW"], case["k"], case["stride"], case["pad"])
        pix, kkc = case["B"] * P * P, case["k"] ** 2 * 3
        return {"bytes": case["B"] * case["HW"] ** 2 * 12 + case["O"] * kkc * (4 if case["weights"] == "f32" else 1 / 8) + pix * case["O"] / 8,
                "flops": 2 * pix * case["O"] * kkc}
    return _net_work(case["net"], case["batch"])


# ------------------------------------------------------------------------------------------ inputs
class _Draw:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def bits(self, *shape, nbits, ldw=None):
        """Fair-coin packed rows [*shape][ldw] with the bits past nbits 0."""
        kw = bnn.nwords(nbits)
        w = torch.randint(-2 ** 31, 2 ** 31, shape + (kw if ldw is None else ldw,), dtype=torch.int32, device="cuda", generator=self.g)
        if nbits % 32:
            w[..., kw - 1] &= (1 << (nbits % 32)) - 1
        w[..., kw:] = 0
        return w

    def ints(self, *shape, lo, hi, dtype=torch.int32):
        return torch.randint(lo, hi + 1, shape, dtype=dtype, device="cuda", generator=self.g)

    def normal(self, *shape, scale=1.0):
        return torch.randn(*shape, device="cuda", generator=self.g) * scale

    def pixels(self, *shape):
        return self.ints(*shape, lo=0, hi=255, dtype=torch.uint8)


def prepare(case, seed):
    d, kind = _Draw(seed), case["kind"]
    s = {"case": case}
    if kind == "fc":
        ldw = bnn.round_up(bnn.nwords(case["K"]), 4)
        s["A"] = d.bits(case["M"], nbits=case["K"], ldw=ldw)
        s["B"] = d.bits(case["N"], nbits=case["K"], ldw=ldw)
        s["thr"] = d.ints(case["N"], lo=-case["K"] // 8, hi=case["K"] // 8)
    elif kind == "fc_general":
        s["A"], s["B"] = d.normal(case["M"], case["K"]), d.normal(case["N"], case["K"])
    elif kind == "conv":
        P, Q = (_out_hw(case[x], case["k"], case["stride"], case["pad"]) for x in "HW")
        s["x"] = d.bits(case["B"], case["H"], case["W"], nbits=case["C"])
        s["filt"] = d.bits(case["O"], case["k"], case["k"], nbits=case["C"])
        s["thr"] = d.ints(case["O"], lo=-64, hi=64)
        s["residual"] = d.ints(case["B"], P, Q, case["O"], lo=-600, hi=600) if case["out"] == "residual" else None
    elif kind == "thrd_pool":
        s["X"] = d.ints(case["B"], case["H"], case["W"], case["C"], lo=-200, hi=200)
        s["thr"] = d.ints(case["C"], lo=-64, hi=64)
    elif kind == "first":
        s["x"] = (d.pixels(case["B"], case["HW"], case["HW"], 3).float() / 255 - 0.45) / 0.225
        O, k = case["O"], case["k"]
        s["w"] = d.bits(O, k, k, nbits=3) if case["weights"] == "bits" else d.normal(O, k, k, 3, scale=0.05)
        s["thr"] = d.normal(O, scale=0.5)
    else:
        s.update(_prepare_net(d, case))
    return s


def _prepare_net(d, case):
    layers, hw = _layers(case["net"])
    net, host = bnn.Net(), []          # host: the same layers, for exact()
    if case["net"] == "mlp":
        net.input_u8(784, 127)
        x = d.pixels(case["batch"], 784)
    else:
        x = (d.pixels(case["batch"], hw, hw, 3).float() - 128) / 128
    for i, L in enumerate(layers):
        if L[0] == "first":
            _, O, k, st, p, weights = L
            thr = torch.zeros(O, device="cuda")
            if weights == "f32":
                w = (d.normal(O, k, k, 3, scale=0.02) * 1024).round().clamp(-127, 127) / 1024
                net.input_conv_f32(w, thr, hw, hw, st, p)
            else:
                w = d.bits(O, k, k, nbits=3)
                net.input_bwn_f32(w, thr, hw, hw, 3, st, p)
            host.append((w, thr))
        elif L[0] == "conv":
            _, C, O, k, p = L
            w, thr = d.bits(O, k, k, nbits=C), d.ints(O, lo=-64, hi=64)
            net.add_conv(w, thr, C, 1, p)
            host.append((w, thr))
        elif L[0] == "pool":
            net.add_pool(2, 2)
            host.append(())
        elif L[0] == "block":
            _, a, b, st = L
            w1, t1 = d.bits(b, 3, 3, nbits=a), d.ints(b, lo=-64, hi=64)
            w2, t2 = d.bits(b, 3, 3, nbits=b), d.ints(b, lo=-64, hi=64)
            wd = d.bits(b, 1, 1, nbits=a) if (st != 1 or a != b) else None
            net.add_block(w1, t1, w2, t2, wd, a, b, st)
            host.append((w1, t1, w2, t2, wd))
        elif L[0] == "fc":
            last = i + 1 == len(layers)
            w = d.bits(L[2], nbits=L[1], ldw=bnn.round_up(bnn.nwords(L[1]), 4))
            thr = None if last else d.ints(L[2], lo=-32, hi=32)
            net.add_fc(w, thr, L[1])
            host.append((w, thr))
        else:
            w = d.normal(L[2], L[1], scale=0.02)
            net.add_head_f32(w)
            host.append((w,))
    return {"net": net, "x": x, "layers": host}


# ------------------------------------------------------------------------------------------ a pass
def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "fc":
        if c["out"] == "int32":
            return bnn.bmm(s["A"], s["B"], c["K"])
        return bnn.bmm_thr(s["A"], s["B"], s["thr"], c["K"])
    if kind == "fc_general":
        return bnn.bmm_general_f32(s["A"], s["B"])
    if kind == "conv":
        if c["out"] == "int32":
            return bnn.bconv(s["x"], s["filt"], c["C"], c["stride"], c["pad"], c["mode"])
        if c["out"] == "residual":
            return bnn.bconv_thr(s["x"], s["filt"], s["thr"], c["C"], c["stride"], c["pad"], c["mode"], residual=s["residual"],
                                 want_sum=True)
        return bnn.bconv_thr(s["x"], s["filt"], s["thr"], c["C"], c["stride"], c["pad"], c["mode"])
    if kind == "thrd_pool":
        bits = bnn.threshold_pack(s["X"], s["thr"])
        return bits, bnn.maxpool_or(bits, c["C"], c["win"], c["win"])
    if kind == "first":
        if c["weights"] == "bits":
            return bnn.bwn_conv_thr(s["x"], s["w"], s["thr"], 3, c["stride"], c["pad"])
        return bnn.conv_f32_split_thr(s["x"], s["w"], s["thr"], c["stride"], c["pad"])
    return s["net"].forward(s["x"])


def tolerance(case):
    if case["kind"] == "first":
        # fp32 sums in another order: a bit differs where its sum is within rounding of its threshold.  Measured between
        # two kernels and against 64 bits: up to 2.5e-6 of the words; in a small output, one word.
        P = _out_hw(case["HW"], case["k"], case["stride"], case["pad"])
        return {"rel": 0.0, "differ": max(1e-5, 1.0 / (case["B"] * P * P * bnn.nwords(case["O"])))}
    if case["kind"] == "net" and case["net"] == "resnet18":
        return {"rel": 7e-7}               # fp32 head, a dot product of 512 terms: 1.6e-7 from 64 bits
    return "exact"


# ------------------------------------------------------------------------------------------ the same in 64 bits
def _unpack(words, nbits):
    """Packed [..., w] -> +1/-1 in float64 [..., nbits]."""
    shifts = torch.arange(32, dtype=torch.int32, device=words.device)
    b = (words.unsqueeze(-1) >> shifts) & 1
    return (b.reshape(*words.shape[:-1], -1)[..., :nbits] * 2 - 1).double()


def _pack(mask, ldw=None):
    n = mask.shape[-1]
    kw = (n + 31) // 32
    full = torch.zeros(*mask.shape[:-1], 32 * (kw if ldw is None else ldw), dtype=torch.int64, device=mask.device)
    full[..., :n] = mask
    v = (full.reshape(*mask.shape[:-1], -1, 32) << torch.arange(32, device=mask.device)).sum(-1)
    return torch.where(v >= 2 ** 31, v - 2 ** 32, v).to(torch.int32)


def _conv(x, f, stride, pad, fill):
    """Cross-correlation in float64: x [N][H][W][C], f [O][k][k][C]; positions outside the image hold `fill`."""
    N, H, W, C = x.shape
    O, k = f.shape[0], f.shape[1]
    P, Q = _out_hw(H, k, stride, pad), _out_hw(W, k, stride, pad)
    xp = torch.full((N, H + 2 * pad, W + 2 * pad, C), float(fill), dtype=torch.float64, device=x.device)
    xp[:, pad:pad + H, pad:pad + W] = x
    y = torch.zeros(N * P * Q, O, dtype=torch.float64, device=x.device)
    for r in range(k):
        for t in range(k):
            y.addmm_(xp[:, r:r + (P - 1) * stride + 1:stride, t:t + (Q - 1) * stride + 1:stride].reshape(-1, C), f[:, r, t].t().contiguous())
    return y.reshape(N, P, Q, O)


def _by_images(fn, x, step=32):
    """fn over slices of the batch, results joined (bounds the memory of the float64 copies)."""
    parts = [fn(x[i:i + step], i) for i in range(0, x.shape[0], step)]
    if isinstance(parts[0], tuple):
        return tuple(torch.cat(p) for p in zip(*parts))
    return torch.cat(parts)


def exact(case, seed):
    s, kind = prepare(case, seed), case["kind"]
    if kind == "fc":
        v = _unpack(s["A"], case["K"]) @ _unpack(s["B"], case["K"]).t().contiguous()
        if case["out"] == "int32":
            return v.to(torch.int32)
        return _pack(v >= s["thr"], bnn.round_up(bnn.nwords(case["N"]), 4))
    if kind == "fc_general":
        one = torch.ones((), dtype=torch.float64, device="cuda")
        return torch.where(s["A"] >= 0, one, -one) @ torch.where(s["B"] >= 0, one, -one).t().contiguous()
    if kind == "conv":
        f = _unpack(s["filt"], case["C"])
        fill = -1 if case["mode"] == MINUS_ONE else 0

        def part(x, i):
            v = _conv(_unpack(x, case["C"]), f, case["stride"], case["pad"], fill)
            if case["out"] == "residual":
                v = v + s["residual"][i:i + x.shape[0]]
                return _pack(v >= s["thr"]), v.to(torch.int32)
            return v.to(torch.int32) if case["out"] == "int32" else _pack(v >= s["thr"])
        return _by_images(part, s["x"])
    if kind == "thrd_pool":
        def part(x, i):
            m = x >= s["thr"]
            w, (P, Q) = case["win"], (case["H"] // case["win"], case["W"] // case["win"])
            pooled = m[:, :P * w, :Q * w].reshape(x.shape[0], P, w, Q, w, -1).amax(dim=(2, 4))
            return _pack(m), _pack(pooled)
        return _by_images(part, s["X"], 8)
    if kind == "first":
        w = _unpack(s["w"], 3) if case["weights"] == "bits" else s["w"].double()
        return _by_images(lambda x, i: _pack(_conv(x.double(), w, case["stride"], case["pad"], 0) >= s["thr"]), s["x"], 16)
    return _by_images(lambda x, i: _exact_net(case, s["layers"], x), s["x"], 1024 if case["net"] == "mlp" else 16)


def _sign(mask):
    return mask.double() * 2 - 1


def _exact_net(case, params, x):
    layers, _ = _layers(case["net"])
    v = _sign(x >= 127) if case["net"] == "mlp" else x.double()
    residual = None                        # running sums of a chain of residual blocks
    for L, p in zip(layers, params):
        if L[0] == "first":
            w = p[0].double() if L[5] == "f32" else _unpack(p[0], 3)
            v = _sign(_conv(v, w, L[3], L[4], 0) >= p[1])
        elif L[0] == "conv":
            v = _sign(_conv(v, _unpack(p[0], L[1]), 1, L[4], -1) >= p[1])
        elif L[0] == "pool":
            P, Q = v.shape[1] // 2, v.shape[2] // 2
            v = v[:, :2 * P, :2 * Q].reshape(v.shape[0], P, 2, Q, 2, -1).amax(dim=(2, 4))
        elif L[0] == "block":
            _, a, b, st = L
            w1, t1, w2, t2, wd = p
            h = _sign(_conv(v, _unpack(w1, a), st, 1, -1) >= t1)
            short = _conv(v, _unpack(wd, a), st, 0, -1) if wd is not None else v if residual is None else residual
            residual = _conv(h, _unpack(w2, b), 1, 1, -1) + short
            v = _sign(residual >= t2)
        elif L[0] == "fc":
            sums = v.reshape(v.shape[0], -1) @ _unpack(p[0], L[1]).t().contiguous()
            if p[1] is None:
                return sums.to(torch.int32)
            v = _sign(sums >= p[1])
        else:
            return v.mean(dim=(1, 2)) @ p[0].double().t().contiguous()
