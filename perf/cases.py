"""Timed cases: the calls that a program using the library makes, through its public binding.

A case is a dict of plain values.  `kind` says which entry points it takes:
  infer    im_attention_fwd without saved tensors
  train    im_attention_fwd + im_attention_bwd, every gradient of a given parameter
  encoder  `layers` x gsit_layer_fwd (inference)
  layer    gsit_layer_fwd_train + gsit_layer_bwd, every parameter gradient
  model    gsit_model_fwd
Lengths t / v / a are the padded segment lengths (text, vision, audio).  `pad` is what the caller
knows about padding: "none", "valid_len" (per-sample lengths, uniform between half and all of a
segment), "key_pad" (a tenth of the positions masked one by one) or "packed" (no padding rows in
memory, lengths with the mean and variance of the CMU-MOSI training split).
A sample's lengths are the quantiles of their distribution in an order drawn from the seed, so that
every seed has the same number of rows.  The key bias is left out where biases are given: it adds a
constant to every score of a row, the softmax does not see it, and its gradient is identically zero.
"""
import math
from statistics import NormalDist

import torch

from paper_2505_01068_amd import binding as B
from paper_2505_01068_amd.synth import MOSI_LENGTH_STATS


def listed():
    c = lambda name, kind, dtype, batch, seg, d, heads, mask="ifm_forward", pad="none", **more: dict(  # noqa: E731
        name=name, kind=kind, dtype=dtype, batch=batch, t=seg[0], v=seg[1], a=seg[2], d=d, heads=heads, mask=mask, pad=pad,
        bias=more.pop("bias", False), **more)
    return [
        # one small call on its own, as in an example or an online request: launch latency
        c("infer_fp32_tiny", "infer", "fp32", 2, (8, 8, 8), 32, 4),
        # training at the published model width in fp32, word-aligned features: 50 steps per modality
        c("train_fp32_short", "train", "fp32", 64, (50, 50, 50), 40, 8, pad="key_pad"),
        # the same, unaligned features at the dataset's maximum lengths, padded to the maximum
        c("train_fp32_long", "train", "fp32", 32, (50, 500, 375), 40, 8, pad="valid_len"),
        # the same without padding rows
        c("train_fp32_packed", "train", "fp32", 32, (50, 500, 375), 40, 8, pad="packed"),
        # one whole encoder layer of fp32 training (attention, LayerNorms, MLP), CMU-MOSEI lengths
        c("layer_fp32", "layer", "fp32", 32, (50, 500, 500), 40, 8, mask="ifm_backward", pad="valid_len", bias=True, d_ff=160),
        # bf16 encoder inference, four layers
        c("encoder_bf16", "encoder", "bf16", 32, (50, 500, 375), 64, 8, pad="valid_len", bias=True, d_ff=256, layers=4),
        # one encoder layer of bf16 training at that width
        c("layer_bf16", "layer", "bf16", 32, (50, 500, 375), 64, 8, bias=True, d_ff=256),
        # one encoder layer of bf16 training at head dimension 64, intra-modal mask
        c("layer_bf16_wide", "layer", "bf16", 8, (50, 500, 500), 256, 4, mask="iem", pad="valid_len", bias=True, d_ff=1024),
        # the whole model scoring a batch (4 + 4 inter-modal and 4 intra-modal layers)
        c("model_bf16_batch", "model", "bf16", 32, (50, 500, 375), 64, 8, pad="none", bias=True, d_ff=256, layers=4, n_out=1),
        # the whole model answering one request: MIntRec lengths, its 20 intents
        c("model_bf16_single", "model", "bf16", 1, (30, 230, 480), 64, 8, pad="valid_len", bias=True, d_ff=256, layers=4, n_out=20),
        # the largest: long sequences at width 512, training
        c("train_bf16_large", "train", "bf16", 8, (512, 2048, 2048), 512, 8),
        # long sequences of odd lengths, two live blocks per row, single masked keys, biases
        c("train_bf16_ragged", "train", "bf16", 3, (333, 1501, 1290), 256, 4, mask="self_only", pad="key_pad", bias=True),
    ]


MASKS = ("ifm_forward", "ifm_forward", "ifm_backward", "iem", "self_only", "structure1_a", "structure2_b", "structure3_a", "dense")


def draw(rng):
    """One more case of the same ranges.  The batch is cut where a draw would cost more than the largest listed case."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    kind, dtype, wide = rng.choice((
        ("infer", "fp32", False), ("train", "fp32", False), ("train", "fp32", False), ("layer", "fp32", False),
        ("encoder", "bf16", False), ("layer", "bf16", False), ("model", "bf16", False), ("model", "bf16", False),
        ("layer", "bf16", True), ("train", "bf16", True), ("train", "bf16", True)))
    case = dict(kind=kind, dtype=dtype, mask=rng.choice(MASKS), pad=rng.choice(("none", "valid_len", "key_pad")),
                bias=rng.random() < 0.5)
    if wide:
        case["heads"] = rng.choice((2, 4, 8))
        case["d"] = 64 * case["heads"]
        top = 2048 if kind == "train" else 500
        case["t"], case["v"], case["a"] = log(30, top // 4), log(100, top), log(100, top)
        case["batch"] = log(1, 16)
    else:
        case["d"], case["heads"] = rng.choice(((32, 4), (40, 8), (48, 6), (64, 8)) if dtype == "fp32" else ((64, 8),))
        if kind == "infer":
            case["t"], case["v"], case["a"], case["batch"] = rng.randint(4, 50), log(8, 200), log(8, 200), log(1, 16)
        else:
            case["t"], case["v"], case["a"] = rng.randint(20, 50), log(50, 500), log(50, 500)
            case["batch"] = log(1, 32) if kind == "model" else log(8, 64)
        if kind == "train" and rng.random() < 0.3:
            case.update(pad="packed", t=50, v=500, a=375)
    if kind in ("encoder", "layer", "model"):
        case["bias"] = True
        case["d_ff"] = 4 * case["d"]
    if kind in ("encoder", "model"):
        case["layers"] = rng.randint(1, 4)
    if kind == "model" and case["pad"] == "key_pad":
        case["pad"] = "valid_len"
    # pairs x width of the largest listed case of the family, with the padded lengths
    seg, lm = (case["t"], case["v"], case["a"]), B.NAMED_MASKS[case["mask"]]
    pairs = sum(seg[i] * seg[j] for i in range(3) for j in range(3) if (lm >> (3 * i + j)) & 1)
    most = (6291456 * 8 * 512 // (1 if kind == "train" else 4)) / case["d"] if wide else 32 * 300000 / case.get("layers", 1) ** 0.5
    if case["pad"] != "packed":
        case["batch"] = max(1, min(case["batch"], int(most / pairs)))
    if kind == "model":
        case["n_out"] = rng.choice((1, 3, 20)) if case["batch"] >= 16 else 20
    return case


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _seg(case):
    return (case["t"], case["v"], case["a"])


def _lengths(case):
    """Per segment the sorted lengths of the batch's samples: the quantiles (i + 1/2) / batch of their distribution."""
    n = case["batch"]
    q = [(i + 0.5) / n for i in range(n)]
    if case["pad"] == "valid_len":
        return [[(T + 1) // 2 + int(u * (T - (T + 1) // 2 + 1)) for u in q] for T in _seg(case)]
    if case["pad"] == "packed":
        out = []
        for T, mean, var in zip(_seg(case), MOSI_LENGTH_STATS["mean"], MOSI_LENGTH_STATS["var"]):
            s2 = math.log1p(var / (mean * mean))
            z = [NormalDist().inv_cdf(u) for u in q]
            out.append([min(T, max(1, round(math.exp(math.log(mean) - 0.5 * s2 + math.sqrt(s2) * x)))) for x in z])
        return out
    return [[T] * n for T in _seg(case)]


class State:
    pass


def _layer_params(d, d_ff, rand, uniform, dt):
    p = {n: uniform(d, d) for n in ("wq", "wk", "wv", "wo")}
    p["w1"], p["w2"] = uniform(d, d_ff), uniform(d_ff, d)
    for n in ("ln1", "ln2"):
        p[n + "_g"], p[n + "_b"] = (1 + 0.1 * rand(d)).to(dt), (0.1 * rand(d)).to(dt)
    for n, m in (("bq", d), ("bv", d), ("bo", d), ("b1", d_ff), ("b2", d)):
        p[n] = (0.1 * rand(m)).to(dt)
    return p


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dt, d, n, seg = _dtype(case), case["d"], case["batch"], _seg(case)
    T = sum(seg)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=gen)  # noqa: E731

    def uniform(r, c):   # Xavier
        return ((torch.rand(r, c, device="cuda", generator=gen) * 2 - 1) * math.sqrt(6.0 / (r + c))).to(dt)

    s = State()
    s.case, s.kind = case, case["kind"]
    lengths = torch.tensor(_lengths(case), dtype=torch.int32)
    if case["pad"] in ("valid_len", "packed"):
        cpu = torch.Generator().manual_seed(int(seed))
        lengths = torch.stack([l[torch.randperm(n, generator=cpu)] for l in lengths])
    lengths = lengths.t().contiguous()   # [batch, 3]
    s.valid_len = s.key_pad = None
    cu, rows = None, n * T
    if case["pad"] == "packed":
        cu = torch.cat([torch.zeros(1, dtype=torch.int64), lengths.reshape(-1).cumsum(0)]).to(torch.int32).cuda()
        rows = int(lengths.sum())
        s.x = rand(rows, d)
    else:
        s.x = rand(n, T, d)
        if case["pad"] == "valid_len":
            s.valid_len = lengths.cuda()
            pos = torch.cat([torch.arange(k, device="cuda") for k in seg])
            which = torch.cat([torch.full((k,), i, device="cuda") for i, k in enumerate(seg)])
            s.x = s.x * (pos[None, :] < s.valid_len[:, which])[:, :, None]
        elif case["pad"] == "key_pad":
            u = torch.rand(n, T, device="cuda", generator=gen)
            off, parts = 0, []
            for k in seg:   # a tenth of every segment of every sample
                rank = u[:, off:off + k].argsort(dim=1).argsort(dim=1)
                parts.append((rank < round(0.1 * k)).to(torch.uint8))
                off += k
            s.key_pad = torch.cat(parts, dim=1).contiguous()
            s.x = s.x * (s.key_pad == 0)[:, :, None]
    s.x = s.x.to(dt)
    lm = 0 if s.kind == "model" else B.NAMED_MASKS[case["mask"]]
    s.shape = B.make_shape(n, seg, d, case["heads"], lm, 1.0 / math.sqrt(d // case["heads"]), case["dtype"], cu_rows=cu, total_rows=rows)
    buf = lambda size: torch.empty(max(int(size), 1), dtype=torch.uint8, device="cuda")  # noqa: E731
    s.y = torch.empty_like(s.x)
    if s.kind in ("train", "layer"):
        s.dy = rand(*s.x.shape).to(dt)
        s.dx = torch.empty_like(s.x)
    if s.kind in ("infer", "train"):
        s.w = {k: uniform(d, d) for k in ("wq", "wk", "wv", "wo")}
        s.b = {k: (0.1 * rand(d)).to(dt) for k in ("bq", "bv", "bo")} if case["bias"] else {}
        saved, ws = B.im_attention_sizes(s.shape)
        s.ws = buf(ws)
        if s.kind == "train":
            s.saved = buf(saved)
            s.grads = {"d" + k: torch.empty(t.shape, dtype=torch.float32, device="cuda") for k, t in {**s.w, **s.b}.items()}
    elif s.kind == "encoder":
        s.p = [_layer_params(d, case["d_ff"], rand, uniform, dt) for _ in range(case["layers"])]
        s.ws = buf(B.gsit_layer_sizes(s.shape, case["d_ff"]))
        s.bufs = (s.y, torch.empty_like(s.x))
    elif s.kind == "layer":
        s.p = _layer_params(d, case["d_ff"], rand, uniform, dt)
        saved, ws = B.gsit_layer_train_sizes(s.shape, case["d_ff"])
        s.saved, s.ws = buf(saved), buf(ws)
        s.grads = {k: torch.empty(t.shape, dtype=torch.float32, device="cuda") for k, t in s.p.items()}
    else:
        stack = lambda w, f: [_layer_params(w, f, rand, uniform, dt) for _ in range(case["layers"])]  # noqa: E731
        weights = {"fwd_layers": stack(d, case["d_ff"]), "bwd_layers": stack(d, case["d_ff"]),
                   "intra_layers": stack(2 * d, 2 * case["d_ff"]), "wf": uniform(6 * d, case["n_out"]),
                   "bf": (0.1 * rand(case["n_out"])).to(dt)}
        s.model = B.make_model(weights, case["d_ff"], 2 * case["d_ff"], case["heads"], 1.0 / math.sqrt(2 * d // case["heads"]))
        s.ws = buf(B.gsit_model_sizes(s.shape, s.model))
        s.out = torch.empty(n, case["n_out"], dtype=dt, device="cuda")
    return s


def run(s):
    pads = dict(valid_len=s.valid_len, key_pad=s.key_pad, workspace=s.ws)
    if s.kind == "infer":
        return B.im_attention_fwd(s.shape, s.x, **s.w, **s.b, y=s.y, **pads)
    if s.kind == "train":
        B.im_attention_fwd(s.shape, s.x, **s.w, **s.b, y=s.y, saved=s.saved, **pads)
        B.im_attention_bwd(s.shape, s.x, **s.w, saved=s.saved, dy=s.dy, dx=s.dx, **s.grads, **pads)
        return {"y": s.y, "dx": s.dx, **s.grads}
    if s.kind == "encoder":
        h = s.x
        for i, p in enumerate(s.p):
            h = B.gsit_layer_fwd(s.shape, s.case["d_ff"], h, p, y=s.bufs[i % 2], **pads)
        return h
    if s.kind == "layer":
        B.gsit_layer_fwd_train(s.shape, s.case["d_ff"], s.x, s.p, s.saved, y=s.y, **pads)
        B.gsit_layer_bwd(s.shape, s.case["d_ff"], s.x, s.p, s.saved, s.dy, s.grads, dx=s.dx, **pads)
        return {"y": s.y, "dx": s.dx, **s.grads}
    return B.gsit_model_fwd(s.shape, s.model, s.x, out=s.out, **pads)


def _pairs(case, mask):
    """(query row in memory, valid live key) pairs over the batch."""
    seg, lens = _seg(case), _lengths(case)
    keys = [sum(l) / case["batch"] * (0.9 if case["pad"] == "key_pad" else 1.0) for l in lens]
    rows = [k if case["pad"] == "packed" else T for k, T in zip(keys, seg)]
    lm = B.NAMED_MASKS[mask]
    return case["batch"] * sum(rows[i] * keys[j] for i in range(3) for j in range(3) if (lm >> (3 * i + j)) & 1)


def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    d, f, kind = case["d"], case.get("d_ff", 0), case["kind"]
    rows = sum(map(sum, _lengths(case))) if case["pad"] == "packed" else case["batch"] * sum(_seg(case))
    fwd = lambda mask, w, ff: 4.0 * _pairs(case, mask) * w + rows * (8.0 * w * w + 4.0 * w * ff)  # noqa: E731
    weights = 4 * d * d + 2 * d * f
    if kind == "infer":
        return {"bytes": es * (2.0 * rows * d + weights), "flops": fwd(case["mask"], d, 0)}
    if kind in ("train", "layer"):
        # forward and 2.5 times its attention, twice its products in the backward; x, dy, y, dx and the fp32 gradients
        attention = 4.0 * _pairs(case, case["mask"]) * d
        return {"bytes": es * (4.0 * rows * d + weights) + 4.0 * weights, "flops": 3 * fwd(case["mask"], d, f) + 0.5 * attention}
    if kind == "encoder":
        return {"bytes": es * (2.0 * rows * d + case["layers"] * weights), "flops": case["layers"] * fwd(case["mask"], d, f)}
    n = case["layers"]
    flops = n * (fwd("ifm_forward", d, f) + fwd("ifm_backward", d, f) + fwd("iem", 2 * d, 2 * f)) + 12.0 * case["batch"] * d * case["n_out"]
    return {"bytes": es * (rows * d + n * 6.0 * weights + case["batch"] * case["n_out"]), "flops": flops}


def tolerance(case):
    # Four times the largest error seen against the fp64 oracle (2-norm; and largest element, over the larger of its value
    # and the output's root mean square), over all outputs of the listed cases and of ten drawn ones.
    if case["dtype"] == "fp32":
        return {"rel": 2.5e-6, "max": 3e-5}   # 5.7e-7 (a LayerNorm gain gradient), 6.1e-6 (dx)
    if case["kind"] == "model":
        return {"rel": 0.03, "max": 0.1}      # 7.8e-3, 2.4e-2: up to twelve layers, few outputs
    return {"rel": 0.022, "max": 0.3}         # 5.6e-3 (dWq), 7.3e-2 (dx)
