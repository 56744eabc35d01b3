"""The measured work of this package: what a training job that freezes layers has
the library do, through the package's public entry points.

Six paths, told apart by case["path"]:

  step      refresh of the reference model and evaluation in one call
            (PlasticityEvaluator.step): snapshot -> int8 weights -> reference
            forward -> one score per layer.
  eval      evaluation with a reference model that is already quantised
            (PlasticityEvaluator.evaluate): what runs every few iterations
            between two refreshes.
  forward   reference forward alone (ref_forward) at the precisions and
            activation codes the evaluator does not drive: float16 / float32
            references and affine uint8 activations.
  metric    the score of two stored activations (plasticity).
  snapshot  quantisation of a weight snapshot alone (quantize_weights).
  cache     one training iteration's use of the activation cache: the coming
            mini-batch put in, the current one read back by sample id.

Inputs are drawn on the GPU from the seed: N(0, 1) mini-batches (post-ReLU ones
for bottlenecks), He / Xavier weights, and as A_T the fp32 forward of slightly
perturbed weights, which is what the training model's hook delivers.
"""
from __future__ import annotations

import math

import torch

from paper_2201_06227_amd import binding as eg
from paper_2201_06227_amd.evaluator import PlasticityEvaluator

DEVICE = "cuda"
KINDS = {"fc": eg.FC_RELU, "basic": eg.BASIC_BLOCK, "bottleneck": eg.BOTTLENECK}
PRECISIONS = {"f16": eg.REF_F16, "f32": eg.REF_F32}


# ---- cases ------------------------------------------------------------------------------------

def _fc(path, batch, c_in, c_out, **more):
    return dict(path=path, kind="fc", batch=batch, c_in=c_in, c_out=c_out, **more)


def _conv(path, kind, batch, c_in, c_mid, height, width, **more):
    return dict(path=path, kind=kind, batch=batch, c_in=c_in, c_mid=c_mid, height=height, width=width, **more)


def _encoder(path, batch, seq, hidden, heads, ffn, layers, **more):
    return dict(path=path, kind="encoder", batch=batch, seq=seq, hidden=hidden, heads=heads, ffn=ffn, layers=layers, **more)


def listed():
    return [
        # One fully connected layer, batch 32: the smallest call; launches and host work are all of it.
        dict(_fc("step", 32, 512, 512, train="f32"), name="fc_step"),
        # Stage-1 basic block of a CIFAR residual network (16 channels): many pixels, hardly any arithmetic.
        dict(_conv("step", "basic", 128, 16, 16, 32, 32, train="f32"), name="narrow_block_step"),
        # Stage-3 bottleneck of an ImageNet residual network, refreshed and scored.
        dict(_conv("step", "bottleneck", 64, 1024, 256, 14, 14, train="f32"), name="bottleneck_step"),
        # A last-stage bottleneck on 7x7 images with the scales a deployed convolutional network has: static
        # activation scales, one weight scale per output channel; the last mini-batch of an epoch (ragged).
        dict(_conv("eval", "bottleneck", 50, 2048, 512, 7, 7, train="f32", static=True, per_channel=True),
             name="static_block_eval"),
        # One Transformer encoder layer, mixed-precision training (bf16 activations).
        dict(_encoder("step", 32, 128, 768, 12, 3072, 1, train="bf16"), name="encoder_step"),
        # The whole 12-layer encoder stack at its full size: one score per layer in one call.
        dict(_encoder("step", 64, 256, 768, 12, 3072, 12, train="f32"), name="stack_step"),
        # Two encoder layers between refreshes, odd sequence length: rows that fill no tile.
        dict(_encoder("eval", 24, 197, 768, 12, 3072, 2, train="bf16"), name="ragged_stack_eval"),
        # The score alone, on a mobile network's last activation: a batch that fills no block, both types.
        dict(path="metric", batch=100, features=62720, train="bf16", ref="f32", name="metric"),
        # A refresh alone: the weights of four encoder layers, one scale per output channel.
        dict(path="snapshot", kind="encoder", hidden=768, ffn=3072, layers=4, weights="f32", per_channel=True,
             name="snapshot"),
        # The float16 reference model, the fallback when int8 fails: one encoder layer.
        dict(_encoder("forward", 32, 128, 768, 12, 3072, 1, precision="f16"), name="float16_forward"),
        # Affine uint8 activation codes, the default of the common quantisation frameworks.
        dict(_conv("forward", "bottleneck", 64, 1024, 256, 14, 14, precision="affine"), name="affine_forward"),
        # Activations of a frozen stage: put of the coming mini-batch, get of one by shuffled sample ids.
        dict(path="cache", batch=64, features=200704, window=5, rows="f32", name="cache"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_conv(rng, path, kinds, **more):
    kind = rng.choice(kinds)
    side = _log(rng, 4, 56)
    height, width = side, max(1, side + rng.choice((0, 0, 0, -1, 1, 3)))
    batch = _log(rng, 4, 128)
    pixels = batch * height * width
    if kind == "basic":
        c = rng.choice((16, 16, 32, 64, _log(rng, 8, 128)))
        while pixels * c > 12_000_000 and c > 8:
            c = max(8, c // 2)
        return _conv(path, kind, batch, c, c, height, width, **more)
    c_in = rng.choice((64, 256, 512, 1024, 2048, _log(rng, 48, 2048)))
    while pixels * c_in > 16_000_000 and c_in > 48:
        c_in = max(48, c_in // 2)
    return _conv(path, kind, batch, c_in, max(16, c_in // 4), height, width, **more)


def _draw_encoder(rng, path, layers, most, **more):
    heads = rng.choice((4, 6, 8, 12, 16))
    hidden = heads * rng.choice((64, 64, 64, 48, 32))
    seq = rng.choice((_log(rng, 16, 384), 64, 128, 256))
    batch = max(1, min(_log(rng, 4, 96), most // seq))
    return _encoder(path, batch, seq, hidden, heads, hidden * 4, layers, **more)


def draw(rng):
    train = rng.choice(("f32", "f32", "bf16"))
    path = rng.choice(("fc", "narrow", "block", "static", "layer", "stack", "metric", "snapshot", "float", "affine", "cache"))
    if path == "fc":
        return _fc(rng.choice(("step", "eval")), _log(rng, 8, 128), _log(rng, 64, 4096), _log(rng, 64, 4096), train=train)
    if path == "narrow":
        c = rng.choice((16, 16, _log(rng, 8, 16)))
        return _conv(rng.choice(("step", "eval")), "basic", _log(rng, 8, 128), c, c, 32, 32 + rng.choice((0, 0, -1, 5)),
                     train=train)
    if path == "block":
        return _draw_conv(rng, rng.choice(("step", "eval")), ("basic", "bottleneck"), train=train)
    if path == "static":
        return _draw_conv(rng, "eval", ("basic", "bottleneck"), train=train, static=True, per_channel=rng.random() < 0.7)
    if path == "layer":
        return _draw_encoder(rng, rng.choice(("step", "eval")), 1, 8192, train=train)
    if path == "stack":
        return _draw_encoder(rng, rng.choice(("step", "eval")), rng.choice((2, 3, 4, 6)), 16384, train=train)
    if path == "metric":
        b = rng.choice((32, 64, 128, _log(rng, 4, 128)))
        d = _log(rng, 1000, 400_000)
        return dict(path="metric", batch=b, features=d if rng.random() < 0.3 else d // 8 * 8, train=train,
                    ref=rng.choice(("f32", "f32", "bf16")))
    if path == "snapshot":
        more = dict(layers=rng.choice((1, 2, 4, 6)), weights=rng.choice(("f32", "bf16")), per_channel=rng.random() < 0.5)
        if rng.random() < 0.5:
            hidden = 64 * rng.choice((4, 8, 12, 16))
            return dict(path="snapshot", kind="encoder", hidden=hidden, ffn=4 * hidden, **more)
        c = rng.choice((16, 64, 256, 512, _log(rng, 16, 512)))
        return dict(path="snapshot", kind="bottleneck", c_in=4 * c, c_mid=c, **more)
    if path == "float":
        if rng.random() < 0.5:
            return _draw_encoder(rng, "forward", 1, 6144, precision=rng.choice(("f16", "f16", "f32")))
        return _draw_conv(rng, "forward", ("basic", "bottleneck"), precision=rng.choice(("f16", "f16", "f32")))
    if path == "affine":
        if rng.random() < 0.3:
            return _draw_encoder(rng, "forward", 1, 8192, precision="affine")
        return _draw_conv(rng, "forward", ("basic", "bottleneck"), precision="affine")
    rows = rng.choice(("f32", "bf16"))
    return dict(path="cache", batch=_log(rng, 8, 128), features=_log(rng, 2000, 250_000) // 8 * 8 + rng.choice((0, 0, 0, 1)),
                window=rng.choice((2, 5, 5)), rows=rows)


# ---- inputs -----------------------------------------------------------------------------------

def _type(name):
    return {"f32": torch.float32, "bf16": torch.bfloat16}[name]


def _shapes(c):
    """Weight shapes of one layer module (or of all its layers), in forward order."""
    if c["kind"] == "fc":
        return [(c["c_out"], c["c_in"])]
    if c["kind"] == "basic":
        return [(c["c_in"], c["c_in"], 3, 3)] * 2
    if c["kind"] == "bottleneck":
        i, m = c["c_in"], c["c_mid"]
        return [(m, i, 1, 1), (m, m, 3, 3), (i, m, 1, 1)] * c.get("layers", 1)
    h, f = c["hidden"], c["ffn"]
    return [(3 * h, h), (h, h), (f, h), (h, f)] * c["layers"]


def _weights(c, randn):
    out = []
    for s in _shapes(c):
        fan_in = math.prod(s[1:])
        var = 2.0 / (s[0] + fan_in) if c["kind"] == "encoder" else (1.0 if c["kind"] == "fc" else 2.0) / fan_in
        out.append(randn(*s) * math.sqrt(var))
    return out


def _conv3x3(x, w):
    """3x3 convolution, padding 1, of NHWC x with [out, in, 3, 3] weights, as nine products."""
    h, wd = x.shape[1], x.shape[2]
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    return sum(p[:, i:i + h, j:j + wd] @ w[:, :, i, j].t() for i in range(3) for j in range(3))


def _train_activations(c, x, weights, biases):
    """A_T of every layer ([batch, D], fp32) and the inputs of the linear layers of a convolution module."""
    b = c["batch"]
    if c["kind"] == "fc":
        return [torch.relu(x @ weights[0].t())], [x]
    if c["kind"] == "basic":
        x = x.permute(0, 2, 3, 1).contiguous()
        h = torch.relu(_conv3x3(x, weights[0]) + biases[0])
        y = torch.relu(_conv3x3(h, weights[1]) + biases[1] + x)
        return [y.reshape(b, -1)], [x, h]
    if c["kind"] == "bottleneck":
        x = x.permute(0, 2, 3, 1).contiguous()
        h1 = torch.relu(x @ weights[0].flatten(1).t() + biases[0])
        h2 = torch.relu(_conv3x3(h1, weights[1]) + biases[1])
        y = torch.relu(h2 @ weights[2].flatten(1).t() + biases[2] + x)
        return [y.reshape(b, -1)], [x, h1, h2]
    outs, hidden, heads = [], c["hidden"], c["heads"]
    split = lambda z: z.reshape(b, c["seq"], heads, hidden // heads).permute(0, 2, 1, 3).contiguous()  # noqa: E731
    norm = lambda z: torch.nn.functional.layer_norm(z, (hidden,), eps=1e-12)  # noqa: E731
    for l in range(c["layers"]):
        wq, wo, w1, w2 = weights[4 * l:4 * l + 4]
        q, k, v = (split(z) for z in (x @ wq.t()).split(hidden, dim=-1))
        att = torch.softmax(q @ k.transpose(-1, -2).contiguous() / math.sqrt(hidden // heads), dim=-1)
        x = norm(x + (att @ v).permute(0, 2, 1, 3).reshape(b, c["seq"], hidden) @ wo.t())
        x = norm(x + torch.nn.functional.gelu(x @ w1.t()) @ w2.t())
        outs.append(x.reshape(b, -1))
    return outs, []


def _dims(c):
    if c["kind"] == "encoder":
        return dict(batch=c["batch"], seq=c["seq"], hidden=c["hidden"], heads=c["heads"], ffn=c["ffn"],
                    n_layers=c["layers"], ln_eps=1e-12)
    if c["kind"] == "fc":
        return dict(batch=c["batch"], c_in=c["c_in"], c_out=c["c_out"])
    return dict(batch=c["batch"], c_in=c["c_in"], c_mid=c["c_mid"], c_out=c["c_in"], height=c["height"], width=c["width"],
                has_residual=1)


def _kind(c):
    if c["kind"] == "encoder":
        return eg.BERT_LAYER if c["layers"] == 1 else eg.BERT_STACK
    return KINDS[c["kind"]]


def _module(c, randn):
    """Mini-batch, snapshot weights, biases of one layer module."""
    if c["kind"] == "fc":
        x = randn(c["batch"], c["c_in"])
    elif c["kind"] == "encoder":
        x = randn(c["batch"], c["seq"], c["hidden"])
    else:
        x = randn(c["batch"], c["c_in"], c["height"], c["width"])
        if c["kind"] == "bottleneck":
            x = x.abs()
    w = _weights(c, randn)
    conv = c["kind"] in ("basic", "bottleneck")
    return x, w, [randn(t.shape[0]) * 0.1 if conv else None for t in w]


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    randn = lambda *s: torch.randn(*s, generator=gen, device=DEVICE)  # noqa: E731
    path = case["path"]
    if path == "metric":
        b, d = case["batch"], case["features"]
        a_r = 0.5 * randn(1, d) + randn(b, d)
        a_t = a_r + 0.02 * randn(b, d)
        return dict(path=path, a_t=a_t.to(_type(case["train"])), a_r=a_r.to(_type(case["ref"])),
                    p=torch.empty(1, device=DEVICE), ws=eg.workspace(eg.plasticity_workspace_bytes(b, d), DEVICE))
    if path == "snapshot":
        w = [t.to(_type(case["weights"])) for t in _weights(case, randn)]
        return dict(path=path, w=w, per_channel=case["per_channel"],
                    ws=eg.workspace(eg.quantize_weights_workspace_bytes(len(w)), DEVICE))
    if path == "cache":
        b, d, dt = case["batch"], case["features"], _type(case["rows"])
        cache = eg.ActivationCache(case["window"], b, d, dt, DEVICE)
        ids = torch.randperm(50_000, generator=gen, device=DEVICE)[:b * case["window"]].reshape(-1, b)
        for k in range(case["window"]):
            rows = randn(b, d).to(dt)
            cache.put(ids[k].contiguous(), rows)
        # the current mini-batch: the coming one in another order, a few samples that were never put in
        want = ids[-1][torch.randperm(b, generator=gen, device=DEVICE)].clone()
        want[::17] = 50_000 + torch.arange(want[::17].numel(), device=DEVICE)
        return dict(path=path, cache=cache, ids=ids[-1].contiguous(), rows=rows, want=want,
                    out=torch.zeros(b, d, dtype=dt, device=DEVICE), hit=torch.zeros(b, dtype=torch.uint8, device=DEVICE))
    x, w, bias = _module(case, randn)
    if path == "forward":
        if case["precision"] == "affine":
            ref = eg.make_reference(_kind(case), _dims(case), w, bias, act_scheme=eg.ACT_AFFINE)
        else:
            ref = eg.make_float_reference(_kind(case), _dims(case), w, bias, PRECISIONS[case["precision"]])
        layers = case.get("layers", 1)
        a_ref = torch.empty(layers, case["batch"], _features(case), device=DEVICE)
        return dict(path=path, ref=ref, x=x, a_ref=a_ref, ws=eg.workspace(eg.workspace_bytes(ref.desc), DEVICE))
    noise = 0.02 if case["kind"] == "encoder" else 0.01
    wt = [t + noise * t.std() * randn(*t.shape) for t in w]
    a_t, inputs = _train_activations(case, x, wt, bias)
    a_t = [t.to(_type(case["train"])).contiguous() for t in a_t]
    scales = torch.stack([t.abs().max() / 127 for t in inputs]) if case.get("static") else None
    ev = PlasticityEvaluator(_kind(case), _dims(case), w, bias, device=DEVICE, act_scales=scales,
                             per_channel=case.get("per_channel", False))
    ev.quantize_weights()
    return dict(path=path, ev=ev, x=x, a_t=a_t)


def run(state):
    path = state["path"]
    if path == "step":
        ev = state["ev"]
        p = ev.step(state["x"], state["a_t"])
        # the scores and the refreshed reference model (of a deep stack the codes alone: its scales are many single values)
        return [p] + ev.w_q + (ev.scales if len(ev.scales) <= 24 else [])
    if path == "eval":
        return state["ev"].evaluate(state["x"], state["a_t"])
    if path == "forward":
        return eg.ref_forward(state["ref"], state["x"], state["a_ref"], state["ws"])
    if path == "metric":
        return eg.plasticity(state["a_t"], state["a_r"], p_out=state["p"], ws=state["ws"])
    if path == "snapshot":
        return eg.quantize_weights(state["w"], ws=state["ws"], per_channel=state["per_channel"])
    state["cache"].put(state["ids"], state["rows"])
    return [state["out"], state["cache"].get(state["want"], state["out"], state["hit"])]


# ---- what a pass cannot do without ------------------------------------------------------------

def _features(c):
    """Features per sample of the hooked activation."""
    if c["kind"] == "fc":
        return c["c_out"]
    return c["seq"] * c["hidden"] if c["kind"] == "encoder" else c["height"] * c["width"] * c["c_in"]


def _size(name):
    return 2 if name == "bf16" else 4


def _metric_flops(b, d):
    return 2.0 * b * (b + 1) * d        # two symmetric b x b Gram matrices


def work(case):
    path = case["path"]
    if path == "metric":
        b, d = case["batch"], case["features"]
        return {"bytes": b * d * (_size(case["train"]) + _size(case["ref"])) + 4, "flops": _metric_flops(b, d)}
    if path == "cache":
        b, row = case["batch"], case["features"] * _size(case["rows"])
        got = b - len(range(0, b, 17))
        return {"bytes": 2 * b * row + 2 * got * row + b * 17, "flops": 0}
    shapes = _shapes(case)
    values = sum(math.prod(s) for s in shapes)
    if path == "snapshot":
        scales = sum(s[0] for s in shapes) if case["per_channel"] else len(shapes)
        return {"bytes": values * (_size(case["weights"]) + 1) + 4 * scales, "flops": 0}
    b, layers = case["batch"], case.get("layers", 1)
    rows, x = b, b * case.get("c_in", 0)
    if case["kind"] == "encoder":
        rows = b * case["seq"]
        x = rows * case["hidden"]
    elif case["kind"] != "fc":
        rows = b * case["height"] * case["width"]
        x = rows * case["c_in"]
    flops = 2.0 * rows * values
    if case["kind"] == "encoder":
        flops += layers * 4.0 * rows * case["seq"] * case["hidden"]
    d = _features(case)
    code = {"f16": 2, "f32": 4}.get(case.get("precision"), 1)
    nbytes = 4 * x + code * values
    if path == "forward":
        return {"bytes": nbytes + 4 * layers * b * d, "flops": flops}
    nbytes += layers * (b * d * _size(case["train"]) + 4)
    if path == "step":
        nbytes += 4 * values
    return {"bytes": nbytes, "flops": flops + layers * _metric_flops(b, d)}


def tolerance(case):
    path = case["path"]
    if path in ("snapshot", "cache"):
        return "exact"
    if path == "forward":
        # float16: a layer input within the rounding of a 32-bit sum of a float16 boundary may round to the other side
        # (2^-11 of the value each, a small share of them); affine codes and float32: 32-bit results
        return {"rel": 1e-3 if case["precision"] == "f16" else 1e-5, "max": 1e-2 if case["precision"] == "f16" else 1e-4}
    # int8 codes and scales are whole numbers and single IEEE operations (no share of them may differ); scores are
    # 32-bit sums, those of an encoder over activations that pass through exp, erf and square roots as well
    return {"rel": 1e-4 if case.get("kind") == "encoder" else 1e-5}
