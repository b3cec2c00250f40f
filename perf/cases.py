"""The work a user of the library has it do, as cases that can be timed and checked.

A case names a model, an input size, a batch, the layer the pass starts from
and the layer it ends at.  ``run`` is one call of the library's public entry
points: ``hapi_extract`` (from the images to a split, the storage side) or
``hapi_extract_range`` (from one split to a later one, the compute side).  The
library is forward-only: the two directions of its path are the half in front
of a split and the half behind it.

``exact`` is the same pass in float64 by plain torch: convolutions as one
matrix product per kernel tap over channel-first images, written from the
models' definitions.
"""
from __future__ import annotations

import math

import torch

import paper_2210_08650_amd as H
from paper_2210_08650_amd import models

# Models, and the deepest layer a case ends at (the frozen part the
# benchmark workloads extract; ResNet-50's pooled features are layer 19).
_SIDES = {"alexnet": (160, 192, 224, 256), "resnet18": (160, 192, 224, 256), "resnet50": (160, 192, 224, 256),
          "vgg16": (160, 192, 224), "densenet121": (160, 192, 224, 256), "vit_b16": (160, 176, 192, 224, 240)}
_LAST = {"alexnet": 8, "resnet18": 11, "resnet50": 19, "vgg16": 18, "densenet121": 13, "vit_b16": 15}
_MAX_BATCH = {"alexnet": 256, "resnet18": 256, "resnet50": 256, "vgg16": 128, "densenet121": 256, "vit_b16": 160}


def _case(name, model, batch, end, start=0, dtype="bf16", side=224, chunk=0):
    c = dict(model=model, dtype=dtype, batch=batch, start=start, end=end, side=side, chunk=chunk)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: four images through the fp32 model.  Twelve short
        # launches, so latency counts.
        _case("alexnet_f32_b4", "alexnet", 4, 8, dtype="f32"),
        # One request of 128 images (the size a storage request has) to the
        # same model: fp32 throughput.
        _case("alexnet_f32_b128", "alexnet", 128, 8, dtype="f32"),
        # The ordinary batch of the small residual network, split after its
        # third stage.
        _case("resnet18_b64", "resnet18", 64, 8),
        # A small storage batch of the benchmark model: some 50 launches of a
        # few microseconds each.
        _case("resnet50_b8", "resnet50", 8, 18),
        # The benchmark's own step.
        _case("resnet50_b256", "resnet50", 256, 18),
        # The compute side of a split: a ragged last batch resumed after stage
        # 2 and taken through the last block.
        _case("resnet50_resume_b37", "resnet50", 37, 18, start=9),
        # The heaviest workload, to its last pooling: long 3x3 convolutions.
        _case("vgg16_b128", "vgg16", 128, 18),
        # An early split (after the third pooling) of a ragged batch: large
        # images, few channels.
        _case("vgg16_pool3_b37", "vgg16", 37, 10),
        # The transformer to its eighth block.
        _case("vit_b16_b128", "vit_b16", 128, 10),
        # One encoder block of a part batch, between two splits.
        _case("vit_b16_block_b48", "vit_b16", 48, 7, start=6),
        # Channel concatenation, at the full batch ...
        _case("densenet121_b256", "densenet121", 256, 12),
        # ... and at a storage batch of 16, to the end of the second block.
        _case("densenet121_b16", "densenet121", 16, 5),
    ]


def draw(rng):
    """Another call of the same kinds: any model, side and batch up to the
    listed cases' cost, any split, some resumed from an earlier split, some
    through the storage batch of 16 or 25 images, ResNet-18 in fp32 too."""
    model = rng.choice(sorted(_LAST))
    side = rng.choice(_SIDES[model])
    batch = max(1, int(round(math.exp(rng.uniform(0.0, math.log(_MAX_BATCH[model]))))))
    last = _LAST[model]
    first = {"alexnet": 2, "vgg16": 3, "vit_b16": 3}.get(model, 2)
    end = rng.randint(first, last)
    start = rng.randint(0, end - 1) if rng.random() < 0.3 else 0
    dtype = "f32" if model == "alexnet" or (model == "resnet18" and rng.random() < 0.2) else "bf16"
    chunk = rng.choice((16, 25)) if batch > 25 and rng.random() < 0.15 else 0
    case = _case(None, model, batch, end, start, dtype, side, chunk)
    top = work(listed()[6])["flops"] / (16 if dtype == "f32" else 1)
    while case["batch"] > 1 and work(case)["flops"] > top:
        case["batch"] = case["batch"] * 3 // 4
    return case


def _layers(case):
    return models.FACTORIES[case["model"]]()


def _tdtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


# ------------------------------------------------------------------- inputs

def _generator(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 64 + what)
    return g


def _draw_param(shape, kind, g):
    dev = dict(device="cuda", dtype=torch.float32)
    if kind == "he":  # Kaiming-normal
        fan_in = math.prod(shape[1:])
        return torch.randn(shape, generator=g, **dev) * math.sqrt(2.0 / fan_in)
    if kind in ("bias", "bn_beta", "bn_mean"):
        return torch.rand(shape, generator=g, **dev) * 0.2 - 0.1
    if kind in ("bn_gamma", "bn_var"):
        return torch.rand(shape, generator=g, **dev) + 0.5
    t = torch.randn(shape, generator=g, **dev).clamp_(-2.0, 2.0).mul_(0.02)
    return t.add_(1.0) if kind == "ln_gamma" else t


def _params(case, seed):
    """The raw weights, tensor by tensor in the library's order: stand-ins for
    pre-trained ones."""
    g = _generator(seed, 1)
    return [_draw_param(tuple(s), k, g) for s, k in models.raw_manifest(_layers(case), (3, case["side"], case["side"]))]


def _input(case, seed):
    """The images, or the tensor of the layer the pass resumes after: N(0, 1)
    tokens and normalised images, and behind a ReLU its positive part."""
    shape = (case["batch"],) + _shapes(case)[case["start"]]
    x = torch.randn(shape, generator=_generator(seed, 2), device="cuda", dtype=torch.float32)
    if case["start"] > 0 and case["model"] != "vit_b16":
        x = x.clamp_(min=0.0)
    return x.to(_tdtype(case))


def _desc(case, **kw):
    return H.Desc(_layers(case), H.HAPI_F32 if case["dtype"] == "f32" else H.HAPI_BF16,
                  in_shape=(3, case["side"], case["side"]), chunk=case["chunk"], **kw)


def prepare(case, seed):
    """What a serving program holds: packed weights, workspace, the input and
    the output buffer."""
    d = _desc(case, stream=torch.cuda.current_stream())
    raw = torch.cat([p.reshape(-1) for p in _params(case, seed)])
    packed = torch.empty(H.hapi_packed_weight_bytes(d), dtype=torch.uint8, device="cuda")
    H.hapi_pack_weights(d, raw, packed)
    need = H.hapi_workspace_bytes(d, case["batch"], case["end"])
    d.set(workspace=torch.empty(need, dtype=torch.uint8, device="cuda"), workspace_bytes=need)
    out = torch.empty((case["batch"],) + H.hapi_layer_shape(d, case["end"]), dtype=_tdtype(case), device="cuda")
    return dict(desc=d, weights=packed, x=_input(case, seed), out=out, batch=case["batch"], start=case["start"],
                end=case["end"])


def run(state):
    s = state
    if s["start"] == 0:
        H.hapi_extract(s["desc"], s["weights"], s["x"], s["batch"], s["end"], s["out"])
    else:
        H.hapi_extract_range(s["desc"], s["weights"], s["x"], s["batch"], s["start"], s["end"], s["out"])
    return s["out"]


# --------------------------------------------------------- shapes and counts

def _walk(case):
    """Per layer: (output shape, multiply-adds per image, weight values)."""
    c, h, w = 3, case["side"], case["side"]
    tok = None
    rows = []

    def conv(cin, cout, k, ho, wo):
        return cout * cin * k * k * ho * wo, cout * cin * k * k

    for L in _layers(case):
        kind, mac, par = L["kind"], 0, 0
        if kind in (H.HAPI_CONV, H.HAPI_PREACT_CONV):
            k, s, p = L["k"], L.get("stride", 1), L.get("pad", 0)
            h, w, c = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1, L["cout"]
            mac, par = conv(L["cin"], c, k, h, w)
        elif kind in (H.HAPI_MAXPOOL, H.HAPI_AVGPOOL):
            k, s, p = L.get("k", 0), L.get("stride", 1), L.get("pad", 0)
            h, w = ((h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1) if k else (1, 1)
        elif kind in (H.HAPI_BASIC_BLOCK, H.HAPI_BOTTLENECK):
            cin, s = L["cin"], L["stride"]
            ho, wo = (h - 1) // s + 1, (w - 1) // s + 1
            if kind == H.HAPI_BASIC_BLOCK:
                c = L["cout"]
                parts = [conv(cin, c, 3, ho, wo), conv(c, c, 3, ho, wo)]
            else:
                wd, c = L["width"], 4 * L["width"]
                parts = [conv(cin, wd, 1, h, w), conv(wd, wd, 3, ho, wo), conv(wd, c, 1, ho, wo)]
            if s != 1 or cin != c:
                parts.append(conv(cin, c, 1, ho, wo))
            mac, par = sum(a for a, _ in parts), sum(b for _, b in parts)
            h, w = ho, wo
        elif kind == H.HAPI_PATCH_EMBED:
            c, h, w = L["cout"], h // L["k"], w // L["k"]
            mac, par = conv(L["cin"], c, L["k"], h, w)
        elif kind == H.HAPI_TOKENS:
            tok, par = 1 + h * w, (2 + h * w) * c
        elif kind == H.HAPI_VIT_BLOCK:
            D, F = L["cout"], L["mlp_dim"]
            par = 4 * D * D + 2 * D * F
            mac = tok * par + 2 * tok * tok * D
        elif kind == H.HAPI_DENSE_BLOCK:
            for ch in range(L["cin"], L["cout"], L["width"]):
                for a, b in (conv(ch, L["mlp_dim"], 1, h, w), conv(L["mlp_dim"], L["width"], 3, h, w)):
                    mac, par = mac + a, par + b
            c = L["cout"]
        rows.append(((tok, c) if tok else (c, h, w), mac, par))
    return rows


def _shapes(case):
    return [(3, case["side"], case["side"])] + [r[0] for r in _walk(case)]


def work(case):
    rows, shapes = _walk(case)[case["start"]:case["end"]], _shapes(case)
    size = 4 if case["dtype"] == "f32" else 2
    values = case["batch"] * (math.prod(shapes[case["start"]]) + math.prod(shapes[case["end"]])) + sum(r[2] for r in rows)
    return {"bytes": size * values, "flops": 2 * case["batch"] * sum(r[1] for r in rows)}


# ------------------------------------------------------------------ checking

def tolerance(case):
    # fp32 sums of up to 3456 products in another order: 5e-7 measured against
    # 64 bits.  bf16 (weights, and each layer's output, rounded once): up to
    # 1.1e-2 after the 18 layers of the deepest network, 3e-3 after one block.
    if case["dtype"] == "f32":
        return {"rel": 2e-6}
    return {"rel": 0.03 if case["end"] - case["start"] > 3 else 0.015}


def _conv64(x, weight, stride, pad):
    """x [C, B, H, W], weight [N, C, k, k]: one product per kernel tap."""
    c, b, h, w = x.shape
    n, _, k, _ = weight.shape
    if pad:
        x = torch.nn.functional.pad(x, (pad, pad, pad, pad))
    ho, wo = (h + 2 * pad - k) // stride + 1, (w + 2 * pad - k) // stride + 1
    y = torch.zeros((n, b * ho * wo), dtype=torch.float64, device=x.device)
    if c < 16:  # images: all taps of a few channels in one product
        cols = [x[:, :, i:i + (ho - 1) * stride + 1:stride, j:j + (wo - 1) * stride + 1:stride].reshape(c, -1)
                for i in range(k) for j in range(k)]
        y = weight.permute(0, 2, 3, 1).reshape(n, -1) @ torch.cat(cols)
    else:
        for i in range(k):
            for j in range(k):
                xs = x[:, :, i:i + (ho - 1) * stride + 1:stride, j:j + (wo - 1) * stride + 1:stride].reshape(c, -1)
                y.addmm_(weight[:, :, i, j].contiguous(), xs)
    return y.view(n, b, ho, wo)


def _pool64(x, L):
    k, s, p = L.get("k", 0), L.get("stride", 1), L.get("pad", 0)
    if L["kind"] == H.HAPI_AVGPOOL:
        if k == 0:
            return x.mean(dim=(2, 3), keepdim=True)
        return x.unfold(2, k, s).unfold(3, k, s).mean(dim=(4, 5))
    if p:
        x = torch.nn.functional.pad(x, (p, p, p, p), value=-math.inf)
    return x.unfold(2, k, s).unfold(3, k, s).amax(dim=(4, 5))


def _forward64(layers, take, x, start, end):
    """Layers start + 1 .. end; ``take(n)`` hands out a layer's tensors in order."""
    for i, L in enumerate(layers[:end]):
        kind = L["kind"]
        run_it = i >= start

        def bn(v, t):
            g, b, m, var = (u.view(-1, 1, 1, 1) for u in t)
            return (v - m) * (g / torch.sqrt(var + 1e-5)) + b

        def ln(v, g, b):
            m = v.mean(-1, keepdim=True)
            return (v - m) / torch.sqrt(((v - m) ** 2).mean(-1, keepdim=True) + 1e-6) * g + b

        if kind == H.HAPI_CONV:
            w, = take(1)
            b = take(1)[0] if L.get("has_bias") else None
            t = take(4) if L.get("has_bn") else None
            if run_it:
                x = _conv64(x, w, L.get("stride", 1), L.get("pad", 0))
                x = x + b.view(-1, 1, 1, 1) if b is not None else x
                x = bn(x, t) if t else x
                x = x.clamp(min=0.0) if L.get("relu") else x
        elif kind in (H.HAPI_MAXPOOL, H.HAPI_AVGPOOL):
            x = _pool64(x, L) if run_it else x
        elif kind in (H.HAPI_BASIC_BLOCK, H.HAPI_BOTTLENECK):
            s = L["stride"]
            geo = ((3, s), (3, 1)) if kind == H.HAPI_BASIC_BLOCK else ((1, 1), (3, s), (1, 1))
            cout = L["cout"]
            ts = [take(5) for _ in geo]
            sc = take(5) if s != 1 or L["cin"] != cout else None
            if run_it:
                y = x
                for n, ((k, st), t) in enumerate(zip(geo, ts)):
                    y = bn(_conv64(y, t[0], st, k // 2), t[1:])
                    y = y.clamp(min=0.0) if n + 1 < len(geo) else y
                x = (y + (bn(_conv64(x, sc[0], s, 0), sc[1:]) if sc else x)).clamp(min=0.0)
        elif kind == H.HAPI_PATCH_EMBED:
            w, b = take(2)
            if run_it:
                x = _conv64(x, w, L["k"], 0) + b.view(-1, 1, 1, 1)
        elif kind == H.HAPI_TOKENS:
            cls, pos = take(2)
            if run_it:
                p = x.permute(1, 2, 3, 0).reshape(x.shape[1], -1, x.shape[0])
                x = torch.cat([cls.expand(p.shape[0], 1, -1), p], 1) + pos
        elif kind == H.HAPI_VIT_BLOCK:
            g1, b1, wi, bi, wo, bo, g2, b2, w1, c1, w2, c2 = take(12)
            if run_it:
                B, T, D = x.shape
                h = L["heads"]
                q, k, v = (ln(x, g1, b1) @ wi.T + bi).view(B, T, 3, h, D // h).permute(2, 0, 3, 1, 4)
                a = torch.softmax(q @ k.transpose(-1, -2).contiguous() / math.sqrt(D // h), -1) @ v.contiguous()
                x = x + a.transpose(1, 2).reshape(B, T, D) @ wo.T + bo
                f = ln(x, g2, b2) @ w1.T + c1
                x = x + (0.5 * f * (1.0 + torch.erf(f / math.sqrt(2.0)))) @ w2.T + c2
        elif kind == H.HAPI_LAYERNORM:
            g, b = take(2)
            x = ln(x, g, b) if run_it else x
        elif kind == H.HAPI_PREACT_CONV:
            t = take(5)
            if run_it:
                x = _conv64(bn(x, t[:4]).clamp(min=0.0), t[4], L.get("stride", 1), L.get("pad", 0))
        elif kind == H.HAPI_BATCHNORM:
            t = take(4)
            if run_it:
                x = bn(x, t)
                x = x.clamp(min=0.0) if L.get("relu") else x
        elif kind == H.HAPI_DENSE_BLOCK:
            for _ in range(L["cin"], L["cout"], L["width"]):
                t = take(10)
                if run_it:
                    y = _conv64(bn(x, t[:4]).clamp(min=0.0), t[4], 1, 0)
                    y = _conv64(bn(y, t[5:9]).clamp(min=0.0), t[9], 1, 1)
                    x = torch.cat([x, y], 0)
        else:
            raise ValueError(f"unknown layer kind {kind}")
    return x


def exact(case, seed):
    params = [p.double() for p in _params(case, seed)]
    x = _input(case, seed)
    layers = _layers(case)
    parts = []
    step = 8  # images at once
    for b0 in range(0, case["batch"], step):
        xb = x[b0:b0 + step].double()
        if xb.dim() == 4:  # channel first: a convolution is a product over [C, B H W]
            xb = xb.transpose(0, 1).contiguous()
        it = iter(params)
        y = _forward64(layers, lambda n: [next(it) for _ in range(n)], xb, case["start"], case["end"])
        parts.append(y.transpose(0, 1) if y.dim() == 4 else y)
    return torch.cat(parts).contiguous()
