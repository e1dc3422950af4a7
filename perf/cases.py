"""Timed cases of the derived operators, called as a program calls the Python binding.

The listed cases are layers of the networks that the operators stand for: a ResNet-18
block's 3x3 convolution at batch 1 and 16, a strided downsampling convolution, a DCGAN
generator's transposed convolution, a CSRNet back-end dilated convolution (fused and in
the default two-stage form), an SRCNN 5x5 convolution, fp32 convolutions of both ends of
the size range, and Longformer's dilated sliding-window attention (fused, masked on a
ragged length, and staged with its scores returned).

A case is a dict of plain values:
  op      "conv" (derived_conv2d), "dilated" (derived_dilated_conv2d),
          "convT" (derived_conv_transpose2d) or "band" (banded_bmm)
  conv    n, h, w, c, k, r, s, stride, pad, dil, out_pad; dtype of x and wt, out dtype;
          fuse (the fused GEMM + eOperator expression); y16 (two-stage scope in bf16);
          tail: "" | "bias_relu" | "residual" (bias + residual + ReLU)
  band    b, l, width (half-window w), dil, scale, mask, staged (scores returned), out dtype
"""
import math

import torch

import paper_2208_02025_amd as ol

DEV = "cuda"
_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
_SIZE = {"f32": 4, "bf16": 2}


def _conv(name, op, n, h, w, c, k, r, s, stride=1, pad=0, dil=1, out_pad=0, dtype="bf16",
          out="f32", fuse=True, y16=False, tail=""):
    d = dict(op=op, n=n, h=h, w=w, c=c, k=k, r=r, s=s, stride=stride, pad=pad, dil=dil,
             out_pad=out_pad, dtype=dtype, out=out, fuse=fuse, y16=y16, tail=tail)
    return dict(d, name=name) if name else d


def _band(name, b, l, width, dil, scale=1.0, mask=False, staged=False, out="f32"):
    d = dict(op="band", b=b, l=l, width=width, dil=dil, scale=scale, mask=mask, staged=staged,
             out=out)
    return dict(d, name=name) if name else d


def listed():
    return [
        # the smallest call: one image of a small fp32 layer, where launches and host time count
        _conv("tiny_conv3x3_f32", "conv", 1, 14, 14, 16, 16, 3, 3, 1, 1, dtype="f32", fuse=False),
        # an ordinary fp32 layer (ResNet stage 1, batch 8): fp32 always takes the two stages
        _conv("resnet1_conv3x3_f32", "conv", 8, 56, 56, 64, 64, 3, 3, 1, 1, dtype="f32",
              fuse=False),
        # batch-1 inference of the last ResNet-18 stage, with its bias and ReLU
        _conv("resnet4_conv3x3_b1", "conv", 1, 7, 7, 512, 512, 3, 3, 1, 1, out="bf16",
              tail="bias_relu"),
        # a residual block's second convolution at batch 16, with the block's tail
        _conv("resnet3_conv3x3_b16", "conv", 16, 14, 14, 256, 256, 3, 3, 1, 1, out="bf16",
              tail="residual"),
        # a downsampling convolution on odd image sizes and odd channel counts
        _conv("down_conv3x3_s2_odd", "conv", 5, 57, 43, 128, 200, 3, 3, 2, 1, out="bf16",
              tail="bias_relu"),
        # a DCGAN generator layer
        _conv("dcgan_convT4x4_b16", "convT", 16, 8, 8, 512, 256, 4, 4, 2, 1),
        # CSRNet's back end on a 768x1024 image: the fused expression, and the two-stage
        # form that the operator evaluates by default
        _conv("csrnet_dilconv_fused", "dilated", 1, 96, 128, 512, 512, 3, 3, 1, 2, 2),
        _conv("csrnet_dilconv_staged", "dilated", 1, 96, 128, 512, 512, 3, 3, 1, 2, 2, fuse=False),
        # SRCNN's 5x5 layer on a 512x512 image
        _conv("srcnn_conv5x5", "conv", 1, 512, 512, 64, 32, 5, 5, 1, 2, out="bf16",
              tail="bias_relu"),
        # Longformer-base dilated attention over 8 sequences of 12 heads
        _band("longformer_band", 96, 4096, 256, 2),
        # one sequence of 12 heads of a ragged length, out-of-range keys masked
        _band("band_masked_ragged", 12, 3001, 200, 3, 0.125, mask=True, out="bf16"),
        # one sequence of 12 heads with the scores returned (the staged path)
        _band("band_staged_scores", 12, 4096, 256, 2, 0.125, staged=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges, drawn again while it would cost more than the
    largest listed ones."""
    while True:
        case = _draw(rng)
        if _affordable(case):
            return case


def _affordable(case):
    if case["op"] == "band":
        entries = case["b"] * case["l"] * (2 * case["width"] + 1)
        return entries <= (12 if case["staged"] else 96) * 4096 * 513
    ho, wo = _conv_out_hw(case)
    if ho < 1 or wo < 1:
        return False
    pix = case["n"] * case["h"] * case["w"]
    if case["op"] == "conv" and case["fuse"]:
        pix = case["n"] * ho * wo
    taps = case["r"] * case["s"]
    flops = 2 * pix * taps * max(case["k"], 64) * case["c"]
    if case["fuse"]:
        return flops <= 40e9
    scope = pix * taps * case["k"]
    return scope <= 40e6 and flops <= (3e9 if case["dtype"] == "f32" else 20e9)


def _draw(rng):
    kind = rng.choice(["conv", "conv", "f32", "channels", "convT", "dilated", "band", "band"])
    if kind == "band":
        staged = rng.random() < 0.3
        b = _log(rng, 1, 16 if staged else 96)
        return _band("", b, _log(rng, 64, 4096), _log(rng, 4, 256), rng.randint(1, 4),
                     rng.choice([1.0, 0.125]), rng.random() < 0.5, staged,
                     rng.choice(["f32", "bf16"]))
    tail = rng.choice(["", "bias_relu", "residual"])
    out = rng.choice(["f32", "bf16"])
    if kind == "f32":
        k = rng.choice([1, 3, 5])
        return _conv("", "conv", rng.randint(1, 8), _log(rng, 7, 64), _log(rng, 7, 64),
                     _log(rng, 3, 128), _log(rng, 8, 128), k, k, rng.randint(1, 2), k // 2,
                     dtype="f32", fuse=False, tail=tail)
    if kind == "channels":   # bf16 channel counts outside the fused expression
        k = rng.choice([3, 5])
        return _conv("", "conv", rng.randint(1, 4), _log(rng, 7, 128), _log(rng, 7, 128),
                     8 * rng.choice([1, 2, 3, 4, 5, 6, 9, 12]), _log(rng, 3, 128), k, k,
                     rng.randint(1, 2), k // 2, out=out, fuse=False, y16=rng.random() < 0.3,
                     tail=tail)
    fuse = rng.random() < 0.75
    c = 64 * rng.choice([1, 2, 3, 4, 8])
    if kind == "convT":
        kp = rng.choice([(4, 2, 1, 0), (3, 2, 1, 1), (2, 2, 0, 0), (5, 2, 2, 1)])
        return _conv("", "convT", rng.choice([1, 16]), _log(rng, 2, 32), _log(rng, 2, 32), c,
                     rng.choice([3, 50, 64, 128, 256]), kp[0], kp[0], kp[1], kp[2], 1, kp[3],
                     out=out, fuse=fuse, tail=tail)
    if kind == "dilated":
        d = rng.randint(2, 4)
        return _conv("", "dilated", rng.randint(1, 2), _log(rng, 14, 96), _log(rng, 14, 96), c,
                     rng.choice([64, 96, 128, 200, 256, 512]), 3, 3, 1, d, d, out=out, fuse=fuse,
                     tail=tail)
    k, stride = rng.choice([(3, 1), (3, 1), (3, 2), (5, 1), (1, 1)])
    h = _log(rng, 7, 112)
    c = c if h < 60 else 64
    return _conv("", "conv", rng.choice([1, 2, 16]) if h < 60 else 1, h, max(4, h + rng.randint(-6, 6)),
                 c, rng.choice([32, 64, 100, 128, 200, 256, 512]) if h < 60 else 64, k, k, stride,
                 k // 2, out=out, fuse=fuse, tail=tail)


# --------------------------------------------------------------------------- states

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _conv_out_hw(case):
    """Output size of the operator (torch's conv2d / conv_transpose2d)."""
    def one(size, ksize):
        if case["op"] == "convT":
            return ((size - 1) * case["stride"] - 2 * case["pad"] + case["dil"] * (ksize - 1) +
                    case["out_pad"] + 1)
        return (size + 2 * case["pad"] - case["dil"] * (ksize - 1) - 1) // case["stride"] + 1
    return one(case["h"], case["r"]), one(case["w"], case["s"])


def prepare(case, seed):
    """Inputs drawn on the GPU: activations after a ReLU (normal in the generator and
    the attention), He-scaled weights, small biases."""
    g = _gen(seed)
    if case["op"] == "band":
        q, k, v = (torch.randn((case["b"], case["l"], 64), generator=g, device=DEV)
                   .to(torch.bfloat16) for _ in range(3))
        return {"case": case, "q": q, "k": k, "v": v}
    dt, c, k = _DT[case["dtype"]], case["c"], case["k"]
    x = torch.randn((case["n"], case["h"], case["w"], c), generator=g, device=DEV)
    if case["op"] != "convT":
        x = torch.relu(x)
    std = math.sqrt(2.0 / (case["r"] * case["s"] * c))
    wt = torch.randn((case["r"], case["s"], k, c), generator=g, device=DEV) * std
    st = {"case": case, "x": x.to(dt), "wt": wt.to(dt), "bias": None, "residual": None}
    if case["tail"]:
        st["bias"] = torch.randn((k,), generator=g, device=DEV) * 0.1
    if case["tail"] == "residual":
        ho, wo = _conv_out_hw(case)
        res = torch.relu(torch.randn((case["n"], ho, wo, k), generator=g, device=DEV))
        st["residual"] = res.to(_DT[case["out"]])
    return st


def run(state):
    case = state["case"]
    out = _DT[case["out"]]
    if case["op"] == "band":
        return ol.banded_bmm(state["q"], state["k"], state["v"], case["width"], case["dil"],
                             case["scale"], mask_invalid=case["mask"], return_s=case["staged"],
                             out_dtype=out)
    tail = dict(bias=state["bias"], residual=state["residual"], relu=bool(case["tail"]))
    if case["op"] == "conv":
        return ol.derived_conv2d(state["x"], state["wt"], case["stride"], case["pad"],
                                 out_dtype=out, y_bf16=case["y16"], fuse=case["fuse"], **tail)
    if case["op"] == "dilated":
        return ol.derived_dilated_conv2d(state["x"], state["wt"], case["stride"], case["pad"],
                                         case["dil"], out_dtype=out, y_bf16=case["y16"],
                                         fuse=case["fuse"], **tail)
    return ol.derived_conv_transpose2d(state["x"], state["wt"], case["stride"], case["pad"],
                                       case["out_pad"], case["dil"], out_dtype=out,
                                       y_bf16=case["y16"], fuse=case["fuse"], **tail)


# ----------------------------------------------------------------- work and accuracy

def _axis_pairs(case, size, ksize, osize):
    """(output, tap) pairs along one axis whose input lies in the image."""
    n = 0
    for o in range(osize):
        for t in range(ksize):
            if case["op"] == "convT":
                i, rem = divmod(o + case["pad"] - t * case["dil"], case["stride"])
                n += rem == 0 and 0 <= i < size
            else:
                n += 0 <= o * case["stride"] - case["pad"] + t * case["dil"] < size
    return n


def work(case):
    if case["op"] == "band":
        b, l, nb = case["b"], case["l"], 2 * case["width"] + 1
        byts = b * l * 64 * (3 * 2 + _SIZE[case["out"]])
        if case["staged"]:
            byts += b * l * nb * 4
        # band entries whose key exists (the others are known to score zero)
        entries = sum(max(0, l - abs(j) * case["dil"])
                      for j in range(-case["width"], case["width"] + 1))
        return {"bytes": byts, "flops": 4 * b * entries * 64}
    ho, wo = _conv_out_hw(case)
    n, c, k = case["n"], case["c"], case["k"]
    el, oel = _SIZE[case["dtype"]], _SIZE[case["out"]]
    byts = n * case["h"] * case["w"] * c * el + case["r"] * case["s"] * k * c * el
    byts += n * ho * wo * k * oel * (2 if case["tail"] == "residual" else 1)
    pairs = (_axis_pairs(case, case["h"], case["r"], ho) *
             _axis_pairs(case, case["w"], case["s"], wo))
    return {"bytes": byts, "flops": 2 * n * pairs * c * k}


def tolerance(case):
    """About four times the error against 64 bits measured over the listed cases and 24
    drawn ones: 2.3e-7 (largest 2.7e-6) for fp32 sums of exact products, 1.7e-3 (3.9e-3)
    where the result or a partial of it is rounded to bf16, 1.7e-3 (1.4e-2) for the
    attention's bf16 probabilities and 2.4e-3 (1.2e-2) with a bf16 result on top."""
    if case["op"] == "band":
        return {"rel": 1e-2 if case["out"] == "bf16" else 7e-3, "max": 0.06}
    if case["out"] == "bf16" or case["y16"]:
        return {"rel": 7e-3, "max": 0.02}
    return {"rel": 1e-6, "max": 1.2e-5}


def _exact_conv(case, seed):
    st = prepare(case, seed)
    x, wt = st["x"].double(), st["wt"].double()
    n, h, w, c, k = (case[key] for key in "nhwck")
    ho, wo = _conv_out_hw(case)
    sd, pd, dl = case["stride"], case["pad"], case["dil"]

    def axis(size, osize, t):
        """Outputs along one axis that tap t lands on, and the inputs they read."""
        o = torch.arange(osize, device=DEV)
        if case["op"] == "convT":
            i = o + pd - t * dl
            ok = (i >= 0) & (i % sd == 0) & (torch.div(i, sd, rounding_mode="floor") < size)
            return o[ok], torch.div(i[ok], sd, rounding_mode="floor")
        i = o * sd - pd + t * dl
        ok = (i >= 0) & (i < size)
        return o[ok], i[ok]

    out = torch.zeros((n, ho, wo, k), dtype=torch.float64, device=DEV)
    for r in range(case["r"]):
        oh, ih = axis(h, ho, r)
        for s in range(case["s"]):
            ow, iw = axis(w, wo, s)
            if len(oh) == 0 or len(ow) == 0:
                continue
            part = x[:, ih][:, :, iw].reshape(-1, c) @ wt[r, s].t().contiguous()
            out[:, oh[:, None], ow[None, :]] += part.reshape(n, len(oh), len(ow), k)
    if st["bias"] is not None:
        out += st["bias"].double()
    if st["residual"] is not None:
        out += st["residual"].double()
    return torch.relu(out) if case["tail"] else out


def _exact_band(case, seed):
    st = prepare(case, seed)
    b, l, w, dil = case["b"], case["l"], case["width"], case["dil"]
    nb, blk = 2 * w + 1, 256
    o = torch.empty((b, l, 64), dtype=torch.float64, device=DEV)
    s_all = torch.empty((b, l, nb), dtype=torch.float64, device=DEV) if case["staged"] else None
    for rho in range(min(dil, l)):
        q, k, v = (st[t][:, rho::dil].double() for t in "qkv")
        lr = q.shape[1]
        pad = torch.zeros((b, w, 64), dtype=torch.float64, device=DEV)
        k, v = torch.cat([pad, k, pad], 1), torch.cat([pad, v, pad], 1)
        for q0 in range(0, lr, blk):
            qn = min(blk, lr - q0)
            keys = slice(q0, q0 + qn + 2 * w)      # padded rows: key of row t is t - w
            sc = torch.bmm(q[:, q0:q0 + qn].contiguous(),
                           k[:, keys].transpose(1, 2).contiguous()) * case["scale"]
            i = torch.arange(qn, device=DEV)[:, None]
            j = torch.arange(qn + 2 * w, device=DEV)[None, :]
            if s_all is not None:
                idx = (i + torch.arange(nb, device=DEV)[None, :]).expand(b, qn, nb)
                rows = torch.arange(rho + q0 * dil, rho + (q0 + qn - 1) * dil + 1, dil, device=DEV)
                s_all[:, rows] = torch.gather(sc, 2, idx)
            ok = (j >= i) & (j <= i + 2 * w)
            if case["mask"]:
                t = q0 + j - w
                ok = ok & (t >= 0) & (t < lr)
            p = torch.softmax(sc.masked_fill(~ok, -math.inf), 2)
            o[:, rho + q0 * dil:rho + (q0 + qn - 1) * dil + 1:dil] = torch.bmm(
                p, v[:, keys].contiguous())
    return (o, s_all) if case["staged"] else o


def exact(case, seed):
    return _exact_band(case, seed) if case["op"] == "band" else _exact_conv(case, seed)
