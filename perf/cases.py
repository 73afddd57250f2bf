"""The calls whose speed this library is measured by: sliding sums, pooling layers and convolution layers, forward and
training, over the sizes, storage types and boundary rules that its users pass.

A case is a dict of plain values; `prepare` makes its inputs on the GPU, `run` makes one pass through the binding's public
functions (outputs allocated by them, as a program that passes no `y=` does), `exact` gives the same outputs in 64 bits
from plain torch.  A training case is a layer's share of one step: its forward call and its adjoints.
"""
import math

import torch
import torch.nn.functional as F

from paper_2305_16513_amd import binding as B

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
OPS = {"add": B.OP_ADD, "max": B.OP_MAX, "min": B.OP_MIN}
MODES = {"mirror": B.SWS_PAD_MIRROR, "periodic": B.SWS_PAD_PERIODIC, "edge": B.SWS_PAD_EDGE, "shrink": B.SWS_PAD_SHRINK}


def slide(rows, length, op, w, dtype="f32", mode="valid"):
    return {"kind": "slide", "rows": rows, "length": length, "op": op, "w": w, "dtype": dtype, "mode": mode}


def pool(n, c, h, w, op, k, s, p, dtype="f32", train=True):
    return {"kind": "pool", "n": n, "c": c, "h": h, "w": w, "op": op, "k": k, "s": s, "p": p, "dtype": dtype, "train": train}


def depthwise(b, c, length, k, d, p, dtype="f32", train=True):
    return {"kind": "depthwise", "b": b, "c": c, "length": length, "k": k, "d": d, "p": p, "dtype": dtype, "train": train}


def dense1d(b, cin, cout, length, k, p, train=True):
    return {"kind": "dense1d", "b": b, "cin": cin, "cout": cout, "length": length, "k": k, "p": p, "train": train}


def dense2d(n, cin, cout, h, w, k, s, p, train=True):
    return {"kind": "dense2d", "n": n, "cin": cin, "cout": cout, "h": h, "w": w, "k": k, "s": s, "p": p, "train": train}


def listed():
    return [
        # A moving average over one series of a million samples: the smallest call, where latency counts.
        dict(slide(1, 1048576, "add", 5), name="mean_one_series"),
        # A sliding maximum over a batch of long multi-channel signals (256 x 128 channels): the largest call.
        dict(slide(32768, 16384, "max", 64), name="max_batch_of_signals"),
        # The same kind of layer on quantised (bfloat16) activations.
        dict(slide(8192, 16384, "add", 64, "bf16"), name="mean_bf16"),
        # Smoothing that keeps the rows' length, with mirrored ends, on rows of no round length.
        dict(slide(3000, 5003, "add", 25, "f32", "mirror"), name="mean_same_size_ragged"),
        # The pooling after an image network's first layer, in training: forward and gradients to the maxima.
        dict(pool(32, 64, 112, 112, "max", 3, 2, 1), name="pool_stem_train"),
        # Global average pooling in front of a classifier, in training: thousands of tiny planes.
        dict(pool(32, 2048, 7, 7, "add", 7, 1, 0), name="pool_head_train"),
        # A depthwise long-kernel layer of a 1-D network, in training: forward and both adjoints.
        dict(depthwise(32, 128, 16384, 31, 1, 15), name="depthwise_train"),
        # A very long dilated kernel over many channels, in inference.
        dict(depthwise(1, 1024, 65536, 51, 8, 0, "f32", False), name="depthwise_dilated"),
        # A dense 1-D layer of 64 channels, in training.
        dict(dense1d(16, 64, 64, 4096, 3, 0), name="dense1d_train"),
        # A 64-channel 3 x 3 layer of a residual network's first stage, in training.
        dict(dense2d(32, 64, 64, 56, 56, 3, 1, 1), name="conv2d_first_stage_train"),
        # A layer that halves the planes between two stages, in training.
        dict(dense2d(32, 128, 128, 56, 56, 3, 2, 1), name="conv2d_down_train"),
        # A late layer: many channels, small planes, in training.
        dict(dense2d(32, 256, 256, 14, 14, 3, 1, 1), name="conv2d_late_train"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng):
    """Channel counts of dense layers: mostly multiples of 32, some multiples of 8, a few of neither."""
    c, r = _log(rng, 16, 512), rng.random()
    return max(32, c // 32 * 32) if r < 0.6 else max(8, c // 8 * 8) if r < 0.85 else c


def draw(rng):
    kind = rng.choice(["slide", "slide", "pool", "depthwise", "dense1d", "dense2d", "dense2d", "dense2d"])
    if kind == "slide":
        length = _log(rng, 200, 1048576)
        rows = max(1, _log(rng, 1048576, 268435456) // length)
        w = min(_log(rng, 2, 512), length // 2)
        op = rng.choice(["add", "add", "max", "min"])
        how = rng.choice(["valid", "valid", "bf16", "f16", "mirror", "edge", "periodic", "shrink"])
        if how in ("bf16", "f16", "valid"):
            return slide(rows, length, op, w, how if how != "valid" else "f32")
        return slide(rows, length, op, w, "f32", how)
    if kind == "pool":
        h, w = _log(rng, 7, 224), _log(rng, 7, 224)
        k, s = rng.choice([(3, 2), (3, 2), (2, 2), (3, 1), (5, 1), (min(h, w, 13), 1)])
        planes = max(32, _log(rng, 1048576, 33554432) // (h * w))
        c = rng.choice([16, 30, 32, 64])
        dtype = rng.choice(["f32", "f32", "f32", "bf16", "f16"])
        return pool(max(1, planes // c), c, h, w, rng.choice(["add", "max"]), k, s, 0 if k == 2 else k // 2, dtype, dtype == "f32")
    if kind == "depthwise":
        length, c = _log(rng, 500, 1048576), rng.choice([1, 16, 45, 64, 128])
        b = max(1, _log(rng, 1048576, 67108864) // (length * c))
        k, d = _log(rng, 3, 63), rng.choice([1, 1, 1, 2, 4, 8])
        d = d if (k - 1) * d < length // 2 else 1
        dtype = "f32" if d > 1 else rng.choice(["f32", "f32", "f32", "bf16", "f16"])
        return depthwise(b, c, length, k, d, rng.choice([0, (k - 1) * d // 2]), dtype, dtype == "f32" and rng.random() < 0.7)
    cin, cout, train = _channels(rng), _channels(rng), rng.random() < 0.75
    cap = 7.4e9 if cin % 32 == 0 and cout % 32 == 0 else 3.7e9      # FLOP of one product over the layer
    if kind == "dense1d":
        length, k = _log(rng, 200, 8192), rng.choice([1, 3, 3, 5])
        b = int(min(rng.choice([1, 8, 16, 32]), max(1, cap / (2.0 * cin * cout * k * length))))
        return dense1d(b, cin, cout, length, k, rng.choice([0, k // 2]), train)
    k = rng.choice([1, 3, 3, 3, 5])
    s = rng.choice([1, 1, 2])
    h = _log(rng, 7, 112)
    w = h if rng.random() < 0.7 else _log(rng, 7, 112)
    n = int(min(rng.choice([1, 8, 32, 64]), max(1, cap * s * s / (2.0 * cin * cout * k * k * h * w))))
    return dense2d(n, cin, cout, h, w, k, s, k // 2, train)


def _out(n, k, s, p, d=1):
    return (n + 2 * p - d * (k - 1) - 1) // s + 1


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = DTYPES[case.get("dtype", "f32")]

    def uniform(*shape):
        return torch.rand(shape, generator=gen, device="cuda").mul_(2).sub_(1).to(dt)

    def normal(*shape, std=1.0, dtype=torch.float32):
        return torch.randn(shape, generator=gen, device="cuda").mul_(std).to(dtype)

    st = {"case": case}
    kind = case["kind"]
    if kind == "slide":
        st["x"] = uniform(case["rows"], case["length"])
    elif kind == "pool":
        n, c, h, w, k, s, p = (case[v] for v in ("n", "c", "h", "w", "k", "s", "p"))
        st["x"] = normal(n, c, h, w, dtype=dt)
        if case["train"]:
            st["gy"] = normal(n, c, _out(h, k, s, p), _out(w, k, s, p))
    elif kind == "depthwise":
        b, c, length, k, d, p = (case[v] for v in ("b", "c", "length", "k", "d", "p"))
        st["x"] = uniform(b, c, length)
        st["wgt"] = normal(c, 1, k, std=k ** -0.5)
        if case["train"]:
            st["gy"] = normal(b, c, _out(length, k, 1, p, d))
    elif kind == "dense1d":
        b, cin, cout, length, k, p = (case[v] for v in ("b", "cin", "cout", "length", "k", "p"))
        st["x"] = normal(b, cin, length)
        st["wgt"] = normal(cout, cin, k, std=(2.0 / (cin * k)) ** 0.5)
        if case["train"]:
            st["gy"] = normal(b, cout, _out(length, k, 1, p))
    else:
        n, cin, cout, h, w, k, s, p = (case[v] for v in ("n", "cin", "cout", "h", "w", "k", "s", "p"))
        st["x"] = normal(n, cin, h, w).clamp_(min=0)            # activations behind a ReLU
        st["wgt"] = normal(cout, cin, k, k, std=(2.0 / (cin * k * k)) ** 0.5)
        if case["train"]:
            st["gy"] = normal(n, cout, _out(h, k, s, p), _out(w, k, s, p))
    return st


def run(state):
    case, x = state["case"], state["x"]
    kind = case["kind"]
    if kind == "slide":
        op, w, scale = OPS[case["op"]], case["w"], 1.0 / case["w"]
        if case["mode"] != "valid":
            return B.sws_slide1d_padded(op, x, w, (w - 1) // 2, w // 2, MODES[case["mode"]], scale)
        return (B.sws_slide1d if case["dtype"] == "f32" else B.sws_slide1d_16)(op, x, w, scale)
    if kind == "pool":
        op, k, s, p, scale = OPS[case["op"]], case["k"], case["s"], case["p"], 1.0 / case["k"] ** 2
        y = (B.sws_pool2d if case["dtype"] == "f32" else B.sws_pool2d_16)(op, x, k, k, s, s, p, p, scale)
        if not case["train"]:
            return y
        if op == B.OP_MAX:
            return {"y": y, "gx": B.sws_maxpool2d_grad(x, state["gy"], k, k, s, s, p, p)}
        return {"y": y, "gx": B.sws_avgpool2d_grad(state["gy"], case["h"], case["w"], k, k, s, s, p, p, B.SWS_DIV_SCALE, scale)}
    wgt = state["wgt"]
    if kind == "depthwise":
        c, k, d, p = case["c"], case["k"], case["d"], case["p"]
        y = (B.sws_conv1d if case["dtype"] == "f32" else B.sws_conv1d_16)(x, wgt, 1, p, d, c)
        if not case["train"]:
            return y
        return {"y": y, "gx": B.sws_conv1d_grad_input(state["gy"], wgt, case["length"], 1, p, d, c),
                "gw": B.sws_conv1d_grad_weight(x, state["gy"], k, 1, p, d, c)}
    if kind == "dense1d":
        k, p = case["k"], case["p"]
        y = B.sws_conv1d(x, wgt, 1, p)
        if not case["train"]:
            return y
        return {"y": y, "gx": B.sws_conv1d_grad_input(state["gy"], wgt, case["length"], 1, p),
                "gw": B.sws_conv1d_grad_weight(x, state["gy"], k, 1, p)}
    k, s, p = case["k"], case["s"], case["p"]
    y = B.sws_conv2d(x, wgt, s, s, p, p)
    if not case["train"]:
        return y
    return {"y": y, "gx": B.sws_conv2d_grad_input(state["gy"], wgt, case["h"], case["w"], s, s, p, p),
            "gw": B.sws_conv2d_grad_weight(x, state["gy"], k, k, s, s, p, p)}


def work(case):
    kind = case["kind"]
    size = 4 if case.get("dtype", "f32") == "f32" else 2
    if kind == "slide":
        lo = case["length"] if case["mode"] != "valid" else case["length"] - case["w"] + 1
        return {"bytes": size * case["rows"] * (case["length"] + lo), "flops": 0}
    if kind == "pool":
        ho, wo = _out(case["h"], case["k"], case["s"], case["p"]), _out(case["w"], case["k"], case["s"], case["p"])
        x, y = case["n"] * case["c"] * case["h"] * case["w"], case["n"] * case["c"] * ho * wo
        return {"bytes": (2 if case["train"] else 1) * size * (x + y), "flops": 0}
    if kind == "depthwise":
        lo = _out(case["length"], case["k"], 1, case["p"], case["d"])
        x, y, wgt = case["b"] * case["c"] * case["length"], case["b"] * case["c"] * lo, case["c"] * case["k"]
        flops = 2.0 * y * case["k"]
    elif kind == "dense1d":
        lo = _out(case["length"], case["k"], 1, case["p"])
        x, y = case["b"] * case["cin"] * case["length"], case["b"] * case["cout"] * lo
        wgt = case["cin"] * case["cout"] * case["k"]
        flops = 2.0 * y * case["cin"] * case["k"]
    else:
        ho, wo = _out(case["h"], case["k"], case["s"], case["p"]), _out(case["w"], case["k"], case["s"], case["p"])
        x, y = case["n"] * case["cin"] * case["h"] * case["w"], case["n"] * case["cout"] * ho * wo
        wgt = case["cin"] * case["cout"] * case["k"] ** 2
        flops = 2.0 * y * case["cin"] * case["k"] ** 2
    if case["train"]:
        return {"bytes": 2 * (4 * wgt + size * (x + y)), "flops": 3 * flops}
    return {"bytes": 4 * wgt + size * (x + y), "flops": flops}


def tolerance(case):
    if case.get("op") in ("max", "min") and not case.get("train"):
        return "exact"                                        # a maximum of representable values is one of them
    if case.get("dtype", "f32") == "bf16":
        return {"rel": 6e-3, "max": 2e-2}                     # one rounding to 8 bits
    if case.get("dtype", "f32") == "f16":
        return {"rel": 8e-4, "max": 4e-3}                     # one rounding to 11 bits
    if case["kind"] in ("slide", "pool"):
        return {"rel": 1e-6, "max": 1e-5}                     # fp32 sums of up to a few hundred terms
    return {"rel": 4e-6, "max": 1e-4}                         # fp32 sums of up to 10^5 .. 10^7 products


# ---- the same outputs in 64 bits -------------------------------------------------------------------------------------

def _windows(x, w, f):
    """f over w consecutive elements of the last axis, by doubling."""
    acc, off, n, p = None, 0, 1, x
    while True:
        if w & n:
            if acc is None:
                acc = p
            else:
                m = x.shape[-1] - off - n + 1
                acc = f(acc[..., :m], p[..., off:off + m])
            off += n
        if off == w:
            return acc
        p, n = f(p[..., :p.shape[-1] - n], p[..., n:]), 2 * n


def _exact_slide(case, x):
    w, add = case["w"], case["op"] == "add"
    f = torch.add if add else torch.maximum if case["op"] == "max" else torch.minimum
    n = x.shape[-1]
    if case["mode"] == "valid":
        y = _windows(x, w, f)
        return y / w if add else y
    left, right = (w - 1) // 2, w // 2
    if case["mode"] == "shrink":
        y = _windows(F.pad(x, (left, right), value=0.0 if add else -math.inf if case["op"] == "max" else math.inf), w, f)
        cells = _windows(F.pad(torch.ones(1, n, dtype=x.dtype, device=x.device), (left, right)), w, torch.add)
        return y / cells if add else y
    e = torch.arange(-left, n + right, device=x.device)
    if case["mode"] == "mirror":
        e = torch.where(e < 0, -e, torch.where(e >= n, 2 * (n - 1) - e, e))
    else:
        e = e % n if case["mode"] == "periodic" else e.clamp(0, n - 1)
    y = _windows(x[:, e], w, f)
    return y / w if add else y


def _exact_pool(case, x, gy):
    k, s, p, add = case["k"], case["s"], case["p"], case["op"] == "add"
    n, c, h, w = x.shape
    ho, wo = _out(h, k, s, p), _out(w, k, s, p)
    xe = F.pad(x, (p, p, p, p), value=0.0 if add else -math.inf)
    at = [(a, b, (slice(None), slice(None), slice(a, a + s * (ho - 1) + 1, s), slice(b, b + s * (wo - 1) + 1, s)))
          for a in range(k) for b in range(k)]
    y, arg = torch.full((n, c, ho, wo), 0.0 if add else -math.inf, dtype=x.dtype, device=x.device), None
    if add:
        for _, _, cut in at:
            y += xe[cut]
        y /= k * k
    else:
        arg = torch.full(y.shape, -1, dtype=torch.int16, device=x.device)
        for i, (_, _, cut) in enumerate(at):                    # row-major, the first of equal maxima
            v = xe[cut]
            more = v > y
            y, arg = torch.where(more, v, y), torch.where(more, torch.full_like(arg, i), arg)
    if gy is None:
        return y
    gx = torch.zeros_like(xe)
    for i, (_, _, cut) in enumerate(at):
        gx[cut] += gy / (k * k) if add else torch.where(arg == i, gy, torch.zeros_like(gy))
    return {"y": y, "gx": gx[:, :, p:p + h, p:p + w].contiguous()}


def _exact_depthwise(case, x, wgt, gy):
    k, d, p = case["k"], case["d"], case["p"]
    lo = _out(x.shape[-1], k, 1, p, d)
    xe = F.pad(x, (p, p))
    y = torch.zeros(x.shape[0], x.shape[1], lo, dtype=x.dtype, device=x.device)
    for t in range(k):
        y.addcmul_(xe[..., t * d:t * d + lo], wgt[:, 0, t, None])
    if gy is None:
        return y
    gx, gw = torch.zeros_like(xe), torch.zeros_like(wgt)
    for t in range(k):
        gx[..., t * d:t * d + lo].addcmul_(gy, wgt[:, 0, t, None])
        gw[:, 0, t] = (xe[..., t * d:t * d + lo] * gy).sum((0, 2))
    return {"y": y, "gx": gx[..., p:p + x.shape[-1]].contiguous(), "gw": gw}


def _exact_dense2d(x, wgt, gy, s, ph, pw):
    """Per tap one product of matrices: channels by channels times positions."""
    n, cin, h, w = x.shape
    cout, _, kh, kw = wgt.shape
    ho, wo = _out(h, kh, s, ph), _out(w, kw, s, pw)
    xe = F.pad(x, (pw, pw, ph, ph)).transpose(0, 1).contiguous()           # [Cin, N, He, We]
    y = torch.zeros(cout, n * ho * wo, dtype=x.dtype, device=x.device)
    g2 = None if gy is None else gy.transpose(0, 1).reshape(cout, -1).contiguous()
    gx, gw = torch.zeros_like(xe), torch.zeros_like(wgt)
    for a in range(kh):
        for b in range(kw):
            cut = (slice(None), slice(None), slice(a, a + s * (ho - 1) + 1, s), slice(b, b + s * (wo - 1) + 1, s))
            xt = xe[cut].reshape(cin, -1).contiguous()
            y += wgt[:, :, a, b].contiguous() @ xt
            if gy is not None:
                gw[:, :, a, b] = g2 @ xt.t().contiguous()
                gx[cut] += (wgt[:, :, a, b].t().contiguous() @ g2).view(cin, n, ho, wo)
    y = y.view(cout, n, ho, wo).transpose(0, 1).contiguous()
    if gy is None:
        return y
    return {"y": y, "gx": gx[:, :, ph:ph + h, pw:pw + w].transpose(0, 1).contiguous(), "gw": gw}


def exact(case, seed):
    st = prepare(case, seed)
    x, wgt, gy = (st[v].double() if v in st else None for v in ("x", "wgt", "gy"))
    kind = case["kind"]
    if kind == "slide":
        return _exact_slide(case, x)
    if kind == "pool":
        return _exact_pool(case, x, gy)
    if kind == "depthwise":
        return _exact_depthwise(case, x, wgt, gy)
    if kind == "dense1d":
        got = _exact_dense2d(x[:, :, None], wgt[:, :, None], None if gy is None else gy[:, :, None], 1, 0, case["p"])
        return {v: t.squeeze(2) for v, t in got.items()} if isinstance(got, dict) else got.squeeze(2)
    return _exact_dense2d(x, wgt, gy, case["s"], case["p"], case["p"])
