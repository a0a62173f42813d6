"""The work whose speed counts, as a user of the library has it done: single convolution passes, whole
convolution layers, gradient aggregation with the model update, and whole SGD iterations.

A case is a plain dict.  `listed()` names the cases, `draw(rng)` makes one more of the same ranges,
`prepare` makes what a program holds before the call, `run` is one pass through the public entry
points, `work` what a pass cannot do without, `tolerance` how far two correct implementations may be
apart and `exact` the same results in 64 bits from plain torch.
"""
import math

import torch
import torch.nn.functional as F

import cg_synth
import paper_1706_00095_amd as cg

# Solver constants of a run whose learning rate has been lowered a few times: a timed pass repeats on
# the same batch, and a small step keeps the model where it was made.
SOLVER = dict(lr=1e-4, mu=0.9, wd=5e-4)
MATH = {"fp32": cg.CG_MATH_FP32, "bf16": cg.CG_MATH_BF16, "bf16x3": cg.CG_MATH_BF16X3}
NETS = {"tiny": (cg_synth.tiny_cnn_layers, 10), "alexnet": (cg_synth.alexnet_layers, 1000),
        "inception": (cg_synth.inception_layers, 1000),
        "googlenet": (lambda: cg_synth.googlenet_layers()[:2], 1000)}


def _conv(passes, B, C, H, W, M, KH, KW, stride, pad, groups, math="fp32"):
    return dict(op="conv", passes=passes, B=B, C=C, H=H, W=W, M=M, KH=KH, KW=KW, stride=stride, pad=pad, groups=groups,
                math=math)


def listed():
    return [
        # --- convolution layers, one pass at a time (fwd: forward, bd: backward-data, bw: backward-weight + bias)
        # the stem of the AlexNet-shaped net on a full per-worker batch: 3 channels, 11x11 window, stride 4
        dict(name="conv1_fwd_b256", **_conv("fwd", 256, 3, 227, 227, 96, 11, 11, 4, 0, 1)),
        # its 5x5 layer in two groups: the gradient that travels on to the layer below
        dict(name="conv2_bwd_data_b256", **_conv("bd", 256, 96, 27, 27, 256, 5, 5, 1, 2, 2)),
        # its widest 3x3 layer forward: the largest plain contraction of the net
        dict(name="conv3_fwd_b256", **_conv("fwd", 256, 256, 13, 13, 384, 3, 3, 1, 1, 1)),
        # a grouped 3x3 layer's gradient on the smaller per-worker batch
        dict(name="conv4_bwd_weight_b64", **_conv("bw", 64, 384, 13, 13, 384, 3, 3, 1, 1, 2)),
        # the three-product bf16 mode, chosen by the caller, on the last convolution
        dict(name="conv5_bwd_data_bf16x3_b256", **_conv("bd", 256, 384, 13, 13, 256, 3, 3, 1, 1, 2, "bf16x3")),
        # a 1x1 reduction of an inception module, forward and both backward passes: little arithmetic per byte
        dict(name="inception_1x1_layer_b32", **_conv("all", 32, 192, 28, 28, 96, 1, 1, 1, 0, 1)),
        # a small layer of odd sizes with a stride: remainders of every tile, few blocks
        dict(name="ragged_strided_layer_b5", **_conv("all", 5, 19, 33, 29, 37, 5, 3, 2, 1, 1)),
        # --- gradient aggregation + update
        # the eight parameter buckets of the AlexNet-shaped net, four peers
        dict(name="update_alexnet_k4", op="update", buckets="alexnet", n=0, K=4, tree=False, grad_scale=1.0),
        # one layer's bucket (the fifth convolution's), eight peers added as the reduction tree does, mean over ranks
        dict(name="update_conv5_tree_k8", op="update", buckets="one", n=442624, K=8, tree=True, grad_scale=1.0 / 9.0),
        # --- whole iterations (forward, backward, aggregation + update on a second stream)
        # the smallest net: nothing but launches
        dict(name="tiny_step_b8", op="step", net="tiny", B=8, K=4, tree=False),
        # the headline workload
        dict(name="alexnet_step_b256", op="step", net="alexnet", B=256, K=4, tree=False),
        # the second benchmark net: 142 layers, most of them small
        dict(name="googlenet_step_b32", op="step", net="googlenet", B=32, K=8, tree=False),
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.random()
    if kind < 0.15:
        many = rng.random() < 0.4
        K = rng.choice([1, 2, 3, 4, 5, 7, 8, 12, 16])
        n = 0 if many else _logint(rng, 1000, 40_000_000)
        return dict(op="update", buckets="alexnet" if many else "one", n=n, K=K, tree=rng.random() < 0.4,
                    grad_scale=1.0 if rng.random() < 0.6 else 1.0 / (K + 1))
    if kind < 0.30:
        net = rng.choice(["tiny", "alexnet", "inception", "googlenet"])
        B = {"tiny": _logint(rng, 2, 128), "alexnet": _logint(rng, 8, 224), "inception": _logint(rng, 2, 64),
             "googlenet": _logint(rng, 2, 30)}[net]
        return dict(op="step", net=net, B=B, K=rng.choice([1, 2, 4, 7, 8]), tree=rng.random() < 0.3)
    while True:
        k = rng.choice([1, 1, 3, 3, 3, 5, 7, 11])
        KH, KW = k, k if rng.random() < 0.8 else rng.choice([1, 3, 5])
        stride = rng.choice([1, 1, 1, 2]) if k < 7 else rng.choice([2, 4])
        stem = k >= 7 or rng.random() < 0.15
        groups = 1 if stem else rng.choice([1, 1, 1, 2])
        C = rng.choice([1, 3, 3, 4]) if stem else groups * _logint(rng, 8, 512 // groups)
        M = groups * _logint(rng, 8, 512 // groups)
        H = _logint(rng, 64, 227) if stem else _logint(rng, 7, 56)
        W = H if rng.random() < 0.7 else max(7, H + rng.randint(-H // 4, H // 4))
        B = _logint(rng, 1, 256)
        pad = rng.choice([0, k // 2])
        if H + 2 * pad < KH or W + 2 * pad < KW:
            continue
        OH, OW = (H + 2 * pad - KH) // stride + 1, (W + 2 * pad - KW) // stride + 1
        gflop = 2e-9 * M * (C // groups) * KH * KW * B * OH * OW
        if not 0.002 <= gflop <= 80 or B * max(C * H * W, M * OH * OW) > 120_000_000:
            continue
        passes = rng.choice(["fwd", "bd", "bw", "all"])
        mode = rng.choice(["fp32"] * 8 + ["bf16", "bf16x3"])
        if mode != "fp32" and stride > 1 and (C // groups) * stride * stride < 8:
            mode = "fp32"          # that backward-data exists in fp32 only
        return _conv(passes, B, C, H, W, M, KH, KW, stride, pad, groups, mode)


# ---- preparation ---------------------------------------------------------------------------------

_STREAMS = []


def _streams():
    """The two streams of a training program, made once."""
    if not _STREAMS:
        _STREAMS.extend([torch.cuda.Stream(), torch.cuda.Stream()])
    return _STREAMS


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(shape, std, gen):
    return torch.empty(shape, device="cuda").normal_(0.0, std, generator=gen)


def _padded(n):
    return -(-n // 64) * 64        # buckets of one flat buffer start on 256-byte boundaries


def _flat(sizes, fill=None):
    """One flat buffer and its views, one per bucket."""
    starts, at = [], 0
    for n in sizes:
        starts.append(at)
        at += _padded(n)
    flat = torch.zeros(at, device="cuda")
    views = [flat[s:s + n] for s, n in zip(starts, sizes)]
    if fill is not None:
        for v in views:
            fill(v)
    return flat, views


def _conv_tensors(c, seed):
    gen = _gen(seed)
    Cg, Mg = c["C"] // c["groups"], c["M"] // c["groups"]
    fan_in, fan_out = Cg * c["KH"] * c["KW"], Mg * c["KH"] * c["KW"]
    OH, OW = _out_size(c)
    x = _randn((c["B"], c["C"], c["H"], c["W"]), fan_in ** -0.5, gen)
    w = _randn((c["M"], Cg, c["KH"], c["KW"]), fan_in ** -0.5, gen)
    b = _randn((c["M"],), 0.1, gen)
    dy = _randn((c["B"], c["M"], OH, OW), fan_out ** -0.5, gen)
    return x, w, b, dy


def _out_size(c):
    return ((c["H"] + 2 * c["pad"] - c["KH"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["KW"]) // c["stride"] + 1)


def _prepare_conv(c, seed):
    d = cg.conv_desc(c["B"], c["C"], c["H"], c["W"], c["M"], c["KH"], c["KW"], stride=c["stride"], pad=c["pad"],
                     groups=c["groups"])
    x, w, b, dy = _conv_tensors(c, seed)
    ws = max(cg.cg_conv_workspace_bytes(d, p) for p in (cg.CG_PASS_FWD, cg.CG_PASS_BWD_DATA, cg.CG_PASS_BWD_WEIGHT))
    return dict(case=c, d=d, x=x, w=w, b=b, dy=dy, y=torch.empty_like(dy), dx=torch.empty_like(x), dw=torch.empty_like(w),
                db=torch.empty_like(b), ws=torch.empty(max(ws, 16), dtype=torch.uint8, device="cuda"))


def _update_sizes(c):
    return list(cg_synth.ALEXNET_BUCKETS.values()) if c["buckets"] == "alexnet" else [c["n"]]


def _prepare_update(c, seed):
    gen, sizes = _gen(seed), _update_sizes(c)
    w, ws = _flat(sizes, lambda t: t.normal_(0.0, 1e-2, generator=gen))
    v, vs = _flat(sizes, lambda t: t.normal_(0.0, 1e-5, generator=gen))
    g, gs = _flat(sizes, lambda t: t.normal_(0.0, 1e-3, generator=gen))
    peers = [_flat(sizes, lambda t: t.normal_(0.0, 1e-3, generator=gen))[1] for _ in range(c["K"])]
    by_bucket = [[p[i] for p in peers] for i in range(len(sizes))]
    return dict(case=c, sizes=sizes, w=w, v=v, g=g, ws=ws, vs=vs, gs=gs, peers=by_bucket,
                sgd=cg.cg_sgd(SOLVER["lr"], SOLVER["mu"], SOLVER["wd"], c["grad_scale"]))


def _prepare_step(c, seed):
    make, classes = NETS[c["net"]]
    layers, in_shape = make()
    gen, B = _gen(seed), c["B"]
    params = cg_synth.param_layers(layers, in_shape)
    shapes = cg_synth.infer_shapes(layers, in_shape)
    sizes = [math.prod(ws) + nb for _, ws, nb in params]
    net = cg.Net(layers, B, in_shape)
    w, ws = _flat(sizes)
    for (_, wshape, nb), t in zip(params, ws):
        t[:t.numel() - nb].normal_(0.0, math.prod(wshape[1:]) ** -0.5, generator=gen)
        t[t.numel() - nb:].normal_(0.0, 0.1, generator=gen)
    v, vs = _flat(sizes, lambda t: t.normal_(0.0, 1e-5, generator=gen))
    g, gs = _flat(sizes)
    peers = [_flat(sizes, lambda t: t.normal_(0.0, 1e-3, generator=gen))[1] for _ in range(c["K"])]
    for i, (li, _, _) in enumerate(params):
        cg.cg_net_bind(net, li, ws[i], vs[i], gs[i], [p[i] for p in peers])
    masks = {}
    for i, ly in enumerate(layers):
        if ly["kind"] == "dropout":
            masks[i] = (torch.rand((B, math.prod(shapes[i])), device="cuda", generator=gen) >= ly["p"]).to(torch.uint8)
    workspace = torch.empty(cg.cg_net_workspace_bytes(net), dtype=torch.uint8, device="cuda")
    logits = cg.cg_net_tensor(net, layers[-1]["inputs"][0], 0, workspace)
    return dict(case=c, net=net, layers=layers, in_shape=in_shape, params=params, w=w, v=v, g=g, w_views=ws, v_views=vs,
                peers=peers, masks=masks, workspace=workspace, logits=logits,
                x=torch.empty((B,) + tuple(in_shape), device="cuda").normal_(generator=gen),
                labels=torch.randint(0, classes, (B,), device="cuda", generator=gen, dtype=torch.int32),
                loss=torch.zeros(1, device="cuda"), streams=_streams(),
                sgd=cg.cg_sgd(SOLVER["lr"], SOLVER["mu"], SOLVER["wd"], 1.0),
                flags=cg.CG_STEP_OVERLAP | (cg.CG_STEP_TREE_SUM if c["tree"] else 0))


def prepare(case, seed):
    return {"conv": _prepare_conv, "update": _prepare_update, "step": _prepare_step}[case["op"]](case, seed)


# ---- one pass ------------------------------------------------------------------------------------

def run(state):
    c = state["case"]
    if c["op"] == "conv":
        s, m, out = state, MATH[c["math"]], {}
        if c["passes"] in ("fwd", "all"):
            cg.cg_conv_fwd_math(s["d"], s["x"], s["w"], s["b"], s["y"], s["ws"], m)
            out["y"] = s["y"]
        if c["passes"] in ("bw", "all"):
            cg.cg_conv_bwd_weight_math(s["d"], s["x"], s["dy"], s["dw"], s["db"], s["ws"], m)
            out["dw"], out["db"] = s["dw"], s["db"]
        if c["passes"] in ("bd", "all"):
            cg.cg_conv_bwd_data_math(s["d"], s["dy"], s["w"], s["dx"], s["ws"], m)
            out["dx"] = s["dx"]
        return out
    if c["op"] == "update":
        s = state
        if c["buckets"] == "one":
            f = cg.cg_grad_reduce_sgd_tree if c["tree"] else cg.cg_grad_reduce_sgd
            f(s["ws"][0], s["vs"][0], s["gs"][0], s["peers"][0], s["sizes"][0], s["sgd"])
        else:
            f = cg.cg_grad_reduce_sgd_tree_multi if c["tree"] else cg.cg_grad_reduce_sgd_multi
            f(s["ws"], s["vs"], s["gs"], s["peers"], s["sizes"], s["sgd"])
        return {"w": s["w"], "v": s["v"]}
    s = state
    cg.cg_train_step(s["net"], s["x"], s["labels"], s["masks"], s["sgd"], s["workspace"], s["streams"][0], s["streams"][1],
                     s["loss"], s["flags"])
    return {"loss": s["loss"], "logits": s["logits"], "g": s["g"], "w": s["w"], "v": s["v"]}


# ---- what a pass cannot do without ---------------------------------------------------------------

def work(case):
    c = case
    if c["op"] == "conv":
        OH, OW = _out_size(c)
        nx, ny = c["B"] * c["C"] * c["H"] * c["W"], c["B"] * c["M"] * OH * OW
        nw = c["M"] * (c["C"] // c["groups"]) * c["KH"] * c["KW"]
        flops = 2.0 * nw * c["B"] * OH * OW
        n = 3 if c["passes"] == "all" else 1
        return {"bytes": 4.0 * n * (nx + ny + nw), "flops": n * flops}
    if c["op"] == "update":
        n = sum(_update_sizes(c))
        return {"bytes": (4.0 * c["K"] + 20.0) * n, "flops": (c["K"] + 6.0) * n}
    layers, in_shape = NETS[c["net"]][0]()
    shapes = cg_synth.infer_shapes(layers, in_shape)
    flops, nparam, acts = 0.0, 0, 0
    for i, wshape, nb in cg_synth.param_layers(layers, in_shape):
        pixels = shapes[i][1] * shapes[i][2] if layers[i]["kind"] == "conv" else 1
        first = layers[i]["inputs"][0] < 0
        flops += (2 if first else 3) * 2.0 * math.prod(wshape) * pixels * c["B"]
        nparam += math.prod(wshape) + nb
        acts += c["B"] * shapes[i][0] * pixels     # kept from forward for backward: written once, read once
    x = c["B"] * math.prod(in_shape)
    return {"bytes": 4.0 * (x + 2 * acts) + (4.0 * c["K"] + 20.0 + 4.0) * nparam, "flops": flops}


def tolerance(case):
    if case["op"] == "update":
        return "exact"          # the entry point fixes the order of its operations
    if case["op"] == "step":
        # A rectifier or a pooling window whose decision hangs on the last bit sends a whole gradient
        # elsewhere: with n such decisions per batch and a share p of them turned, the gradients move by
        # about sqrt(p).  Against 64 bits the gradients of the AlexNet-shaped net are 1e-3 .. 3.4e-3 off
        # (its LRN makes many near-ties), those of the others up to 1.4e-4 (2e-7 without a turned one).
        return {"rel": 1.4e-2, "max": 0.75} if case["net"] == "alexnet" else {"rel": 2e-3, "max": 0.2}
    if case["math"] == "bf16":
        return {"rel": 1e-2, "max": 0.1}          # 2.4e-3 off 64 bits
    if case["math"] == "bf16x3":
        return {"rel": 2e-5, "max": 1e-4}         # 4.4e-6 and 2.5e-5 off 64 bits
    return {"rel": 4e-6, "max": 4e-5}             # up to 9.8e-7 and 8.3e-6 off 64 bits


# ---- the same in 64 bits -------------------------------------------------------------------------

def _cols(x, c):
    """[groups][Cg*KH*KW, B*OH*OW] patch matrices of an image batch."""
    u = F.unfold(x, (c["KH"], c["KW"]), padding=c["pad"], stride=c["stride"])          # [B, C*KH*KW, P]
    B, R, P = u.shape
    return u.view(B, c["groups"], R // c["groups"], P).permute(1, 2, 0, 3).reshape(c["groups"], R // c["groups"], B * P)


def _conv64(x, w, b, c):
    """Forward convolution by patch matrices, differentiable, a few images at a time."""
    OH, OW = _out_size(c)
    Mg = c["M"] // c["groups"]
    per_image = x.shape[1] * c["KH"] * c["KW"] * OH * OW
    step = max(1, min(x.shape[0], 150_000_000 // max(1, per_image)))
    out = []
    for i in range(0, x.shape[0], step):
        xi = x[i:i + step]
        cols = _cols(xi, c)
        y = torch.cat([w[g * Mg:(g + 1) * Mg].reshape(Mg, -1) @ cols[g] for g in range(c["groups"])])
        out.append(y.view(c["M"], xi.shape[0], OH, OW).permute(1, 0, 2, 3) + b.view(1, -1, 1, 1))
    return torch.cat(out)


def _exact_conv(c, seed):
    x, w, b, dy = (t.double() for t in _conv_tensors(c, seed))
    OH, OW = _out_size(c)
    G, Mg, Cg = c["groups"], c["M"] // c["groups"], c["C"] // c["groups"]
    per_image = c["C"] * c["KH"] * c["KW"] * OH * OW
    step = max(1, min(c["B"], 150_000_000 // max(1, per_image)))
    out = {}
    if c["passes"] in ("fwd", "all"):
        out["y"] = _conv64(x, w, b, c)
    if c["passes"] in ("bw", "all"):
        dw = torch.zeros(G, Mg, Cg * c["KH"] * c["KW"], dtype=torch.float64, device="cuda")
        for i in range(0, c["B"], step):
            cols = _cols(x[i:i + step], c)
            d = dy[i:i + step].reshape(-1, G, Mg, OH * OW).permute(1, 2, 0, 3).reshape(G, Mg, -1)
            for g in range(G):
                dw[g] += d[g] @ cols[g].t().contiguous()
        out["dw"], out["db"] = dw.view(w.shape), dy.sum((0, 2, 3))
    if c["passes"] in ("bd", "all"):
        dx = []
        for i in range(0, c["B"], step):
            d = dy[i:i + step].reshape(-1, G, Mg, OH * OW).permute(1, 2, 0, 3).reshape(G, Mg, -1)
            n = d.shape[2] // (OH * OW)
            cols = torch.stack([w[g * Mg:(g + 1) * Mg].reshape(Mg, -1).t().contiguous() @ d[g] for g in range(G)])
            cols = cols.view(G * Cg * c["KH"] * c["KW"], n, OH * OW).permute(1, 0, 2).contiguous()
            dx.append(F.fold(cols, (c["H"], c["W"]), (c["KH"], c["KW"]), padding=c["pad"], stride=c["stride"]))
        out["dx"] = torch.cat(dx)
    return out


def _update64(w, v, gsum, lr, mu, wd):
    vn = mu * v + lr * (gsum + wd * w)
    return w - vn, vn


def _float32(x):
    """The value a C float holds, as the solver's constants reach the library."""
    return float(torch.tensor(x, dtype=torch.float32))


def _solver64():
    return _float32(SOLVER["lr"]), _float32(SOLVER["mu"]), _float32(SOLVER["wd"])


def _exact_update(c, seed):
    s = _prepare_update(c, seed)
    w, v, total = s["w"].double(), s["v"].double(), s["g"].double()
    at = 0
    for i, n in enumerate(s["sizes"]):
        for p in s["peers"][i]:
            total[at:at + n] += p.double()
        at += _padded(n)
    w, v = _update64(w, v, total * _float32(c["grad_scale"]), *_solver64())
    return {"w": w, "v": v}


def _forward64(layers, x, params, labels, masks):
    acts = []

    def src(i):
        return x if i < 0 else acts[i]

    for i, ly in enumerate(layers):
        t, kind = src(ly["inputs"][0]), ly["kind"]
        if kind == "conv":
            c = dict(M=ly["M"], KH=ly["k"], KW=ly["k"], stride=ly["stride"], pad=ly["pad"], groups=ly["groups"],
                     H=t.shape[2], W=t.shape[3])
            t = _conv64(t, *params[i], c)
        elif kind == "relu":
            t = F.relu(t)
        elif kind == "lrn":
            t = F.local_response_norm(t, ly["size"], ly["alpha"], ly["beta"], ly["kappa"])
        elif kind == "maxpool":
            t = F.max_pool2d(t, ly["k"], ly["stride"], ly["pad"], ceil_mode=True)
        elif kind == "avgpool":
            t = t.mean((2, 3), keepdim=True)
        elif kind == "fc":
            t = (t.flatten(1) @ params[i][0].t() + params[i][1])[:, :, None, None]
        elif kind == "dropout":
            t = t * masks[i].view(t.shape).to(t.dtype) / (1.0 - ly["p"])
        elif kind == "concat":
            t = torch.cat([src(j) for j in ly["inputs"]], 1)
        elif kind == "softmax_ce":
            t = F.cross_entropy(t.flatten(1), labels.long())
        acts.append(t)
    return acts


def _exact_step(c, seed):
    s = _prepare_step(c, seed)
    params, leaves = {}, []
    for (li, wshape, nb), t in zip(s["params"], s["w_views"]):
        leaf = t.double().requires_grad_(True)
        leaves.append(leaf)
        params[li] = (leaf[:leaf.numel() - nb].view(wshape), leaf[leaf.numel() - nb:])
    acts = _forward64(s["layers"], s["x"].double(), params, s["labels"], s["masks"])
    grads = torch.autograd.grad(acts[-1], leaves)
    g, w, v = torch.zeros_like(s["g"], dtype=torch.float64), s["w"].double(), s["v"].double()
    total, at = torch.zeros_like(g), 0
    for i, gr in enumerate(grads):
        n = gr.numel()
        g[at:at + n] = gr
        total[at:at + n] = gr
        for p in s["peers"]:
            total[at:at + n] += p[i].double()
        at += _padded(n)
    w, v = _update64(w, v, total, *_solver64())
    logits = acts[s["layers"][-1]["inputs"][0]].detach().reshape(-1)
    return {"loss": acts[-1].detach().reshape(1), "logits": logits, "g": g, "w": w, "v": v}


def exact(case, seed):
    return {"conv": _exact_conv, "update": _exact_update, "step": _exact_step}[case["op"]](case, seed)
