"""The work that a user of this framework has it do, as cases that can be timed.

A case is a dict of plain values.  Its ``kind`` says which public entry points a
pass goes through:

  forward   one convolution layer's forward pass (bias, and ReLU where set)
  backward  one convolution layer's backward pass: the gradients of its input,
            weights and bias from the gradient of its output
  layer     a forward pass and the backward pass of the same layer
  fc        the same for an inner product (the 1x1 convolution of a 1x1 image)
  glue      max-pool + LRN forward, then their backward
  train     one SGD iteration of LeNet: forward, softmax loss, backward, update
  step      forward and backward of the CaffeNet conv1-5 chain with its glue,
            without the gradient of the input images (as in training)
  serve     the whole CaffeNet's forward pass, images to scores

``dtype`` is "f32", "bf16" (bfloat16 input and weights) or "bf16_f32in" (bfloat16
weights, float input that the library rounds).  Buffers, workspaces and networks
are made in ``prepare``, as a program that runs many passes keeps them.
"""
import math

import torch
import torch.nn.functional as F

import paper_1408_5093_amd as lib
from paper_1408_5093_amd.net import ConvStack, SGDTrainer
from paper_1408_5093_amd.workloads import (CAFFENET, CAFFENET_FC, CAFFENET_LRN, CAFFENET_NET,
                                           CAFFENET_NET_GLUE, CAFFENET_POOL, LENET_NET,
                                           LENET_NET_GLUE, LENET_SOLVER)

STEP_GLUE = {l: CAFFENET_NET_GLUE[l] for l in (0, 1)}


def _conv(name, kind, dtype, N, L):
    return dict(name=name, kind=kind, dtype=dtype, N=N, C=L.C, H=L.H, W=L.W, K=L.K, k=L.k, s=L.s,
                p=L.p, g=L.g, relu=L.relu)


def listed():
    conv1, conv2, conv3 = CAFFENET[:3]
    fc6 = CAFFENET_FC[0]
    return [
        # one image classified by the whole network: the smallest call, launch
        # latency and the streaming of 61 M weights
        dict(name="serve_n1", kind="serve", dtype="f32", N=1),
        # the LeNet example's training iteration at its batch of 64: many small
        # launches and host calls
        dict(name="lenet_train_n64", kind="train", dtype="f32", N=64),
        # a strided layer on few channels (the image layer of a network), both
        # directions at the training batch
        _conv("conv1_forward_f32", "forward", "f32", 256, conv1),
        _conv("conv1_backward_f32", "backward", "f32", 256, conv1),
        # a grouped 5x5 layer's backward at the training batch: the largest
        # single layer of the network
        _conv("conv2_backward_f32", "backward", "f32", 256, conv2),
        # a 3x3 layer's forward on bfloat16 operands, as the bfloat16 network
        # runs it (float activations in, bfloat16 weights)
        _conv("conv3_forward_bf16", "forward", "bf16_f32in", 512, conv3),
        # the largest layer's backward on bfloat16 operands
        _conv("conv2_backward_bf16", "backward", "bf16", 512, conv2),
        # a small layer none of whose sizes is round, forward and backward
        dict(name="odd_layer_f32", kind="layer", dtype="f32", N=19, C=35, H=45, W=37, K=50, k=3,
             s=1, p=1, g=1, relu=True),
        # the largest inner product, forward and backward: a weight matrix of
        # 151 MB read twice and its gradient written
        _conv("fc6_f32", "fc", "f32", 256, fc6),
        # the bandwidth-bound layers after conv1, both directions
        dict(name="glue_n256", kind="glue", dtype="f32", N=256, C=96, H=55, W=55),
        # the headline: the conv stack's training step, float
        dict(name="step_f32_n256", kind="step", dtype="f32", N=256),
        # the same on bfloat16 operands at twice the batch
        dict(name="step_bf16_n512", kind="step", dtype="bf16", N=512),
    ]


# ------------------------------------------------------------------ drawn cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_conv(rng, kind):
    while True:
        k = rng.choice((1, 3, 3, 3, 5, 5, 7, 11))
        s = rng.choice([v for v in (1, 1, 1, 2, 3, 4) if v <= max(1, k)])
        g = rng.choice((1, 1, 1, 2))
        c = dict(kind=kind, dtype=rng.choice(("f32", "f32", "bf16", "bf16_f32in")),
                 N=_log(rng, 1, 256), C=g * _log(rng, 1, 256), H=_log(rng, 7, 112),
                 W=_log(rng, 7, 112), K=g * _log(rng, 8, 256), k=k, s=s, p=rng.randint(0, k // 2),
                 g=g, relu=rng.random() < 0.7)
        if c["H"] + 2 * c["p"] < k or c["W"] + 2 * c["p"] < k:
            continue
        Ho, Wo = _out(c)
        flops = 2 * c["N"] * c["K"] * Ho * Wo * c["C"] // g * k * k
        blobs = c["N"] * max(c["C"] * c["H"] * c["W"], c["K"] * Ho * Wo)
        if 1e7 <= flops <= 8e10 and blobs <= 5e7:
            return c


def draw(rng):
    kind = rng.choice(("forward", "forward", "backward", "backward", "layer", "fc", "glue",
                       "train", "step", "serve"))
    if kind in ("forward", "backward", "layer"):
        return _draw_conv(rng, kind)
    if kind == "fc":
        return dict(kind="fc", dtype="f32", N=_log(rng, 1, 256), C=_log(rng, 64, 9216), H=1, W=1,
                    K=_log(rng, 10, 4096), k=1, s=1, p=0, g=1, relu=rng.random() < 0.7)
    if kind == "glue":
        return dict(kind="glue", dtype="f32", N=_log(rng, 1, 256), C=_log(rng, 8, 128),
                    H=_log(rng, 9, 80), W=_log(rng, 9, 80))
    if kind == "train":
        return dict(kind="train", dtype="f32", N=_log(rng, 8, 512))
    if kind == "step":
        bf16 = rng.random() < 0.5
        return dict(kind="step", dtype="bf16" if bf16 else "f32",
                    N=_log(rng, 16, 500 if bf16 else 250))
    return dict(kind="serve", dtype="f32", N=_log(rng, 2, 100))


# ------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(gen, shape, std=1.0):
    return torch.randn(shape, generator=gen, device="cuda").mul_(std)


def _out(c):
    return ((c["H"] + 2 * c["p"] - c["k"]) // c["s"] + 1,
            (c["W"] + 2 * c["p"] - c["k"]) // c["s"] + 1)


def _conv_inputs(c, seed):
    """x: mean-subtracted pixels for an image layer (at most 3 channels), else
    post-ReLU activations; w ~ N(0, 0.01) (N(0, 0.005) for the inner products);
    b = 0.1; the output's gradient ~ N(0, 1e-3); the output that the backward
    pass takes its ReLU mask from: a ReLU's, about half of it 0."""
    gen = _gen(seed)
    image = c["C"] <= 3
    x = _randn(gen, (c["N"], c["C"], c["H"], c["W"]), 50.0 if image else 1.0)
    if not image:
        x.abs_()
    w = _randn(gen, (c["K"], c["C"] // c["g"], c["k"], c["k"]), 0.005 if c["kind"] == "fc" else 0.01)
    b = torch.full((c["K"],), 0.1, device="cuda")
    dy = _randn(gen, (c["N"], c["K"]) + _out(c), 1e-3)
    y = _randn(gen, dy.shape).clamp_(min=0.0) if c["kind"] != "forward" and c["relu"] else None
    if c["dtype"] != "f32":
        w = w.to(torch.bfloat16)
    if c["dtype"] == "bf16":
        x = x.to(torch.bfloat16)
    return x, w, b, dy, y


def _net_inputs(layers, N, seed):
    gen = _gen(seed)
    x = _randn(gen, (N, 3, 227, 227), 50.0)
    Ws, bs = [], []
    for L in layers:
        Ws.append(_randn(gen, (L.K, L.C // L.g, L.k, L.k), 0.005 if L.name in ("fc6", "fc7") else 0.01))
        bs.append(torch.full((L.K,), 0.0 if L.name in ("conv1", "fc8") else 0.1, device="cuda"))
    dtop = _randn(gen, (N, layers[-1].K) + layers[-1].out_hw(), 1e-3)
    return x, Ws, bs, dtop


def _lenet_inputs(N, seed):
    gen = _gen(seed)
    x = torch.rand((N, 1, 28, 28), generator=gen, device="cuda")
    labels = torch.randint(0, 10, (N,), generator=gen, device="cuda", dtype=torch.int32)
    Ws = []
    for L in LENET_NET:
        a = math.sqrt(3.0 / (L.C // L.g * L.k * L.k))
        Ws.append(torch.rand((L.K, L.C // L.g, L.k, L.k), generator=gen, device="cuda") * (2 * a) - a)
    return x, labels, Ws, [torch.zeros(L.K, device="cuda") for L in LENET_NET]


def _glue_inputs(c, seed):
    gen = _gen(seed)
    x = _randn(gen, (c["N"], c["C"], c["H"], c["W"]), 30.0).clamp_(min=0.0)  # a ReLU's output
    Ho, Wo = (c["H"] - 3) // 2 + 1, (c["W"] - 3) // 2 + 1
    return x, _randn(gen, (c["N"], c["C"], Ho, Wo), 1e-3)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c}
    if kind in ("forward", "backward", "layer", "fc"):
        x, w, b, dy, y = _conv_inputs(c, seed)
        s.update(x=x, w=w, b=b, dy=dy, y=y, ws=lib.Workspace(x.device))
        if kind != "backward":
            s["top"] = torch.empty_like(dy)
        if kind != "forward":
            s["outs"] = (torch.empty(x.shape, device="cuda"), torch.empty(w.shape, device="cuda"),
                         torch.empty(c["K"], device="cuda"))
    elif kind == "glue":
        s["x"], s["dy"] = _glue_inputs(c, seed)
        s["pooled"], s["out"] = torch.empty_like(s["dy"]), torch.empty_like(s["dy"])
        s["mask"] = torch.empty(s["dy"].shape, dtype=torch.int32, device="cuda")
        s["dx"] = torch.empty_like(s["x"])
    elif kind == "train":
        s["x"], s["labels"], Ws, bs = _lenet_inputs(c["N"], seed)
        net = ConvStack(LENET_NET, c["N"], Ws, bs, LENET_NET_GLUE)
        s["trainer"] = SGDTrainer(net, **LENET_SOLVER)
    elif kind == "step":
        s["x"], Ws, bs, s["dtop"] = _net_inputs(CAFFENET, c["N"], seed)
        s["net"] = ConvStack(CAFFENET, c["N"], Ws, bs, STEP_GLUE, bf16=c["dtype"] == "bf16")
    else:
        s["x"], Ws, bs, _ = _net_inputs(CAFFENET_NET, c["N"], seed)
        s["net"] = ConvStack(CAFFENET_NET, c["N"], Ws, bs, CAFFENET_NET_GLUE)
    return s


# --------------------------------------------------------------------- passes
def run(state):
    c, kind = state["case"], state["case"]["kind"]
    if kind in ("forward", "layer", "fc"):
        top = lib.conv_forward(state["x"], state["w"], state["b"], c["s"], c["p"], c["g"],
                               c["relu"], out=state["top"], ws=state["ws"])
        if kind == "forward":
            return top
    if kind in ("backward", "layer", "fc"):
        dx, dw, db = lib.conv_backward(state["x"], state["w"], state["dy"], state["y"], c["s"],
                                       c["p"], c["g"], c["relu"], outs=state["outs"],
                                       ws=state["ws"])
        if kind == "backward":
            return {"dx": dx, "dw": dw, "db": db}
        return {"top": top, "dx": dx, "dw": dw, "db": db}
    if kind == "glue":
        P, R = CAFFENET_POOL, CAFFENET_LRN
        geometry = (P["kernel"], P["stride"], P["pad"], R["size"], R["alpha"], R["beta"], R["k"])
        lib.pool_lrn_forward(state["x"], *geometry, pooled=state["pooled"], mask=state["mask"],
                             out=state["out"], flags=lib.POOL_RELU_INPUT)
        lib.lrn_pool_backward(state["x"].shape, state["pooled"], state["out"], state["dy"],
                              state["mask"], *geometry, out=state["dx"])
        return {k: state[k] for k in ("pooled", "mask", "out", "dx")}
    if kind == "train":
        t = state["trainer"]
        loss = t.step(state["x"], state["labels"])
        return {"loss": loss, "dW": list(t.net.dW), "db": list(t.net.db), "W": list(t.net.W),
                "b": list(t.net.b)}
    if kind == "step":
        net = state["net"]
        top = net.forward(state["x"])
        net.backward(state["dtop"], data_grad_bottom=False)
        return {"top": top, "dW": list(net.dW), "db": list(net.db)}
    return state["net"].forward(state["x"])


# ----------------------------------------------------------------- accounting
def work(case):
    c, kind = case, case["kind"]
    if kind in ("forward", "backward", "layer", "fc"):
        Ho, Wo = _out(c)
        flops = 2 * c["N"] * c["K"] * Ho * Wo * (c["C"] // c["g"]) * c["k"] ** 2
        x, top = c["N"] * c["C"] * c["H"] * c["W"], c["N"] * c["K"] * Ho * Wo
        w = c["K"] * (c["C"] // c["g"]) * c["k"] ** 2
        xb, wb = (2 if c["dtype"] == "bf16" else 4) * x, (4 if c["dtype"] == "f32" else 2) * w
        # forward: x, w, b -> top; backward: x, w, dy (and the ReLU's top) -> dx, dw, db
        fwd = xb + wb + 4 * (c["K"] + top)
        bwd = xb + wb + 4 * (top * (2 if c["relu"] else 1) + x + w + c["K"])
        return {"bytes": (0 if kind == "backward" else fwd) + (0 if kind == "forward" else bwd),
                "flops": flops * {"forward": 1, "backward": 2}.get(kind, 3)}
    if kind == "glue":
        x = c["N"] * c["C"] * c["H"] * c["W"]
        y = c["N"] * c["C"] * ((c["H"] - 3) // 2 + 1) * ((c["W"] - 3) // 2 + 1)
        # x -> pooled, mask, out; pooled, mask, dy -> dx
        return {"bytes": 4 * (x + 3 * y + 3 * y + x), "flops": 0}
    layers = {"train": LENET_NET, "step": CAFFENET, "serve": CAFFENET_NET}[kind]
    N = c["N"]
    fl = sum(L.flops(N) for L in layers)
    params = sum(L.K * (L.C // L.g) * L.k ** 2 + L.K for L in layers)
    x = N * layers[0].C * layers[0].H * layers[0].W
    Ho, Wo = layers[-1].out_hw()
    top = N * layers[-1].K * Ho * Wo
    if kind == "serve":
        return {"bytes": 4 * (x + params + top), "flops": fl}
    flops = 3 * fl - layers[0].flops(N)  # no gradient of the input images
    if kind == "train":  # images, labels; weights and histories read and written, gradients written
        return {"bytes": 4 * (x + N + 5 * params), "flops": flops}
    return {"bytes": 4 * (x + 2 * top + params) + (2 if c["dtype"] == "bf16" else 4) * params,
            "flops": flops}


def tolerance(case):
    """About four times what the same sums in another order, or in 64 bits, differ
    by (measured: single layers up to 7e-7, the glue 5e-8, the network's scores
    3e-7).  In the training cases a rounding difference can turn a max-pool's
    winner or a ReLU's side, which moves single gradients: two orders of the
    float step's sums differ by 2e-3 in a weight gradient, of the bfloat16
    step's backward sums alone by 1e-3."""
    kind = case["kind"]
    if kind == "glue":
        return {"rel": 4e-7, "max": 4e-5}
    if kind == "train":
        return {"rel": 4e-3, "max": 0.2}
    if kind == "step":
        return {"rel": 1e-2, "max": 0.3}
    return {"rel": 4e-6, "max": 2e-4}


# -------------------------------------------------- the same in 64-bit torch
def _cols64(x, c):
    """im2col of a few images in float64: per group (Cg k k, n Ho Wo)."""
    u = F.unfold(x, c["k"], padding=c["p"], stride=c["s"])  # (n, C k k, Ho Wo)
    n, _, hw = u.shape
    u = u.view(n, c["g"], -1, hw)
    return [u[:, t].permute(1, 0, 2).reshape(u.shape[2], n * hw) for t in range(c["g"])]


def _chunks(c):
    Ho, Wo = _out(c)
    per_image = 8 * c["C"] * c["k"] ** 2 * Ho * Wo
    n = max(1, int(1e9) // per_image)
    return [(i, min(c["N"], i + n)) for i in range(0, c["N"], n)]


def _conv64(x, w, b, c):
    Ho, Wo = _out(c)
    Kg = c["K"] // c["g"]
    w64 = w.double().view(c["g"], Kg, -1)
    top = torch.empty((c["N"], c["K"], Ho, Wo), dtype=torch.float64, device=x.device)
    for i, j in _chunks(c):
        for t, cols in enumerate(_cols64(x[i:j].double(), c)):
            z = (w64[t] @ cols).view(Kg, j - i, Ho, Wo).permute(1, 0, 2, 3)
            top[i:j, t * Kg:(t + 1) * Kg] = z + b.double()[t * Kg:(t + 1) * Kg].view(1, -1, 1, 1)
    return top.clamp_(min=0.0) if c["relu"] else top


def _conv64_backward(x, w, dy, y, c):
    """(dx, dw, db); with bfloat16 operands the masked gradient enters the
    products rounded to bfloat16, and the bias gradient unrounded."""
    Kg, Cg = c["K"] // c["g"], c["C"] // c["g"]
    D = dy * (y > 0) if c["relu"] else dy
    db = D.double().sum((0, 2, 3))
    if c["dtype"] != "f32":
        D = D.to(torch.bfloat16)
    w64 = w.double().view(c["g"], Kg, -1)
    dw = torch.zeros_like(w64)
    dx = torch.empty(x.shape, dtype=torch.float64, device=x.device)
    for i, j in _chunks(c):
        n = j - i
        D64 = D[i:j].double().view(n, c["g"], Kg, -1)
        parts = []
        for t, cols in enumerate(_cols64(x[i:j].double(), c)):
            d = D64[:, t].permute(1, 0, 2).reshape(Kg, -1)
            dw[t] += d @ cols.t()
            parts.append((w64[t].t() @ d).view(Cg * c["k"] ** 2, n, -1).permute(1, 0, 2))
        dx[i:j] = F.fold(torch.cat(parts, 1).contiguous(), (c["H"], c["W"]), c["k"],
                         padding=c["p"], stride=c["s"])
    return dx, dw.view(w.shape), db


def _lrn64(x):
    n, alpha, beta, k = (CAFFENET_LRN[v] for v in ("size", "alpha", "beta", "k"))
    sq = F.pad(x.square(), (0, 0, 0, 0, (n - 1) // 2, n - 1 - (n - 1) // 2))
    C = x.shape[1]
    scale = k + alpha / n * sum(sq[:, i:i + C] for i in range(n))
    return x * scale ** -beta, scale


def _lrn64_backward(x, y, scale, dy):
    n, alpha, beta = (CAFFENET_LRN[v] for v in ("size", "alpha", "beta"))
    r = F.pad(dy * y / scale, (0, 0, 0, 0, n - 1 - (n - 1) // 2, (n - 1) // 2))
    C = x.shape[1]
    return dy * scale ** -beta - 2 * alpha * beta / n * x * sum(r[:, i:i + C] for i in range(n))


def _forward64(layers, glue, x, Ws, bs, bf16=False):
    """The chain's last output; with bfloat16 operands each convolution's input
    and weights are rounded to bfloat16, as the library documents."""
    cur = x.double()
    for l, L in enumerate(layers):
        c = dict(N=x.shape[0], C=L.C, H=L.H, W=L.W, K=L.K, k=L.k, s=L.s, p=L.p, g=L.g, relu=L.relu)
        cur, w = cur.reshape(c["N"], L.C, L.H, L.W), Ws[l]
        if bf16:
            cur, w = cur.to(torch.bfloat16), w.to(torch.bfloat16)
        cur = _conv64(cur, w, bs[l], c)
        for what, prm in glue.get(l, ()):
            if what == "pool":
                cur = F.max_pool2d(cur, prm["kernel"], prm["stride"])
            else:
                cur = _lrn64(cur)[0]
    return cur


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("forward", "backward", "layer", "fc"):
        x, w, b, dy, y = _conv_inputs(c, seed)
        if c["dtype"] == "bf16_f32in":
            x = x.to(torch.bfloat16)
        if kind == "forward":
            return _conv64(x, w, b, c)
        dx, dw, db = _conv64_backward(x, w, dy, y, c)
        if kind == "backward":
            return {"dx": dx, "dw": dw, "db": db}
        return {"top": _conv64(x, w, b, c), "dx": dx, "dw": dw, "db": db}
    if kind == "glue":
        x, dy = _glue_inputs(c, seed)
        pooled, at = F.max_pool2d(x, 3, 2, return_indices=True)
        won = pooled > 0  # a window without a positive value has no winner
        p64 = pooled.double()
        y, scale = _lrn64(p64)
        dp = _lrn64_backward(p64, y, scale, dy.double())
        dx = torch.zeros((c["N"], c["C"], c["H"] * c["W"]), dtype=torch.float64, device=x.device)
        dx.scatter_add_(2, at.flatten(2), (dp * won).flatten(2))
        return {"pooled": p64, "mask": None, "out": y, "dx": dx.view(x.shape)}
    if kind == "train":
        x, labels, Ws, bs = _lenet_inputs(c["N"], seed)
        z = _forward64(LENET_NET, LENET_NET_GLUE, x, Ws, bs).flatten(1)
        loss = F.cross_entropy(z, labels.long()).reshape(1)
        # the gradients (and the weights they update) jump where rounding
        # decides a max-pool's winner or a ReLU's side
        none = [None] * len(LENET_NET)
        return {"loss": loss, "dW": none, "db": none, "W": none, "b": none}
    if kind == "step":
        x, Ws, bs, _ = _net_inputs(CAFFENET, c["N"], seed)
        top = _forward64(CAFFENET, STEP_GLUE, x, Ws, bs, c["dtype"] == "bf16")
        none = [None] * len(CAFFENET)  # (as for LeNet's)
        return {"top": top, "dW": none, "db": none}
    x, Ws, bs, _ = _net_inputs(CAFFENET_NET, c["N"], seed)
    return _forward64(CAFFENET_NET, CAFFENET_NET_GLUE, x, Ws, bs)
