"""The work a user of this library has it do, as cases that can be timed.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same
ranges, ``prepare(case, seed)`` builds on the GPU what a user's program holds
before the call, and ``run(state)`` is one pass through the public entry
points (``paper_1603_07846_amd.net.Net`` and the operators of
``paper_1603_07846_amd.singa``).  ``work`` is what a pass cannot do without,
``exact`` the same results in 64 bits by plain torch.

Kinds of case:
  step      one training step of a whole network (``Net.train_one_batch``)
  conv      one convolution layer: forward with bias and ReLU and, when it
            trains, the source gradient (with the ReLU backward of the layer
            below folded in, unless it is the first layer) and the parameter
            gradients
  fc        one fully connected layer: forward and, when it trains, the source
            gradient and the parameter gradients with the SGD step
  normpool  response normalization and 3x3/2 max pooling, forward and backward
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_1603_07846_amd import net as gnet
from paper_1603_07846_amd import singa
from paper_1603_07846_amd import workloads as wl

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _conv(name, dtype, n, c, h, w, k, r, pad, stride=1, first=False, train=True, layout="NHWC"):
    return {"name": name, "kind": "conv", "dtype": dtype, "n": n, "c": c, "h": h, "w": w, "k": k, "r": r, "pad": pad,
            "stride": stride, "first": first, "train": train, "layout": layout}


def _fc(name, dtype, n, c, h, k, relu, train):
    return {"name": name, "kind": "fc", "dtype": dtype, "n": n, "c": c, "h": h, "k": k, "relu": relu, "train": train}


def listed():
    return [
        # The benchmark's workload: the AlexNet-shaped training step in bf16 at
        # the batch a single GPU trains with.
        {"name": "step_alexnet_b256", "kind": "step", "workload": 5, "n": 256, "updater": "sgd"},
        # The full network with response normalization at the share that each
        # of eight workers gets of a batch of 256.
        {"name": "step_alexnet_lrn_b32", "kind": "step", "workload": 6, "n": 32, "updater": "sgd"},
        # The CIFAR-10-shaped network in fp32 at its own batch: a short step of
        # many small layers, where launches count.
        {"name": "step_cifar_b100", "kind": "step", "workload": 2, "n": 100, "updater": "sgd"},
        # The single-layer workload: a first layer on a handful of small images,
        # the smallest training call there is.
        _conv("conv_5x5_f32_b16", "f32", 16, 3, 32, 32, 32, 5, 2, first=True),
        # A strided first layer on colour images of ImageNet's size.
        _conv("conv_11x11s4_bf16_b128", "bf16", 128, 3, 227, 227, 96, 11, 0, 4, first=True),
        # The layer with most of the multiply-adds, at a quarter of the batch.
        _conv("conv_5x5_bf16_b64", "bf16", 64, 96, 27, 27, 256, 5, 2),
        # A deep 3x3 layer at a batch that is no multiple of a tile.
        _conv("conv_3x3_bf16_b100", "bf16", 100, 384, 13, 13, 384, 3, 1),
        # The same kind of layer in fp32, as the fp32 convolution stack runs it.
        _conv("conv_3x3_f32_b32", "f32", 32, 256, 13, 13, 384, 3, 1),
        # Caffe's layout: a program that keeps NCHW activations.
        _conv("conv_3x3_nchw_bf16_b50", "bf16", 50, 64, 28, 28, 128, 3, 1, layout="NCHW"),
        # The largest fully connected layer, trained at half the batch.
        _fc("fc_9216_4096_bf16_b128", "bf16", 128, 256, 6, 4096, True, True),
        # One image through a fully connected layer: prediction, latency counts.
        _fc("fc_4096_4096_bf16_b1", "bf16", 1, 4096, 1, 4096, True, False),
        # The bandwidth-bound layers between the first two convolutions.
        {"name": "normpool_bf16_b64", "kind": "normpool", "dtype": "bf16", "n": 64, "c": 96, "h": 55, "size": 5},
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread evenly over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("conv", "fc", "normpool", "step"), (10, 4, 2, 4))[0]
    if kind == "step":
        workload = rng.choice((2, 5, 6))
        n = _log(rng, 10, 400) if workload == 2 else _log(rng, 4, 200)
        return {"kind": "step", "workload": workload, "n": n, "updater": rng.choice(("sgd", "sgd", "sgd", "adagrad"))}
    dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
    if kind == "normpool":
        return {"kind": "normpool", "dtype": dtype, "n": _log(rng, 2, 96), "c": 8 * _log(rng, 4, 32),
                "h": rng.randint(13, 55), "size": rng.choice((5, 5, 3))}
    if kind == "fc":
        h = rng.choice((1, 1, 4, 6))
        c = 8 * _log(rng, 8, 32) if h > 1 else 8 * _log(rng, 32, 512)
        k = rng.choice((10, 100, 1000, 4096, 8 * _log(rng, 8, 512)))
        case = _fc("", dtype, _log(rng, 1, 256), c, h, k, rng.random() < 0.7, rng.random() < 0.7)
        del case["name"]
        return case
    first = rng.random() < 0.2
    while True:
        r = rng.choice((1, 3, 3, 3, 5, 5, 7, 11) if first else (1, 3, 3, 3, 3, 5, 5))
        stride = rng.choice((1, 2, 4)) if first else rng.choice((1, 1, 1, 1, 1, 2))
        h = rng.randint(24, 230) if first else rng.randint(7, 57)
        w = h if rng.random() < 0.7 else max(r, h + rng.randint(-5, 5))
        c = rng.choice((1, 3, 3, 3)) if first else 8 * _log(rng, 2, 64)
        k = 8 * _log(rng, 2, 64)
        if not first and rng.random() < 0.1:  # channel counts that are no multiple of a vector
            c, k = c + rng.randint(1, 7), k + rng.randint(1, 7)
        pad = rng.choice((0, r // 2, r // 2))
        layout = "NCHW" if rng.random() < 0.2 else "NHWC"
        case = _conv("", dtype, _log(rng, 1, 256), c, h, w, k, r, pad, stride, first, rng.random() < 0.8, layout)
        del case["name"]
        if stride > r or min(h, w) + 2 * pad < r:
            continue
        limit = 2e11 if dtype == "bf16" and c % 8 == 0 and k % 8 == 0 else 4e10
        x, y = case["n"] * c * h * w, case["n"] * k * math.prod(_out(case))
        if work(case)["flops"] <= limit and max(x, y) <= 5e7:
            return case


# ----------------------------------------------------------------- inputs


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, shape, std=1.0):
    return torch.randn(shape, generator=g, device="cuda") * std


def _relu_grad(g, shape, std):
    """A gradient that has come through a ReLU's backward: about half zeros."""
    return _normal(g, shape, std) * (torch.rand(shape, generator=g, device="cuda") < 0.5)


def _out(case):
    return tuple((case[a] + 2 * case["pad"] - case["r"]) // case["stride"] + 1 for a in ("h", "w"))


def _conv_inputs(case, seed):
    """x, w, bias, dy of a convolution layer in its layout.  x is the output
    of a ReLU, except the images of a first layer."""
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    n, c, h, w, k, r = (case[a] for a in ("n", "c", "h", "w", "k", "r"))
    p, q = _out(case)
    nchw = case["layout"] == "NCHW"
    x = _normal(g, (n, c, h, w) if nchw else (n, h, w, c))
    x = (x if case["first"] else x.clamp_min(0)).to(dt)
    wt = _normal(g, (k, c, r, r) if nchw else (k, r, r, c), math.sqrt(2 / (c * r * r))).to(dt)
    b = _normal(g, (k,), 0.1)
    dy = _relu_grad(g, (n, k, p, q) if nchw else (n, p, q, k), 0.01).to(dt)
    return x, wt, b, dy


def _fc_inputs(case, seed):
    """x, master weights and momentum, bias and its momentum, dy."""
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    n, c, h, k = (case[a] for a in ("n", "c", "h", "k"))
    x = _normal(g, (n, h, h, c)).clamp_min(0).to(dt)
    fan = c * h * h
    w = _normal(g, (k, h, h, c), math.sqrt(2 / fan))
    v = _normal(g, (k, h, h, c), 1e-3 / math.sqrt(fan))
    b, vb = _normal(g, (k,), 0.1), _normal(g, (k,), 1e-3)
    dy = (_relu_grad if case["relu"] else _normal)(g, (n, 1, 1, k), 0.01).to(dt)
    return x, w, v, b, vb, dy


FC_STEP = dict(lr=0.01, momentum=0.9, weight_decay=5e-4)


def _normpool_inputs(case, seed):
    """x (the output of a ReLU) and the gradient at the pooling's output."""
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    n, c, h = case["n"], case["c"], case["h"]
    p = -(-(h - 3) // 2) + 1
    return _normal(g, (n, h, h, c)).clamp_min(0).to(dt), _normal(g, (n, p, p, c), 0.01).to(dt)


def _step_inputs(case, seed):
    """Images, labels and, per layer with parameters, its weights, bias and
    updater state (momentum, or AdaGrad's sums of squares) as (w, b, v, vb)
    in the filter layout KRSC."""
    g, spec = _gen(seed), wl.WORKLOADS[case["workload"]]
    n, (c, h, w_) = case["n"], spec.in_shape
    x = (torch.rand((n, h, w_, c), generator=g, device="cuda") if spec.input_dist == "uniform01"
         else _normal(g, (n, h, w_, c)))
    labels = torch.randint(0, spec.classes, (n,), generator=g, device="cuda").to(torch.int32)
    params = []
    for l in spec.layers:
        if isinstance(l, (wl.Conv, wl.FC)):
            fc = isinstance(l, wl.FC)
            k, r, s = (l.out_features, h, w_) if fc else (l.out_channels, l.kernel, l.kernel)
            fan = r * s * c
            wt = _normal(g, (k, r, s, c), math.sqrt(2 / fan))
            b = torch.zeros(k, device="cuda")
            v, vb = _normal(g, (k, r, s, c), 1e-2 / math.sqrt(fan)), _normal(g, (k,), 1e-2)
            if case["updater"] == "adagrad":
                v, vb = v.square(), vb.square()
            params.append((wt, b, v, vb))
        if isinstance(l, (wl.Conv, wl.FC, wl.Pool)):
            c, h, w_ = l.out_shape
    return x.to(DTYPES[spec.dtype]), labels, params


# ------------------------------------------------------------- prepare, run


def _workspace(*sizes):
    return torch.empty(max(256, *sizes), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        spec = wl.WORKLOADS[case["workload"]]
        x, labels, params = _step_inputs(case, seed)
        net = gnet.Net(spec, batch=case["n"], device="cuda", updater=case["updater"])
        for l, (w, b, v, vb) in zip(net.param_layers(), params):
            l.w.copy_(w)
            l.b.copy_(b)
            l.v.copy_(v)
            l.vb.copy_(vb)
        if net.wb_flat is not None:
            net.wb_flat.copy_(net.w_flat)
        return {"kind": kind, "net": net, "x": x, "labels": labels}
    if kind == "conv":
        x, w, b, dy = _conv_inputs(case, seed)
        xs, ws, how = tuple(x.shape), tuple(w.shape), (case["pad"], case["stride"], case["layout"])
        ops = [singa.OP_FWD]
        if case["train"]:
            ops += [singa.OP_BWD_FILTER] + ([] if case["first"] else [singa.OP_BWD_DATA])
        return {"kind": kind, "case": case, "x": x, "w": w, "b": b, "dy": dy, "y": torch.empty_like(dy),
                "dx": torch.empty_like(x), "dw": torch.empty(ws, device="cuda"), "db": torch.empty_like(b),
                "ws": _workspace(*(singa.conv_workspace_bytes(op, x.dtype, xs, ws, *how) for op in ops))}
    if kind == "fc":
        x, w, v, b, vb, dy = _fc_inputs(case, seed)
        xs, ws = tuple(x.shape), tuple(w.shape)
        ops = [singa.OP_FWD] + ([singa.OP_BWD_DATA, singa.OP_BWD_FILTER_SGD] if case["train"] else [])
        bf16 = x.dtype == torch.bfloat16
        return {"kind": kind, "case": case, "x": x, "w": w, "v": v, "b": b, "vb": vb, "dy": dy,
                "wb": w.to(x.dtype) if bf16 else None, "bb": b.to(x.dtype) if bf16 else None,
                "y": torch.empty_like(dy), "dx": torch.empty_like(x),
                "ws": _workspace(*(singa.conv_workspace_bytes(op, x.dtype, xs, ws) for op in ops))}
    x, dy = _normpool_inputs(case, seed)
    return {"kind": kind, "size": case["size"], "x": x, "dy": dy, "h": torch.empty_like(x), "y": torch.empty_like(dy),
            "argmax": torch.empty(dy.shape, dtype=torch.uint8, device="cuda"), "dh": torch.empty_like(x),
            "dx": torch.empty_like(x)}


def run(s):
    kind = s["kind"]
    if kind == "step":
        net = s["net"]
        net.train_one_batch(s["x"], s["labels"])
        out = {"loss": net.layers[-1].loss, "logits": net.layers[-2].y, "w": net.w_flat, "v": net.v_flat}
        if net.wb_flat is not None:
            out["w_bf16"] = net.wb_flat
        return out
    if kind == "conv":
        case, x, w, dy, ws = s["case"], s["x"], s["w"], s["dy"], s["ws"]
        how = dict(pad=case["pad"], stride=case["stride"], layout=case["layout"], workspace=ws)
        out = {"y": singa.conv_fwd(x, w, s["b"], relu=True, out=s["y"], **how)}
        if case["train"]:
            if not case["first"]:
                out["dx"] = singa.conv_bwd_data(dy, w, tuple(x.shape), out=s["dx"], relu_y=x, **how)
            out["dw"], out["db"] = singa.conv_bwd_filter(x, dy, tuple(w.shape), dw=s["dw"], db=s["db"], **how)
        return out
    if kind == "fc":
        case, x, w, dy, ws = s["case"], s["x"], s["w"], s["dy"], s["ws"]
        wc = w if s["wb"] is None else s["wb"]
        out = {"y": singa.conv_fwd(x, wc, s["b"], relu=case["relu"], out=s["y"], workspace=ws)}
        if case["train"]:
            out["dx"] = singa.conv_bwd_data(dy, wc, tuple(x.shape), out=s["dx"], relu_y=x, workspace=ws)
            singa.conv_bwd_filter_sgd(x, dy, tuple(w.shape), w, s["v"], s["wb"], s["b"], s["vb"], s["bb"],
                                      workspace=ws, **FC_STEP)
            out.update(w=w, v=s["v"], b=s["b"], vb=s["vb"])
            if s["wb"] is not None:
                out.update(wb=s["wb"], bb=s["bb"])
        return out
    size = s["size"]
    h = singa.lrn_fwd(s["x"], size=size, out=s["h"])
    y, argmax = singa.pool_fwd(h, "max", out=s["y"], argmax=s["argmax"])
    dh = singa.pool_bwd(s["dy"], argmax, tuple(h.shape), "max", out=s["dh"])
    dx = singa.lrn_bwd(s["x"], dh, size=size, out=s["dx"])
    return {"h": h, "y": y, "argmax": argmax, "dh": dh, "dx": dx}


# ------------------------------------------------------- work and tolerance


def work(case):
    kind = case["kind"]
    if kind == "step":
        spec, n = wl.WORKLOADS[case["workload"]], case["n"]
        es = 2 if spec.dtype == "bf16" else 4
        c, h, w = spec.in_shape
        nbytes, flops, first = n * c * h * w * es, 0, True
        for l in spec.layers:
            if isinstance(l, (wl.Conv, wl.FC)):
                taps = c * l.kernel * l.kernel if isinstance(l, wl.Conv) else c * h * w
                k, p, q = l.out_shape
                # forward, parameter gradients and (not below the first layer) the source gradient
                flops += 2 * n * k * p * q * taps * (2 if first else 3)
                # master weights and updater state read and written, the bf16 copy read and written
                nbytes += (taps * k + k) * (16 + (4 if es == 2 else 0))
                first = False
            if isinstance(l, (wl.Conv, wl.FC, wl.Pool)):
                c, h, w = l.out_shape
        return {"bytes": nbytes + n * spec.classes * es, "flops": flops}
    es = 2 if case["dtype"] == "bf16" else 4
    if kind == "conv":
        n, c, h, w, k, r = (case[a] for a in ("n", "c", "h", "w", "k", "r"))
        p, q = _out(case)
        x, f, y, macs = n * c * h * w, k * r * r * c, n * p * q * k, n * p * q * k * r * r * c
        nbytes, passes = (x + f + y) * es, 1
        if case["train"]:
            passes += 1 if case["first"] else 2
            nbytes += y * es + f * 4 + (0 if case["first"] else x * es)
        return {"bytes": nbytes, "flops": 2 * macs * passes}
    if kind == "fc":
        n, j, k = case["n"], case["c"] * case["h"] ** 2, case["k"]
        nbytes, flops = (n * j + n * k + j * k) * es, 2 * n * j * k
        if case["train"]:
            nbytes += (n * j + n * k) * es + j * k * (18 if es == 2 else 12)
            flops *= 3
        return {"bytes": nbytes, "flops": flops}
    n, c, h = case["n"], case["c"], case["h"]
    p = -(-(h - 3) // 2) + 1
    x, y = n * c * h * h, n * c * p * p
    # x, the normalized blob and its gradient, dx; the pooling's output, arg-max and gradient
    return {"bytes": 4 * x * es + 2 * y * es + y, "flops": 0}


def tolerance(case):
    if case["kind"] == "step":
        return {"rel": 3e-2, "max": 0.9} if case["workload"] != 2 else {"rel": 1e-4, "max": 1e-2}
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 5e-2}
    return {"rel": 1e-5, "max": 1e-4}


# ------------------------------------------------------------------- exact


def _nchw(t):
    return t.double().permute(0, 3, 1, 2)


def _nhwc(t):
    return t.detach().permute(0, 2, 3, 1)


def _exact_conv(case, seed):
    x, w, b, dy = _conv_inputs(case, seed)
    if case["layout"] == "NHWC":
        x, w, dy = _nchw(x), _nchw(w), _nchw(dy)
    x, w, b, dy = (t.double().contiguous() for t in (x, w, b, dy))
    back = _nhwc if case["layout"] == "NHWC" else (lambda t: t.detach())
    y, dx, dw = [], [], torch.zeros_like(w)
    for i in range(0, x.shape[0], 32):
        xi = x[i:i + 32].clone().requires_grad_(not case["first"])
        wi = w.clone().requires_grad_()
        z = F.conv2d(xi, wi, b, case["stride"], case["pad"])
        y.append(z.detach().clamp_min(0))
        if case["train"]:
            z.backward(dy[i:i + 32])
            dw += wi.grad
            if not case["first"]:
                dx.append(xi.grad * (x[i:i + 32] > 0))
    out = {"y": back(torch.cat(y))}
    if case["train"]:
        if not case["first"]:
            out["dx"] = back(torch.cat(dx))
        out["dw"], out["db"] = back(dw), dy.sum((0, 2, 3))
    return out


def _sgd(w, v, g, lr, momentum, weight_decay):
    v = momentum * v + lr * (g + weight_decay * w)
    return w - v, v


def _exact_fc(case, seed):
    x, w, v, b, vb, dy = _fc_inputs(case, seed)
    xf, wc = x.double().flatten(1), w.to(x.dtype).double().flatten(1)
    dyf = dy.double().flatten(1)
    y = xf @ wc.T + b.double()
    out = {"y": (y.clamp_min(0) if case["relu"] else y).view(dy.shape)}
    if case["train"]:
        out["dx"] = ((dyf @ wc) * (xf > 0)).view(x.shape)
        w2, v2 = _sgd(w.double(), v.double(), (dyf.T @ xf).view(w.shape), **FC_STEP)
        b2, vb2 = _sgd(b.double(), vb.double(), dyf.sum(0), **FC_STEP)
        out.update(w=w2, v=v2, b=b2, vb=vb2)
        if x.dtype == torch.bfloat16:
            out.update(wb=w2, bb=b2)
    return out


def _exact_normpool(case, seed):
    x, dy = _normpool_inputs(case, seed)
    x = _nchw(x).contiguous().requires_grad_()
    # arg-maxes and the pooled values are taken on the normalized blob as it is stored
    h = F.local_response_norm(x, case["size"], 1e-4, 0.75, 1.0)
    stored = h.detach().to(DTYPES[case["dtype"]]).double().requires_grad_()
    y = F.max_pool2d(stored, 3, 2, ceil_mode=True)
    y.backward(_nchw(dy).contiguous())
    h.backward(stored.grad)
    return {"h": _nhwc(h), "y": _nhwc(y), "argmax": None, "dh": _nhwc(stored.grad), "dx": _nhwc(x.grad)}


def _exact_step(case, seed):
    spec = wl.WORKLOADS[case["workload"]]
    x, labels, params = _step_inputs(case, seed)
    bf16 = spec.dtype == "bf16"
    compute = [_nchw(w.to(x.dtype)).contiguous().requires_grad_() for w, _, _, _ in params]
    biases = [b.double().requires_grad_() for _, b, _, _ in params]
    loss_rows, logits = [], []
    for i in range(0, case["n"], 64):
        h, at = _nchw(x[i:i + 64]).contiguous(), 0
        for l in spec.layers:
            if isinstance(l, wl.Conv):
                h = F.conv2d(h, compute[at], biases[at], l.stride, l.pad)
                at += 1
            elif isinstance(l, wl.FC):
                h = (h.flatten(1) @ compute[at].flatten(1).T + biases[at])[:, :, None, None]
                at += 1
            elif isinstance(l, wl.Relu):
                h = h.clamp_min(0)
            elif isinstance(l, wl.Lrn):
                h = F.local_response_norm(h, l.size, l.alpha, l.beta, l.k)
            elif isinstance(l, wl.Pool):
                pool = F.max_pool2d if l.mode == "max" else F.avg_pool2d
                h = pool(h, l.kernel, l.stride, l.pad, ceil_mode=l.ceil_mode)
        rows = F.cross_entropy(h.flatten(1), labels[i:i + 64].long(), reduction="none")
        (rows.sum() / case["n"]).backward()
        loss_rows.append(rows.detach())
        logits.append(h.detach())
    rows = torch.cat(loss_rows)
    w_flat, v_flat = [], []

    def put(w, v, g):
        w, v = w.double(), v.double()
        if case["updater"] == "adagrad":
            g = g + spec.weight_decay * w
            v = v + g * g
            w = w - spec.lr * g / (1e-6 + v.sqrt())
        else:
            w, v = _sgd(w, v, g, spec.lr, spec.momentum, spec.weight_decay)
        gap = torch.zeros(-w.numel() % 64, dtype=w.dtype, device=w.device)  # the flat buffers' padding
        w_flat.extend((w.flatten(), gap))
        v_flat.extend((v.flatten(), gap))

    for (w, b, v, vb), wc, bc in zip(params, compute, biases):
        put(w, v, _nhwc(wc.grad))
        put(b, vb, bc.grad)
    w, v = torch.cat(w_flat), torch.cat(v_flat)
    out = {"loss": torch.cat((rows.mean()[None], rows)), "logits": _nhwc(torch.cat(logits)), "w": w, "v": v}
    if bf16:
        out["w_bf16"] = w
    return out


def exact(case, seed):
    """What run() returns for these inputs, in 64 bits by plain torch."""
    how = {"step": _exact_step, "conv": _exact_conv, "fc": _exact_fc, "normpool": _exact_normpool}
    return how[case["kind"]](case, seed)
