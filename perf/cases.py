"""Timing cases of the Parle training step: what they run, their inputs, their work and their tolerances.

A case is a dict of plain values.  `kind` names the part of the path it runs:

* ``step``    one inner step of a network (forward, loss, backward, fused update) through ``Parle.parle_inner_step``
* ``eval``    loss, errors and spread at the reference through ``Parle.parle_eval``
* ``conv``    one convolutional or fully connected layer as a training step runs it: forward, input gradient, weight
              (and bias) gradient, through the ``parle_k_conv_*`` entry points
* ``bn``      one batch-norm + ReLU layer, forward and backward, through ``parle_k_bn_*``
* ``update``  the fused update of a flat parameter vector through ``Parle.parle_inner_step`` (and, with ``outer``, the
              replica mean and outer update behind it)

``prepare`` makes inputs and contexts on the GPU, ``run`` is one pass, ``exact`` the same results from plain torch in
64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_1707_00424_amd import binding as pb
from paper_1707_00424_amd import synth

DEVICE = "cuda:0"

MODELS = {
    # name: (library model, weight initialisation, image side, image channels)
    "mlp": (pb.MODEL_MLP, "uniform", 28, 1),
    "lenet": (pb.MODEL_LENET, "uniform", 28, 1),
    "allcnn": (pb.MODEL_ALLCNN_C, "he_normal", 32, 3),
    "wrn": (pb.MODEL_WRN, "he_normal", 32, 3),
}
CLASSES = 10


def listed():
    return [
        # The 784-128-10 network of the small workload: the shortest step there is, all launches and latency.
        dict(name="mlp_step_f32", kind="step", model="mlp", bf16=False, n=3, batch=128, arch0=128, arch1=0, arch2=0, arch3=0),
        # LeNet with six replicas, fp32: small contractions of odd sizes (20 and 50 channels, 5x5 windows).
        dict(name="lenet_step_f32", kind="step", model="lenet", bf16=False, n=6, batch=128, arch0=20, arch1=50, arch2=5, arch3=500),
        # All-CNN-C with three replicas, bf16 compute: the whole training step of a convolutional network.
        dict(name="allcnn_step_bf16", kind="step", model="allcnn", bf16=True, n=3, batch=128, arch0=96, arch1=192, arch2=0, arch3=0),
        # Evaluation of the averaged model between outer steps (WRN-16-4): forward only, one row of parameters.
        dict(name="wrn16_4_eval_bf16", kind="eval", model="wrn", bf16=True, n=3, batch=128, arch0=16, arch1=4, arch2=2, arch3=0,
             count=384),
        # All-CNN-C's second convolution: full resolution, 96 channels, bias and ReLU.
        dict(name="conv3x3_96_bf16", kind="conv", bf16=True, n=3, batch=128, h=32, w=32, cin=96, cout=96, k=3, stride=1,
             pad=1, bias=True),
        # A middle layer of WRN-28-10: the largest contractions the framework's networks have.
        dict(name="conv3x3_320_bf16", kind="conv", bf16=True, n=3, batch=128, h=16, w=16, cin=320, cout=320, k=3, stride=1,
             pad=1, bias=False),
        # The convolution that opens group 2 of WRN-16-4: halves the resolution and doubles the width.
        dict(name="conv3x3_s2_bf16", kind="conv", bf16=True, n=3, batch=128, h=32, w=32, cin=64, cout=128, k=3, stride=2,
             pad=1, bias=False),
        # A convolution of the same networks on 28x28 images, one replica (Entropy-SGD) and a batch of 100: image rows that
        # are no power of two.
        dict(name="conv3x3_28px_bf16", kind="conv", bf16=True, n=1, batch=100, h=28, w=28, cin=96, cout=96, k=3, stride=1,
             pad=1, bias=True),
        # All-CNN-C's second convolution in the default compute type.
        dict(name="conv3x3_96_f32", kind="conv", bf16=False, n=3, batch=128, h=32, w=32, cin=96, cout=96, k=3, stride=1,
             pad=1, bias=True),
        # LeNet's first fully connected layer, six replicas.
        dict(name="fc_800_500_f32", kind="conv", bf16=False, n=6, batch=128, h=1, w=1, cin=800, cout=500, k=1, stride=1,
             pad=0, bias=True),
        # Batch-norm + ReLU of a residual block at full resolution (WRN-16-4), with the identity shortcut's gradient.
        dict(name="bn_relu_64_bf16", kind="bn", bf16=True, n=3, batch=128, h=32, w=32, c=64, add=True),
        # The update-only workload: eight replicas of a WRN-28-10-sized vector.
        dict(name="update_flat_f32", kind="update", n=8, params=36_500_000, outer=False),
    ]


# A drawn case does no more work of its kind than the largest listed one (for convolutions: than the largest of any
# type, since odd sizes run at a lower rate).
CONV_FLOPS_CAP = 1.9e11
BN_BYTES_CAP = 3.5e8
UPDATE_CAP = 8 * 36_500_000


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "conv", "conv", "conv", "conv", "fc", "bn", "update", "eval"])
    if kind in ("step", "eval"):
        model = rng.choice(["mlp", "lenet", "allcnn"]) if kind == "step" else rng.choice(["mlp", "lenet", "allcnn", "wrn"])
        case = dict(kind=kind, model=model, bf16=model in ("allcnn", "wrn"), n=rng.randint(1, 6 if model in ("mlp", "lenet") else 3),
                    batch=_log_int(rng, 16, 128), arch0=0, arch1=0, arch2=0, arch3=0)
        if model == "mlp":
            case.update(arch0=_log_int(rng, 32, 512))
        elif model == "lenet":
            case.update(arch0=rng.choice([12, 16, 20]), arch1=rng.choice([32, 40, 50]), arch2=5, arch3=_log_int(rng, 64, 500))
        elif model == "allcnn":
            ca = rng.choice([32, 48, 64, 96])
            case.update(arch0=ca, arch1=2 * ca)
        else:
            case.update(arch0=16, arch1=rng.choice([1, 2, 4]), arch2=rng.choice([1, 2]))
        if kind == "eval":
            case["count"] = rng.randint(1, case["n"] * case["batch"])
        return case
    if kind == "conv":
        bf16 = rng.random() < 0.6
        while True:
            side = rng.choice([7, 8, 12, 14, 15, 16, 24, 28, 32])
            k = rng.choice([1, 3, 3, 3, 5])
            case = dict(kind="conv", bf16=bf16, n=rng.randint(1, 8), batch=_log_int(rng, 16, 128), h=side, w=side,
                        cin=_channels(rng), cout=_channels(rng), k=k, stride=rng.choice([1, 1, 1, 2]), pad=k // 2,
                        bias=rng.random() < 0.5)
            if work(case)["flops"] <= CONV_FLOPS_CAP:
                return case
    if kind == "fc":
        return dict(kind="conv", bf16=rng.random() < 0.3, n=rng.randint(1, 8), batch=_log_int(rng, 16, 128), h=1, w=1,
                    cin=_log_int(rng, 64, 1024), cout=_log_int(rng, 10, 512), k=1, stride=1, pad=0, bias=True)
    if kind == "bn":
        while True:
            side = rng.choice([7, 8, 14, 16, 28, 32])
            case = dict(kind="bn", bf16=rng.random() < 0.7, n=rng.randint(1, 8), batch=_log_int(rng, 16, 128), h=side, w=side,
                        c=rng.choice([16, 20, 32, 50, 64, 128, 160, 256, 320, 640]), add=rng.random() < 0.5)
            if work(case)["bytes"] <= BN_BYTES_CAP:
                return case
    n = rng.randint(1, 8)
    return dict(kind="update", n=n, params=min(_log_int(rng, 10_000, 36_500_000), UPDATE_CAP // n), outer=rng.random() < 0.5)


def _channels(rng):
    """Mostly the widths of the framework's networks, sometimes any number."""
    return rng.choice([16, 20, 32, 50, 64, 96, 128, 160, 192, 256, 320]) if rng.random() < 0.8 else _log_int(rng, 12, 320)


# ---------------------------------------------------------------------------------------------------- shared helpers


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(1_000_003 * seed + 17)


def _normal(gen, shape, std=1.0, dtype=torch.float32):
    return torch.empty(shape, dtype=torch.float32, device=DEVICE).normal_(0.0, std, generator=gen).to(dtype)


def _model_config(case):
    model, _, side, channels = MODELS[case["model"]]
    return pb.make_config(model=model, n_replicas=case["n"], batch=case["batch"], compute_bf16=int(case["bf16"]), in_h=side,
                          in_w=side, in_c=channels, n_classes=CLASSES,
                          arch=(case["arch0"], case["arch1"], case["arch2"], case["arch3"]), eta_inner=0.01, eta_outer=0.01,
                          gamma0=0.03, rho0=1.0, fuse_outer=1)


def _initial_replicas(case, seed):
    """fp32 ``[n, n_params]``: one seeded initialisation, each replica moved a little (as after an outer step)."""
    cfg = _model_config(case)
    row = synth.init_params(pb.parle_query_layout(cfg), seed, MODELS[case["model"]][1])
    rng = np.random.default_rng([seed, 11])
    spread = 0.02 * float(np.std(row))
    return (row[None] + spread * rng.standard_normal((case["n"], row.size))).astype(np.float32)


def _images(case, seed, shape):
    """Class-conditional Gaussian images ``shape + (H, W, C)`` and their labels ``shape``."""
    _, _, side, channels = MODELS[case["model"]]
    gen = _generator(seed)
    means = _normal(gen, (CLASSES, side, side, channels))
    labels = torch.randint(0, CLASSES, shape, generator=gen, device=DEVICE)
    images = means[labels] + _normal(gen, tuple(shape) + (side, side, channels))
    return images.contiguous(), labels.to(torch.int32)


def _conv_desc(case):
    return pb.parle_conv_desc(int(case["bf16"]), case["n"], case["batch"], case["h"], case["w"], case["cin"], case["cout"],
                              case["k"], case["stride"], case["pad"])


def _conv_out(case):
    return tuple((case[d] + 2 * case["pad"] - case["k"]) // case["stride"] + 1 for d in ("h", "w"))


def _conv_inputs(case, seed):
    gen = _generator(seed)
    dt = torch.bfloat16 if case["bf16"] else torch.float32
    n, b, k, ci, co = case["n"], case["batch"], case["k"], case["cin"], case["cout"]
    ho, wo = _conv_out(case)
    x = _normal(gen, (n, b, case["h"], case["w"], ci)).clamp_(min=0).to(dt)  # the output of the ReLU in front
    w = _normal(gen, (n, co, k, k, ci), math.sqrt(2.0 / (k * k * ci)), dt)
    bias = _normal(gen, (n, co), 0.1) if case["bias"] else None
    dy = _normal(gen, (n, b, ho, wo, co), 1e-2, dt)
    return x, w, bias, dy


def _bn_inputs(case, seed):
    gen = _generator(seed)
    dt = torch.bfloat16 if case["bf16"] else torch.float32
    shape = (case["n"], case["batch"], case["h"], case["w"], case["c"])
    x = (_normal(gen, shape) * 1.5 + _normal(gen, (case["n"], 1, 1, 1, case["c"]), 0.5)).to(dt)
    dout = _normal(gen, shape, 1e-2, dt)
    add = _normal(gen, shape, 1e-2, dt) if case["add"] else None
    gamma = 1.0 + _normal(gen, (case["n"], case["c"]), 0.1)
    beta = _normal(gen, (case["n"], case["c"]), 0.1)
    return x, dout, add, gamma, beta


def _update_config(case):
    return pb.make_config(model=pb.MODEL_FLAT, n_replicas=case["n"], n_params=case["params"], eta_inner=0.1, eta_outer=0.1,
                          momentum=0.9, alpha=0.75, gamma0=0.03, rho0=1.0, fuse_outer=1)


def _update_inputs(case, seed):
    gen = _generator(seed)
    shape = (case["n"], case["params"])
    x, grad = _normal(gen, shape, 0.05), _normal(gen, shape, 1e-2)
    return x, grad


# --------------------------------------------------------------------------------------------------- prepare and run


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "eval"):
        state = dict(case=case, P=pb.Parle(_model_config(case), _initial_replicas(case, seed)))
        shape = (case["n"], case["batch"]) if kind == "step" else (case["count"],)
        state["images"], state["labels"] = _images(case, seed, shape)
        state["loss"] = torch.zeros(case["n"], dtype=torch.float32, device=DEVICE)
        return state
    if kind == "conv":
        x, w, bias, dy = _conv_inputs(case, seed)
        desc = _conv_desc(case)
        n, co = case["n"], case["cout"]
        wsize = w[0].numel()
        act = pb.parle_act_desc(int(case["bf16"]), n, case["batch"], *_conv_out(case), co)
        return dict(case=case, desc=desc, act=act, x=x, w=w, bias=bias, dy=dy, y=torch.empty_like(dy), dx=torch.empty_like(x),
                    wt=torch.empty_like(w), wsize=wsize,
                    scratch=torch.empty(max(pb.parle_k_conv_scratch_bytes(desc), 256), dtype=torch.uint8, device=DEVICE),
                    act_scratch=torch.empty(pb.parle_k_layer_scratch_bytes(act), dtype=torch.uint8, device=DEVICE),
                    dwb=torch.zeros((n, wsize + (co if case["bias"] else 0)), dtype=torch.float32, device=DEVICE),
                    db=torch.zeros((n, co), dtype=torch.float32, device=DEVICE))
    if kind == "bn":
        x, dout, add, gamma, beta = _bn_inputs(case, seed)
        n, c = case["n"], case["c"]
        desc = pb.parle_act_desc(int(case["bf16"]), n, case["batch"], case["h"], case["w"], c)
        row = dict(dtype=torch.float32, device=DEVICE)
        running = torch.zeros((n, 2, c), **row)
        running[:, 1] = 1.0
        return dict(case=case, desc=desc, x=x, dout=dout, add=add, gamma=gamma, beta=beta, out=torch.empty_like(x),
                    dx=torch.empty_like(x), saved=torch.empty((n, 2, c), **row), sums=torch.empty((n, 2, c), **row),
                    dgamma=torch.empty((n, c), **row), dbeta=torch.empty((n, c), **row), running=running,
                    scratch=torch.empty(pb.parle_k_layer_scratch_bytes(desc), dtype=torch.uint8, device=DEVICE))
    x, grad = _update_inputs(case, seed)
    P = pb.Parle(_update_config(case), x)
    P.grad[:, :case["params"]].copy_(grad)
    return dict(case=case, P=P)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        P = state["P"]
        P.parle_inner_step(state["images"], state["labels"], state["loss"])
        return state["loss"], P.grad[:, :P.sizes.n_params], P.y[:, :P.sizes.n_params]
    if kind == "eval":
        loss, errors, spread = state["P"].parle_eval(-1, state["images"], state["labels"])
        return float(loss), float(errors), float(spread)
    if kind == "conv":
        s = state
        pb.parle_k_conv_forward(s["desc"], s["x"], s["w"], s["bias"], None, case["bias"], s["y"])
        pb.parle_k_conv_backward_data(s["desc"], s["dy"], s["w"], s["x"] if case["bias"] else None, False, s["wt"], s["dx"])
        if not case["bias"]:
            pb.parle_k_conv_backward_weight(s["desc"], s["dy"], s["x"], s["scratch"], s["dwb"])
            return s["y"], s["dx"], s["dwb"]
        db = s["dwb"][:, s["wsize"]:]
        if not pb.parle_k_conv_backward_weight_bias(s["desc"], s["dy"], s["x"], s["scratch"], s["dwb"]):
            pb.parle_k_bias_grad(s["act"], s["dy"], s["act_scratch"], s["db"])
            db = s["db"]
        return s["y"], s["dx"], s["dwb"][:, :s["wsize"]], db
    if kind == "bn":
        s = state
        pb.parle_k_bn_forward(s["desc"], s["x"], s["gamma"], s["beta"], s["scratch"], s["saved"], s["running"], s["out"])
        pb.parle_k_bn_backward(s["desc"], s["x"], s["dout"], s["gamma"], s["beta"], s["saved"], s["add"], s["scratch"],
                               s["sums"], s["dgamma"], s["dbeta"], s["dx"])
        return s["out"], s["dx"], s["saved"], s["dgamma"], s["dbeta"]
    P = state["P"]
    P.parle_inner_step()
    N = case["params"]
    if not case["outer"]:
        return P.y[:, :N], P.vy[:, :N], P.z[:, :N]
    P.parle_outer_step()
    return P.x[:, :N], P.vx[:, :N], P.x_ref[:N]


# ---------------------------------------------------------------------------------------------- work and tolerances


def work(case):
    kind = case["kind"]
    if kind in ("step", "eval"):
        cfg = _model_config(case)
        sizes = pb.parle_query_sizes(cfg)
        flops = sizes.forward_flops_per_image
        if kind == "eval":  # images, labels and the evaluated row; the spread reads every replica and the reference
            return {"bytes": case["count"] * (sizes.image_elems * 4 + 4) + (case["n"] + 1) * sizes.n_params * 4,
                    "flops": flops * case["count"]}
        # three contractions per layer, but nothing needs the first layer's input gradient
        _, _, side, channels = MODELS[case["model"]]
        first = {"mlp": side * side * case["arch0"], "lenet": (side - 4) ** 2 * 25 * case["arch0"],
                 "allcnn": side * side * 9 * channels * case["arch0"]}[case["model"]]
        images = case["n"] * case["batch"]
        # state: y, x, vy, z read; grad, y, vy, z written
        return {"bytes": images * (sizes.image_elems * 4 + 4) + case["n"] * sizes.n_params * 32,
                "flops": images * (3 * flops - 2 * first)}
    if kind == "conv":
        es = 2 if case["bf16"] else 4
        ho, wo = _conv_out(case)
        nb = case["n"] * case["batch"]
        x, y = nb * case["h"] * case["w"] * case["cin"], nb * ho * wo * case["cout"]
        wsize = case["n"] * case["cout"] * case["k"] ** 2 * case["cin"]
        bias = 2 * case["n"] * case["cout"] * 4 if case["bias"] else 0
        return {"bytes": (2 * x + 2 * y + wsize) * es + wsize * 4 + bias,
                "flops": 3 * 2 * nb * ho * wo * case["cout"] * case["k"] ** 2 * case["cin"]}
    if kind == "bn":
        elems = case["n"] * case["batch"] * case["h"] * case["w"] * case["c"]
        # x, dout (and add) read; out and dx written
        return {"bytes": elems * (2 if case["bf16"] else 4) * (5 if case["add"] else 4), "flops": 16 * elems}
    elems = case["n"] * case["params"]
    # grad, y, x, vy, z read; y, vy, z written; the outer step reads x, z, vx and writes x, vx, y, z, vy
    return {"bytes": elems * (64 if case["outer"] else 32) + (4 * case["params"] if case["outer"] else 0),
            "flops": elems * (24 if case["outer"] else 12)}


def tolerance(case):
    """About four times the distance from the 64-bit result that the path shows (2-norm)."""
    kind = case["kind"]
    if kind == "step":
        # bf16: 7e-3 on All-CNN-C's gradient, the roundings of nine layers.  fp32: 4e-7, and room for a ReLU or max-pool
        # decision that another order of summation takes the other way.
        return {"rel": 3e-2} if case["bf16"] else {"rel": 1e-4}
    if kind == "eval":  # the loss, and the error count, in which one tie among a few hundred images may fall the other way
        return {"rel": 1e-2} if case["bf16"] else {"rel": 1e-4}
    if kind == "update":  # 3e-8: a handful of fp32 roundings per element
        return {"rel": 2e-7}
    # bf16 results: 1.7e-3, one rounding on the store.  fp32: 2e-6 on sums over 131 072 rows.
    return {"rel": 7e-3} if case["bf16"] else {"rel": 1e-5}


# --------------------------------------------------------------------------------------------- the same in 64 bits


def _layer64(x, w, bias, stride, pad):
    """Convolution of ``[B, H, W, C]`` with ``[Cout, k, k, Cin]`` as one matrix product."""
    cout, k, _, cin = w.shape
    if k == 1 and stride == 1 and pad == 0:
        out = x.reshape(-1, cin) @ w.reshape(cout, cin).t()
        ho, wo = x.shape[1], x.shape[2]
    else:
        cols = F.unfold(x.permute(0, 3, 1, 2), k, padding=pad, stride=stride)  # [B, C*k*k, P]
        ho, wo = ((s + 2 * pad - k) // stride + 1 for s in (x.shape[1], x.shape[2]))
        out = cols.permute(0, 2, 1).reshape(-1, cin * k * k) @ w.permute(0, 3, 1, 2).reshape(cout, -1).t()
    out = out.reshape(x.shape[0], ho, wo, cout)
    return out if bias is None else out + bias


def _pool64(x):
    b, h, w, c = x.shape
    x = x[:, :h // 2 * 2, :w // 2 * 2].reshape(b, h // 2, 2, w // 2, 2, c).permute(0, 1, 3, 2, 4, 5)
    return x.reshape(b, h // 2, w // 2, 4, c).amax(3)


def _logits64(case, p, x):
    """Forward pass of one replica: ``p`` maps segment names to 64-bit tensors, ``x`` is ``[B, H, W, C]``."""
    def conv(name, h, stride=1, pad=0):
        w = p[name + ".w"]
        w = w if w.dim() == 4 else w.reshape(w.shape[0], 1, 1, w.shape[1])
        return _layer64(h, w, p.get(name + ".b"), stride, pad)

    def flat(h):
        return h.reshape(h.shape[0], 1, 1, -1)

    model = case["model"]
    if model == "mlp":
        return conv("fc2", conv("fc1", flat(x)).relu())[:, 0, 0]
    if model == "lenet":
        h = _pool64(conv("conv1", x).relu())
        h = _pool64(conv("conv2", h).relu())
        return conv("fc2", conv("fc1", flat(h)).relu())[:, 0, 0]
    if model == "allcnn":
        for i, stride in enumerate((1, 1, 2, 1, 1, 2, 1, 1, 1)):
            x = conv(f"conv{i + 1}", x, stride, 1 if i < 7 else 0)
            x = x.relu() if i < 8 else x
        return x.mean((1, 2))

    def bn(name, h):  # evaluation of a fresh context: running mean 0, running variance 1
        return (h * (p[name + ".g"] / math.sqrt(1.0 + 1e-5)) + p[name + ".b"]).relu()

    h = conv("conv1", x, 1, 1)
    blocks = sorted({name.split(".")[0] for name in p if name.startswith("g")})
    for blk in blocks:
        stride = 2 if blk in ("g2b1", "g3b1") else 1
        o = bn(blk + ".bn1", h)
        short = conv(blk + ".sc", o, stride) if blk + ".sc.w" in p else h
        h = conv(blk + ".conv2", bn(blk + ".bn2", conv(blk + ".conv1", o, stride, 1)), 1, 1) + short
    return conv("fc", bn("bn_out", h).mean((1, 2), keepdim=True))[:, 0, 0]


def _segments64(case, row):
    """Segments of one parameter row as 64-bit tensors, contraction weights rounded to the compute type."""
    out = {}
    for seg in pb.parle_query_layout(_model_config(case)):
        v = row[seg["offset"]:seg["offset"] + seg["size"]].reshape(seg["shape"])
        out[seg["name"]] = (v.bfloat16() if case["bf16"] and seg["kind"] == "weight" else v).double()
    return out


def _exact_model(case, seed):
    x0 = torch.as_tensor(_initial_replicas(case, seed), device=DEVICE)
    if case["kind"] == "eval":
        images, labels = _images(case, seed, (case["count"],))
        ref = x0.double().mean(0)
        spread = (x0.double() - ref).square().sum()
        with torch.no_grad():
            logits = _logits64(case, _segments64(case, ref.float()), _image64(case, images))
        loss = F.cross_entropy(logits, labels.long())
        errors = (logits.argmax(1) != labels).sum()
        return float(loss), float(errors), float(spread)
    images, labels = _images(case, seed, (case["n"], case["batch"]))
    losses, grads = [], []
    for a in range(case["n"]):
        segs = _segments64(case, x0[a])
        for v in segs.values():
            v.requires_grad_(True)
        loss = F.cross_entropy(_logits64(case, segs, _image64(case, images[a])), labels[a].long())
        g = torch.autograd.grad(loss, list(segs.values()))
        losses.append(loss.detach())
        grads.append(torch.cat([t.reshape(-1) for t in g]))
    grad = torch.stack(grads)
    # first step from v = 0 and y = x: d = grad, y <- y - eta (1 + mu) d
    cfg = _model_config(case)
    return torch.stack(losses), grad, x0.double() - cfg.eta_inner * (1.0 + cfg.momentum) * grad


def _image64(case, images):
    return (images.bfloat16() if case["bf16"] else images).double()


def _exact_conv(case, seed):
    x, w, bias, dy = _conv_inputs(case, seed)
    ho, wo = _conv_out(case)
    s, pad, k = case["stride"], case["pad"], case["k"]
    ys, dxs, dws = [], [], []
    for a in range(case["n"]):
        xp = F.pad(x[a].double(), (0, 0, pad, pad, pad, pad))
        wa, da = w[a].double(), dy[a].double().reshape(-1, case["cout"])
        y = torch.zeros((da.shape[0], case["cout"]), dtype=torch.float64, device=DEVICE)
        dxp, dw = torch.zeros_like(xp), torch.zeros_like(wa)
        for r in range(k):
            for c in range(k):
                rows, cols = slice(r, r + s * (ho - 1) + 1, s), slice(c, c + s * (wo - 1) + 1, s)
                xs = xp[:, rows, cols].reshape(-1, case["cin"])
                y += xs @ wa[:, r, c].t()
                dxp[:, rows, cols] += (da @ wa[:, r, c]).reshape(case["batch"], ho, wo, case["cin"])
                dw[:, r, c] = da.t() @ xs
        y = y.reshape(case["batch"], ho, wo, case["cout"])
        dx = dxp[:, pad:pad + case["h"], pad:pad + case["w"]]
        if case["bias"]:
            y = (y + bias[a].double()).relu()
            dx = dx * (x[a] > 0)
        ys.append(y), dxs.append(dx), dws.append(dw.reshape(-1))
    out = (torch.stack(ys), torch.stack(dxs), torch.stack(dws))
    return out + (dy.double().sum((1, 2, 3)),) if case["bias"] else out


def _exact_bn(case, seed):
    x, dout, add, gamma, beta = (t if t is None else t.double() for t in _bn_inputs(case, seed))
    mean = x.mean((1, 2, 3), keepdim=True)
    rstd = (x.var((1, 2, 3), unbiased=False, keepdim=True) + 1e-5).rsqrt()
    xhat = (x - mean) * rstd
    g, b = gamma[:, None, None, None], beta[:, None, None, None]
    pre = g * xhat + b
    d = dout * (pre > 0)
    dbeta, dgamma = d.sum((1, 2, 3)), (d * xhat).sum((1, 2, 3))
    m = x[0, ..., 0].numel()
    dx = g * rstd * (d - (dbeta[:, None, None, None] + xhat * dgamma[:, None, None, None]) / m)
    dx = dx if add is None else dx + add
    saved = torch.stack([mean.reshape(gamma.shape), rstd.reshape(gamma.shape)], 1)
    return pre.relu(), dx, saved, dgamma, dbeta


def _exact_update(case, seed):
    x, grad = (t.double() for t in _update_inputs(case, seed))
    cfg = _update_config(case)
    eta, mu, alpha = cfg.eta_inner, cfg.momentum, cfg.alpha
    vy = grad  # from y = z = x and v = 0
    y = x - eta * (1.0 + mu) * vy
    z = alpha * x + (1.0 - alpha) * y
    if not case["outer"]:
        return y, vy, z
    ref = x.mean(0)
    vx = cfg.gamma0 * (x - z) + cfg.rho0 * (x - ref)
    return x - cfg.eta_outer * (1.0 + mu) * vx, vx, ref


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "eval"):
        return _exact_model(case, seed)
    return {"conv": _exact_conv, "bn": _exact_bn, "update": _exact_update}[kind](case, seed)
