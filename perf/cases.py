"""The work that a program training or running InPlace-ABN layers has this
library do, as measurable cases.

Every case is one or more calls of the Python binding on a layer (or, for the
backbone, on all its layers).  A training pass calls the forward on one
layer's activations and the backward on stored activations and gradients of
another: in a network a layer's backward never follows its own forward
directly.  All calls work in place, so a second pass on the same state reads
what the first wrote; the values are chosen so that this stays in range (the
forward normalises; the backward's gain gamma/sigma is 1; inference
contracts).
"""

import math

import torch

import paper_1712_02616_amd as iabn

EPS, MOMENTUM, SLOPE = 1e-5, 0.1, 0.01
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}

# What each kind of pass must read and write once, in storage units per
# element of a layer: the training forward 2 (x in, z out), the backward 3
# (z and dz in, dx out), the standard block's backward 4 (x too), the
# checkpointing's forward 3 (xhat and z out) and recomputation 2.
UNITS = {"step": 5, "step_ii": 5, "forward_noalloc": 2, "eval": 2, "std": 6, "ckpt": 8, "blocks": 14}
# Arithmetic per element: a forward about 7 operations (shifted sums, affine,
# activation), a backward about 13, inference 4.
FLOPS = {"step": 20, "step_ii": 20, "forward_noalloc": 7, "eval": 4, "std": 20, "ckpt": 24, "blocks": 44}

# The activations and gradients of a state (the rest is per channel).
TENSORS = ("x", "dz", "xs", "xhat", "dz_ckpt", "z", "x_ckpt", "z_out", "z_again", "z_ckpt")

# The layers of a ResNet-101-like backbone at batch 8 and output stride 8 on
# 512x512 inputs, fp16: the library's benchmark workload.
BACKBONE = ([(8, 256, 128, 128)] * 3 + [(8, 512, 64, 64)] * 4 + [(8, 1024, 64, 64)] * 23 +
            [(8, 2048, 64, 64)] * 3)


def _case(name, op, dtype, n, c, h, w, workspace=True, gamma_sign=False):
    """workspace: the program keeps a workspace and passes it (otherwise the
    binding takes one from torch's allocator on each call)."""
    return {"name": name, "op": op, "dtype": dtype, "n": n, "c": c, "h": h, "w": w,
            "workspace": workspace, "gamma_sign": gamma_sign}


def listed():
    return [
        # The smallest layer of the test workloads: the cost of a call.
        _case("tiny_step_f32", "step", "f32", 2, 16, 8, 8, workspace=False),
        # The last stage of a ResNet-50 at batch 32: 49-value rows.
        _case("stage4_step_f16", "step", "f16", 32, 2048, 7, 7, workspace=False),
        # Its third stage: rows that end inside a cache line.
        _case("stage3_step_bf16", "step", "bf16", 32, 1024, 14, 14),
        # Its first stage's wide layers, in fp32.
        _case("stage1_step_f32", "step", "f32", 32, 256, 56, 56),
        # Its stem: few channels, large maps.
        _case("stem_step_f16", "step", "f16", 32, 64, 112, 112),
        # A segmentation network's first layers at high resolution.
        _case("highres_step_f16", "step", "f16", 8, 64, 256, 256),
        # A segmentation head on 192x192 maps, scales of either sign.
        _case("segcrop_step_f16", "step", "f16", 4, 256, 192, 192, gamma_sign=True),
        # A wide deep layer, in bf16.
        _case("wide_step_bf16", "step", "bf16", 16, 2048, 28, 28),
        # Odd maps: an output-stride-8 network on 513x513 crops.
        _case("odd_step_f16", "step", "f16", 8, 512, 65, 65, workspace=False),
        # Inference with the running statistics.
        _case("eval_f16", "eval", "f16", 8, 1024, 64, 64),
        # The blocks the method is compared with (standard, checkpointing).
        _case("blocks_f16", "blocks", "f16", 8, 256, 128, 128),
        # A whole backbone's training pass, 33 layers.
        _case("backbone_f16", "backbone", "f16", 0, 0, 0, 0),
    ]


def draw(rng):
    """A layer between the smallest of the listed ones and 2^26 values, of
    any channel count, map size, storage type and kind of pass."""
    op = rng.choice(["step"] * 5 + ["step_ii", "forward_noalloc", "eval", "eval", "std", "ckpt"])
    dtype = rng.choice(sorted(DTYPES))
    total = 2 ** rng.uniform(11, 26)
    c = int(round(2 ** rng.uniform(3, 11)))
    n = int(round(2 ** rng.uniform(0, 6)))
    hw = total / (n * c)
    while hw < 9 and n > 1:
        n = (n + 1) // 2
        hw = total / (n * c)
    h = max(3, int(math.sqrt(hw) * rng.uniform(0.8, 1.25)))
    w = max(3, int(hw / h))
    if rng.random() < 0.4:  # maps of whole multiples of 8, as crops often are
        h, w = max(8, h // 8 * 8), max(8, w // 8 * 8)
    case = _case("", op, dtype, n, c, h, w, workspace=rng.random() < 0.5,
                 gamma_sign=rng.random() < 0.3)
    del case["name"]
    return case


def _layers(case):
    if case["op"] == "backbone":
        return BACKBONE
    return [(case["n"], case["c"], case["h"], case["w"])]


def _has_backward(op):
    return op not in ("eval", "forward_noalloc")


def _inputs(case, seed):
    """Storage-type inputs of all the case's layers, the activations of each
    kind in one flat tensor, a layer after the other.
      x       the forward's (or inference's) input
      n_      the backward's normalised activation, z = f(gamma n_ + beta),
              xs = mu + |gamma| n_ (what the standard block keeps), dz
    """
    op, dt = case["op"], DTYPES[case["dtype"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    layers = _layers(case)
    total = sum(n * c * h * w for n, c, h, w in layers)
    channels = sum(c for _, c, _, _ in layers)

    def chan(lo, hi):
        return torch.rand(channels, generator=gen, device="cuda") * (hi - lo) + lo

    flat = {"mu": chan(-2.0, 2.0), "sigma": chan(0.5, 3.0), "gamma": chan(0.5, 1.5),
            "beta": 0.1 * torch.randn(channels, generator=gen, device="cuda"),
            "running_mean": torch.zeros(channels, device="cuda"),
            "running_var": torch.ones(channels, device="cuda")}
    if case["gamma_sign"]:
        flat["gamma"] *= torch.where(chan(0.0, 1.0) < 0.5, -1.0, 1.0)
    if op == "eval":
        flat["sigma"] = 2.0 * flat["gamma"].abs()
        flat["running_mean"] = flat["mu"].clone()
        flat["running_var"] = flat["sigma"] ** 2
    flat["back_var"] = flat["gamma"] ** 2
    kinds = ["x"]
    if _has_backward(op):
        kinds += ["dz"]
        if op in ("std", "blocks"):
            kinds += ["xs"]
        if op in ("ckpt", "blocks"):
            kinds += ["xhat", "dz_ckpt"]
        if op != "ckpt":
            kinds += ["z"]
        if op == "blocks":
            kinds += ["x_ckpt"]
    for k in kinds:
        flat[k] = torch.empty(total, dtype=dt, device="cuda")
    e0 = c0 = 0
    for n, c, h, w in layers:
        e1, c1 = e0 + n * c * h * w, c0 + c

        def view(v):
            return v[c0:c1].view(1, c, 1)

        def normal():
            return torch.randn((n, c, h * w), generator=gen, device="cuda")

        x = normal() * view(flat["sigma"]) + view(flat["mu"])
        flat["x"][e0:e1] = x.view(-1).to(dt)
        if "x_ckpt" in flat:
            flat["x_ckpt"][e0:e1] = flat["x"][e0:e1]
        if _has_backward(op):
            flat["dz"][e0:e1] = (0.1 * normal()).view(-1).to(dt)
            if "dz_ckpt" in flat:
                flat["dz_ckpt"][e0:e1] = flat["dz"][e0:e1]
            v = normal()
            if "xhat" in flat:
                flat["xhat"][e0:e1] = v.view(-1).to(dt)
            if "xs" in flat:
                flat["xs"][e0:e1] = (v * view(flat["gamma"]).abs() + view(flat["mu"])).view(-1).to(dt)
            if "z" in flat:
                y = v * view(flat["gamma"]) + view(flat["beta"])
                flat["z"][e0:e1] = torch.where(y >= 0, y, SLOPE * y).view(-1).to(dt)
        e0, c0 = e1, c1
    return flat


def prepare(case, seed):
    flat = _inputs(case, seed)
    op, dt = case["op"], DTYPES[case["dtype"]]
    layers = _layers(case)
    channels = flat["gamma"].numel()
    for k in ("save_mean", "save_var", "dgamma", "dbeta"):
        flat[k] = torch.zeros(channels, device="cuda")
    if op in ("std", "ckpt", "blocks"):
        flat["z_out"] = torch.zeros_like(flat["x"])
    if op in ("ckpt", "blocks"):
        flat["z_again"] = torch.zeros_like(flat["x"])
    if op == "blocks":
        flat["z_ckpt"] = torch.zeros_like(flat["x"])
        for k in ("dgamma_ckpt", "dbeta_ckpt"):
            flat[k] = torch.zeros(channels, device="cuda")
    workspace = None
    if case["workspace"]:
        need = max(iabn.iabn_workspace_size(n, c, h * w, dt) for n, c, h, w in layers)
        workspace = torch.empty(need, dtype=torch.uint8, device="cuda")
    parts, e0, c0 = [], 0, 0
    for n, c, h, w in layers:
        e1, c1 = e0 + n * c * h * w, c0 + c
        parts.append({k: v[e0:e1].view(n, c, h, w) if k in TENSORS else v[c0:c1]
                      for k, v in flat.items()})
        e0, c0 = e1, c1
    return {"op": op, "flat": flat, "parts": parts, "workspace": workspace}


def _forward(t, ws):
    iabn.iabn_forward_train(t["x"], t["gamma"], t["beta"], t["running_mean"], t["running_var"],
                            t["save_mean"], t["save_var"], EPS, MOMENTUM, SLOPE, workspace=ws)


def _backward(t, ws):
    iabn.iabn_backward(t["z"], t["dz"], t["gamma"], t["beta"], t["back_var"], t["dgamma"],
                       t["dbeta"], EPS, SLOPE, workspace=ws)


def _std(t, ws):
    iabn.iabn_std_forward_train(t["x"], t["z_out"], t["gamma"], t["beta"], t["running_mean"],
                                t["running_var"], t["save_mean"], t["save_var"], EPS, MOMENTUM,
                                SLOPE, workspace=ws)
    iabn.iabn_std_backward(t["xs"], t["z"], t["dz"], t["gamma"], t["beta"], t["mu"], t["back_var"],
                           t["dgamma"], t["dbeta"], EPS, SLOPE, workspace=ws)


def _ckpt(t, ws, x, z, dz, dgamma, dbeta):
    iabn.iabn_ckpt_forward_train(t[x], t[z], t["gamma"], t["beta"], t["running_mean"],
                                 t["running_var"], t["save_mean"], t["save_var"], EPS, MOMENTUM,
                                 SLOPE, workspace=ws)
    iabn.iabn_ckpt_recompute(t["xhat"], t["z_again"], t["gamma"], t["beta"], SLOPE)
    iabn.iabn_ckpt_backward(t["xhat"], t[dz], t["gamma"], t["beta"], t["back_var"], t[dgamma],
                            t[dbeta], EPS, SLOPE, workspace=ws)


STATISTICS = ("save_mean", "save_var", "running_mean", "running_var")
RESULTS = {
    "step": ("x", "dz", "dgamma", "dbeta") + STATISTICS,
    "step_ii": ("x", "dz", "dgamma", "dbeta") + STATISTICS,
    "backbone": ("x", "dz", "dgamma", "dbeta") + STATISTICS,
    "forward_noalloc": ("x",) + STATISTICS,
    "eval": ("x",),
    "std": ("z_out", "dz", "dgamma", "dbeta") + STATISTICS,
    "ckpt": ("x", "z_out", "z_again", "dz", "dgamma", "dbeta") + STATISTICS,
    "blocks": ("z_out", "dz", "dgamma", "dbeta", "x_ckpt", "z_ckpt", "z_again", "dz_ckpt",
               "dgamma_ckpt", "dbeta_ckpt") + STATISTICS,
}


def run(state):
    op, ws = state["op"], state["workspace"]
    parts = state["parts"]
    if op == "step":
        _forward(parts[0], ws)
        _backward(parts[0], ws)
    elif op == "step_ii":
        t = parts[0]
        _forward(t, ws)
        iabn.iabn_backward_ii(t["z"], t["dz"], t["gamma"], t["beta"], t["back_var"], t["dgamma"],
                              t["dbeta"], EPS, SLOPE, workspace=ws)
    elif op == "backbone":
        for t in parts:
            _forward(t, ws)
        for t in reversed(parts):
            _backward(t, ws)
    elif op == "forward_noalloc":
        t = parts[0]
        iabn.iabn_forward_train_noalloc(t["x"], t["gamma"], t["beta"], t["running_mean"],
                                        t["running_var"], t["save_mean"], t["save_var"], EPS,
                                        MOMENTUM, SLOPE)
    elif op == "eval":
        t = parts[0]
        iabn.iabn_forward_eval(t["x"], t["gamma"], t["beta"], t["running_mean"], t["running_var"],
                               EPS, SLOPE)
    elif op == "std":
        _std(parts[0], ws)
    elif op == "ckpt":
        _ckpt(parts[0], ws, "x", "z_out", "dz", "dgamma", "dbeta")
    else:  # blocks
        _std(parts[0], ws)
        _ckpt(parts[0], ws, "x_ckpt", "z_ckpt", "dz_ckpt", "dgamma_ckpt", "dbeta_ckpt")
    flat = state["flat"]
    return {k: flat[k] for k in RESULTS[op]}


def work(case):
    layers = _layers(case)
    units = UNITS["step" if case["op"] == "backbone" else case["op"]]
    flops = FLOPS["step" if case["op"] == "backbone" else case["op"]]
    elements = sum(n * c * h * w for n, c, h, w in layers)
    channels = sum(c for _, c, _, _ in layers)
    # Per channel about 16 fp32 parameters, statistics and sums.
    return {"bytes": elements * units * BYTES[case["dtype"]] + 64 * channels,
            "flops": elements * flops}


def tolerance(case):
    """Each output is rounded once to its storage type (half an ulp: relative
    error at most 2^-24, 2^-11 or 2^-8 per value, 0.4 of that in the 2-norm),
    fp32 arithmetic and sums in another order move fp32 results by a few
    1e-7, and a second pass on the first one's outputs carries its rounding
    on.  Measured against exact(): 2e-7 (fp32 statistics 8e-7), 2.1e-4 and
    1.7e-3; about four times that is allowed, and single values a few ulps."""
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 2e-4}
    if case["dtype"] == "f16":
        return {"rel": 1e-3, "max": 1e-2}
    return {"rel": 7e-3, "max": 8e-2}


def exact(case, seed):
    """What run() returns for one pass, in float64, from the definitions:
    batch statistics (biased variance; the running variance takes m/(m-1)),
    z = f(gamma (x - mu)/sqrt(var + eps) + beta), and the batch-norm gradient
    dx = gamma/sqrt(var + eps) (dy - mean(dy) - xhat mean(dy xhat))."""
    op, dt = case["op"], DTYPES[case["dtype"]]
    flat = _inputs(case, seed)
    layers = _layers(case)
    eps, mom, slope = (float(torch.tensor(v, dtype=torch.float32)) for v in (EPS, MOMENTUM, SLOPE))
    out = {k: [] for k in RESULTS[op]}
    e0 = c0 = 0
    for n, c, h, w in layers:
        e1, c1 = e0 + n * c * h * w, c0 + c

        def tensor(k):
            return flat[k][e0:e1].view(n, c, h * w).double()

        def chan(k):
            return flat[k][c0:c1].double().view(1, c, 1)

        gamma, beta = chan("gamma"), chan("beta")
        m = n * h * w

        def act(y):
            return torch.where(y >= 0, y, slope * y)

        def put(k, v):
            if k in out:
                out[k].append(v.reshape(-1))

        x = tensor("x")
        if op == "eval":
            put("x", act(gamma * (x - chan("running_mean")) / (chan("running_var") + eps).sqrt() + beta))
        else:
            mu = x.mean((0, 2), keepdim=True)
            var = (x - mu).square().mean((0, 2), keepdim=True)
            xhat = (x - mu) / (var + eps).sqrt()
            put("save_mean", mu)
            put("save_var", var)
            rm, rv = chan("running_mean"), chan("running_var")
            for _ in range(2 if op == "blocks" else 1):  # two blocks update the same estimates
                rm = (1 - mom) * rm + mom * mu
                rv = (1 - mom) * rv + mom * var * m / (m - 1)
            put("running_mean", rm)
            put("running_var", rv)
            if op in ("ckpt", "blocks"):
                # z comes from xhat as stored
                stored = xhat.to(dt).double()
                put("x" if op == "ckpt" else "x_ckpt", xhat)
                put("z_out" if op == "ckpt" else "z_ckpt", act(gamma * stored + beta))
                put("z_again", act(gamma * tensor("xhat") + beta))
            if op not in ("ckpt", "std"):
                put("x", act(gamma * xhat + beta))
            if op in ("std", "blocks"):
                put("z_out", act(gamma * xhat + beta))
            del x, xhat

            def gradient(xh, negative, dz, names):
                dy = torch.where(negative, slope * dz, dz)
                dbeta = dy.sum((0, 2), keepdim=True)
                dgamma = (dy * xh).sum((0, 2), keepdim=True)
                put(names[0], gamma / (chan("back_var") + eps).sqrt() * (dy - dbeta / m - xh * dgamma / m))
                put(names[1], dgamma)
                put(names[2], dbeta)

            if op in ("step", "step_ii", "backbone"):
                z = tensor("z")
                gradient((torch.where(z < 0, z / slope, z) - beta) / gamma, z < 0, tensor("dz"),
                         ("dz", "dgamma", "dbeta"))
            if op in ("std", "blocks"):
                gradient((tensor("xs") - chan("mu")) / (chan("back_var") + eps).sqrt(),
                         tensor("z") < 0, tensor("dz"), ("dz", "dgamma", "dbeta"))
            if op in ("ckpt", "blocks"):
                xh = tensor("xhat")
                gradient(xh, gamma * xh + beta < 0, tensor("dz" if op == "ckpt" else "dz_ckpt"),
                         ("dz", "dgamma", "dbeta") if op == "ckpt" else
                         ("dz_ckpt", "dgamma_ckpt", "dbeta_ckpt"))
        e0, c0 = e1, c1
    return {k: torch.cat(v) for k, v in out.items()}
