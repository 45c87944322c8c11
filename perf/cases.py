"""Performance cases of the framework: the calls that a training program makes, over their range.

Five kinds of work, each through the public entry points of paper_1712_04432_amd:

* ``step``   one SGD iteration of a fully connected stack (``mlp_train_step``), as a single-process
             program runs it;
* ``grads``  forward, loss and backward with the gradients stored (``mlp_fwd``, ``mlp_bwd``), as a program
             with its own optimiser or an all-reduce of its own runs it;
* ``grid``   the calls of one process of a P_r x P_c grid in an iteration: each layer's local forward, the
             loss on the gathered logits, each layer's local backward and the update of the weight block;
* ``conv``   forward and backward of a domain-parallel 3x3 convolution tile;
* ``update`` the update of one layer's weights from a reduced gradient (``sgd_step``).
"""
from __future__ import annotations

import math

import torch

import paper_1712_04432_amd as imbd

DEV = "cuda"


# ------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # The smallest network (784-256-128-10, 64 samples, fp32): launches and latency are all there is.
        {"name": "step_mlp784_f32", "kind": "step", "dims": "784-256-128-10", "batch": 64, "dtype": "f32"},
        # The fully connected layers of AlexNet at the batch the paper trains with.
        {"name": "step_alexnet_b256", "kind": "step", "dims": "9216-4096-4096-1000", "batch": 256, "dtype": "bf16"},
        # The same stack at the large end of the batch sweep, where the products are compute-bound.
        {"name": "step_alexnet_b2048", "kind": "step", "dims": "9216-4096-4096-1000", "batch": 2048, "dtype": "bf16"},
        # The fully connected layers of VGG, the largest weights.
        {"name": "step_vgg_b512", "kind": "step", "dims": "25088-4096-4096-1000", "batch": 512, "dtype": "bf16"},
        # The AlexNet stack trained in single precision.
        {"name": "step_alexnet_f32_b256", "kind": "step", "dims": "9216-4096-4096-1000", "batch": 256, "dtype": "f32",
         "lr": 0.001},
        # Gradients handed to the caller, with the input's gradient, on widths that are no multiple of anything.
        {"name": "grads_odd_bf16", "kind": "grads", "dims": "4095-1023-517-101", "batch": 200, "dtype": "bf16",
         "dx1": True},
        # One process of a 4 x 16 grid at a global batch of 1024: small blocks, many calls.
        {"name": "grid_4x16_bf16", "kind": "grid", "dims": "9216-4096-4096-1000", "P_r": 4, "P_c": 16, "batch": 1024,
         "dtype": "bf16"},
        # A 56 x 56 tile of a 224 x 224 image, 256 channels on both sides.
        {"name": "conv_56x56_256", "kind": "conv", "N": 32, "H": 56, "W": 56, "Ci": 256, "Co": 256, "out": "bf16"},
        # AlexNet's 3x3 convolution on 13 x 13 x 384 activations: small odd images, whole (no tile split).
        {"name": "conv_13x13_384", "kind": "conv", "N": 64, "H": 13, "W": 13, "Ci": 384, "Co": 384, "out": "bf16"},
        # An early layer: few channels, many positions (a quarter of a 112 x 112 image), channels doubling.
        {"name": "conv_56x56_64_128", "kind": "conv", "N": 32, "H": 56, "W": 56, "Ci": 64, "Co": 128, "out": "bf16"},
        # A late layer: many channels, few positions, outputs kept in fp32 for a reduction that follows.
        {"name": "conv_14x14_512_f32out", "kind": "conv", "N": 32, "H": 14, "W": 14, "Ci": 512, "Co": 512, "out": "f32"},
        # The update of AlexNet's first fully connected layer after an all-reduce: pure streaming.
        {"name": "update_9216x4096", "kind": "update", "n": 9216 * 4096, "lp": True},
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread evenly over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _width(rng, lo, hi):
    """A layer width: most are multiples of 8 as programs choose them, the others as they come."""
    w = _log(rng, lo, hi)
    how = rng.random()
    if how < 0.4:
        return max(8, w // 64 * 64) if w >= 64 else max(8, w // 8 * 8)
    return max(8, w // 8 * 8) if how < 0.7 else w


MOST_FLOPS = {"bf16": 5.0e11, "f32": 6.5e10, "conv": 3.3e11}


def draw(rng):
    while True:
        kind = rng.choice(["step", "step", "grads", "grid", "conv", "conv", "conv", "update"])
        if kind == "conv":
            c = {"kind": "conv", "N": _log(rng, 1, 64), "H": _log(rng, 4, 64), "W": _log(rng, 4, 64),
                 "Ci": 64 * rng.choice([1, 2, 3, 4, 4, 5, 6, 8]), "Co": 64 * rng.choice([1, 2, 3, 4, 4, 5, 6, 8]),
                 "out": rng.choice(["bf16", "bf16", "f32"])}
            top = MOST_FLOPS["conv"]
        elif kind == "update":
            return {"kind": "update", "n": _log(rng, 1000, 36_000_000), "lp": rng.random() < 0.7}
        else:
            layers = rng.choice([1, 2, 3, 3])
            dims = [_width(rng, 64, 12000)] + [_width(rng, 32, 4096) for _ in range(layers - 1)] + [_width(rng, 2, 1000)]
            c = {"kind": kind, "dims": "-".join(str(d) for d in dims), "batch": _log(rng, 1, 2048),
                 "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"])}
            if kind == "step":
                c["lr"] = 0.01 if c["dtype"] == "bf16" else 0.001
            if kind == "grads":
                c["dx1"] = rng.random() < 0.5
            if kind == "grid":
                c["P_r"], c["P_c"] = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4, 16])
                if c["batch"] < c["P_c"] or min(dims[1:]) < c["P_r"]:
                    continue
            top = MOST_FLOPS[c["dtype"]]
        if work(c)["flops"] <= top:
            return c


# ------------------------------------------------------------------------------------ inputs
def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, *shape, scale=1.0):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32).mul_(scale)


def _weights(g, d_out, d_in):
    return _normal(g, d_out, d_in, scale=math.sqrt(2.0 / d_in))  # He-initialised, as the networks are


def _tdtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _block(d, P_r):
    """Rows [lo, hi) of a d-row matrix that process row P_r // 2 of P_r holds."""
    r, per = P_r // 2, d // P_r
    return r * per, d if r == P_r - 1 else (r + 1) * per


def prepare(case, seed):
    g = _gen(seed)
    if case["kind"] in ("step", "grads"):
        dims, B, dt = _dims(case), case["batch"], _tdtype(case)
        # post-ReLU features of the layers below, labels uniform, biases zero
        x = _normal(g, B, dims[0]).clamp_(min=0.0).to(dt)
        labels = torch.randint(0, dims[-1], (B,), generator=g, device=DEV, dtype=torch.int32)
        net = imbd.MLP(dims, B, case["dtype"])
        layers = []
        for i in range(1, len(dims)):
            w = _weights(g, dims[i], dims[i - 1])
            ly = {"w": w, "w_lp": w.to(torch.bfloat16) if case["dtype"] == "bf16" else w,
                  "b": torch.zeros(dims[i], device=DEV)}
            if case["kind"] == "grads":
                ly["dw"] = torch.empty_like(w)
                ly["db"] = torch.empty(dims[i], device=DEV)
            layers.append(ly)
        ws = torch.empty(imbd.mlp_workspace_bytes(net), dtype=torch.uint8, device=DEV)
        loss = torch.zeros(1, device=DEV)
        dx1 = torch.empty(B, dims[0], dtype=dt, device=DEV) if case.get("dx1") else None
        out = {"loss": loss, "logits": imbd.ws_view(net, ws, imbd.IMBD_WS_LOGITS)}
        for i, ly in enumerate(layers):
            if case["kind"] == "grads":
                out["dw%d" % i], out["db%d" % i] = ly["dw"], ly["db"]
                continue
            out["w%d" % i], out["b%d" % i] = ly["w"], ly["b"]
            if case["dtype"] == "bf16":
                out["w_lp%d" % i] = ly["w_lp"]
        if dx1 is not None:
            out["dx1"] = dx1
        return {"case": case, "net": net, "x": x, "labels": labels, "layers": layers, "lr": case.get("lr", 0.01), "ws": ws,
                "loss": loss, "dx1": dx1, "out": out}
    if case["kind"] == "grid":
        dims, dt = _dims(case), _tdtype(case)
        P_r, P_c, b = case["P_r"], case["P_c"], case["batch"] // case["P_c"]
        code = imbd.dtype_code(dt)
        layers, need = [], 16
        for i in range(1, len(dims)):
            lo, hi = _block(dims[i], P_r)
            w = _weights(g, hi - lo, dims[i - 1])
            top = i == len(dims) - 1
            # the gathered activations of the layer below, and the reduced gradient of its outputs (the top
            # layer's comes from the loss); both hold whole rows, of which the process uses its columns
            x = _normal(g, b, dims[i - 1])
            if i > 1:
                x.clamp_(min=0.0)
            ly = {"w": w, "w_lp": w.to(dt) if dt == torch.bfloat16 else w, "bias": _normal(g, hi - lo, scale=0.1),
                  "x": x.to(dt), "dy": _normal(g, b, dims[i]).to(dt), "lo": lo, "hi": hi, "top": top,
                  "y": torch.empty(b, hi - lo, dtype=torch.float32 if top else dt, device=DEV),
                  "dw": torch.empty(hi - lo, dims[i - 1], device=DEV), "db": torch.empty(hi - lo, device=DEV),
                  "dx": torch.empty(b, dims[i - 1], device=DEV) if i > 1 else None}
            ly["dy_blk"] = ly["dy"][:, lo:hi]
            for which in (0, 1):
                need = max(need, imbd.mlp_local_workspace_bytes(which, code, hi - lo, dims[i - 1], b))
            layers.append(ly)
        loss, rows = torch.zeros(1, device=DEV), torch.zeros(b, device=DEV)
        out = {"loss": loss, "rows": rows, "dz": layers[-1]["dy"]}
        for i, ly in enumerate(layers):
            out.update({"%s%d" % (k, i): ly[k] for k in ("y", "dw", "db", "dx", "w") if ly[k] is not None})
            if case["dtype"] == "bf16":
                out["w_lp%d" % i] = ly["w_lp"]
        return {"case": case, "layers": layers, "P_r": P_r, "P_c": P_c, "lr": 0.01,
                "logits": _normal(g, b, dims[-1], scale=2.0),
                "labels": torch.randint(0, dims[-1], (b,), generator=g, device=DEV, dtype=torch.int32),
                "loss": loss, "rows": rows, "out": out,
                "ws": torch.empty(need, dtype=torch.uint8, device=DEV)}
    if case["kind"] == "conv":
        N, H, W, Ci, Co = (case[k] for k in ("N", "H", "W", "Ci", "Co"))
        odt = torch.bfloat16 if case["out"] == "bf16" else torch.float32
        x = _normal(g, N, H + 2, W + 2, Ci).clamp_(min=0.0)  # post-ReLU activations
        dy = _normal(g, N, H + 2, W + 2, Co)
        for t in (x, dy):  # a tile in a corner of the image: two halo sides are its border
            t[:, 0] = 0
            t[:, :, 0] = 0
        return {"case": case, "x": x.to(torch.bfloat16), "dy": dy.to(torch.bfloat16),
                "w": _normal(g, Co, 3, 3, Ci, scale=math.sqrt(2.0 / (9 * Ci))).to(torch.bfloat16),
                "y": torch.empty(N, H, W, Co, dtype=odt, device=DEV),
                "dx": torch.empty(N, H, W, Ci, dtype=odt, device=DEV),
                "dw": torch.empty(Co, 3, 3, Ci, device=DEV),
                "ws": torch.empty(max(16, imbd.conv3x3_wgrad_workspace_bytes(N, H, W, Ci, Co)), dtype=torch.uint8,
                                  device=DEV)}
    w = _normal(g, case["n"], scale=0.015)
    return {"case": case, "w": w, "w_lp": w.to(torch.bfloat16) if case["lp"] else None,
            "g": _normal(g, case["n"], scale=0.01), "lr": 0.01}


# ------------------------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    if case["kind"] == "step":
        imbd.mlp_train_step(state["net"], state["layers"], state["x"], state["labels"], state["ws"], state["lr"],
                            state["loss"])
        return state["out"]
    if case["kind"] == "grads":
        imbd.mlp_fwd(state["net"], state["layers"], state["x"], state["labels"], state["ws"], state["loss"])
        imbd.mlp_bwd(state["net"], state["layers"], state["x"], state["ws"], False, 0.0, dx1=state["dx1"])
        return state["out"]
    if case["kind"] == "grid":
        P_r, P_c, ws, layers = state["P_r"], state["P_c"], state["ws"], state["layers"]
        for ly in layers:
            imbd.mlp_local_fwd(ly["w_lp"], ly["x"], ly["y"], P_r, P_c, bias=ly["bias"], relu=not ly["top"], ws=ws)
        # the raw per-sample gradient of the gathered logits (the products apply 1/B)
        imbd.softmax_xent(state["logits"], state["labels"], 1.0, state["loss"], state["rows"], dz=layers[-1]["dy"])
        for i, ly in reversed(list(enumerate(layers))):
            imbd.mlp_local_bwd(ly["w_lp"], ly["dy_blk"], ly["x"], ly["dw"], P_r, P_c,
                               db_part=ly["db"], dx_part=ly["dx"], mask_relu=i > 0, ws=ws)
        for ly in layers:
            imbd.sgd_step(ly["w"], ly["dw"], state["lr"], w_lp=ly["w_lp"] if case["dtype"] == "bf16" else None)
        return state["out"]
    if case["kind"] == "conv":
        imbd.conv3x3_tile_fwd(state["x"], state["w"], state["y"])
        imbd.conv3x3_tile_bwd(state["x"], state["w"], state["dy"], state["dw"], dx=state["dx"], ws=state["ws"])
        return {"y": state["y"], "dx": state["dx"], "dw": state["dw"]}
    imbd.sgd_step(state["w"], state["g"], state["lr"], w_lp=state["w_lp"])
    out = {"w": state["w"]}
    if state["w_lp"] is not None:
        out["w_lp"] = state["w_lp"]
    return out


# ------------------------------------------------------------------------------------ what a pass needs
def work(case):
    """Each input read once and each output written once; the products' multiplications and additions."""
    if case["kind"] == "conv":
        N, H, W, Ci, Co = (case[k] for k in ("N", "H", "W", "Ci", "Co"))
        oe = 2 if case["out"] == "bf16" else 4
        read = 2 * N * (H + 2) * (W + 2) * (Ci + Co) + 2 * 9 * Ci * Co
        return {"bytes": read + oe * N * H * W * (Ci + Co) + 4 * 9 * Ci * Co,
                "flops": 3 * 2 * N * H * W * 9 * Ci * Co}
    if case["kind"] == "update":
        return {"bytes": case["n"] * (14 if case["lp"] else 12), "flops": 2 * case["n"]}
    dims, bf16 = _dims(case), case["dtype"] == "bf16"
    es, L = 2 if bf16 else 4, len(dims) - 1
    nbytes = flops = 0
    if case["kind"] == "grid":
        b = case["batch"] // case["P_c"]
        for i in range(1, L + 1):
            lo, hi = _block(dims[i], case["P_r"])
            p, m, k = (hi - lo) * dims[i - 1], hi - lo, dims[i - 1]
            # the operands, Delta_W, the master read and written and its copy written, Y, Delta_X
            nbytes += p * (es + 4 + 8 + (2 if bf16 else 0)) + b * (k * es + m * es) + 12 * m
            nbytes += b * m * (4 if i == L else es) + (4 * b * k if i > 1 else 0)
            flops += 2 * b * p * (3 if i > 1 else 2) + 2 * p
        nbytes += b * dims[-1] * (4 + es) + 12 * b
        return {"bytes": nbytes, "flops": flops}
    B = case["batch"]
    for i in range(1, L + 1):
        p = dims[i] * dims[i - 1]
        # the operand; the master read and written and its copy written, or the gradient written
        if case["kind"] == "step":
            nbytes += p * ((2 + 8 + 2) if bf16 else 8)
        else:
            nbytes += p * (es + 4)
        nbytes += 8 * dims[i]
        flops += 2 * B * p * (3 if i > 1 or case.get("dx1") else 2)
    nbytes += B * dims[0] * es * (2 if case.get("dx1") else 1) + B * dims[-1] * 4 + 4 * B
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "update":
        return {"rel": 1e-6, "max": 0.01}  # one fp32 rounding; the bf16 copy may round the other way
    if case["kind"] == "conv":
        # identical bf16 operands and fp32 sums (4e-7 off 64 bits); a bf16 output is rounded once (1.7e-3)
        return {"rel": 5e-3, "max": 0.02} if case["out"] == "bf16" else {"rel": 2e-6, "max": 1e-4}
    if case["kind"] == "grid":
        # single products of given operands: fp32 sums (6e-7 at most), one rounding of a bf16 output (1.7e-3)
        return {"rel": 5e-3, "max": 0.05} if case["dtype"] == "bf16" else {"rel": 2e-6, "max": 1e-4}
    if case["dtype"] == "f32":
        # sums of 3e-7, but past a hidden layer a pre-activation that close to zero may be kept or dropped by
        # the ReLU, which takes one sample's term from that unit's gradients (1.1e-3 of the bias gradient)
        return {"rel": 5e-3, "max": 0.9} if case["dims"].count("-") > 1 else {"rel": 2e-6, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.9}  # the same with bf16 activations and gradients between the layers


# ------------------------------------------------------------------------------------ the same in 64 bits
def _xent(z, labels, scale):
    z = z - z.max(dim=1, keepdim=True).values
    lse = z.exp().sum(dim=1).log()
    rows = lse - z.gather(1, labels.long()[:, None])[:, 0]
    dz = (z - lse[:, None]).exp()
    dz[torch.arange(z.shape[0], device=z.device), labels.long()] -= 1.0
    return rows, dz * scale


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "update":
        w = s["w"].double() - s["lr"] * s["g"].double()
        return {"w": w, "w_lp": w} if case["lp"] else {"w": w}
    if case["kind"] == "conv":
        x, w, dy = s["x"].double(), s["w"].double(), s["dy"].double()
        N, H, W = case["N"], case["H"], case["W"]
        y = torch.zeros(N * H * W, case["Co"], dtype=torch.float64, device=DEV)
        dx = torch.zeros(N * H * W, case["Ci"], dtype=torch.float64, device=DEV)
        dw = torch.empty_like(w)
        inner = dy[:, 1:H + 1, 1:W + 1].reshape(N * H * W, -1)
        for r in range(3):
            for c in range(3):
                xs = x[:, r:r + H, c:c + W].reshape(N * H * W, -1)
                y += xs @ w[:, r, c].t()
                dw[:, r, c] = inner.t() @ xs
                dx += dy[:, 2 - r:2 - r + H, 2 - c:2 - c + W].reshape(N * H * W, -1) @ w[:, r, c]
        return {"y": y.view(N, H, W, -1), "dx": dx.view(N, H, W, -1), "dw": dw}
    if case["kind"] == "grid":
        scale = 1.0 / (s["rows"].numel() * case["P_c"])
        rows, dz = _xent(s["logits"].double(), s["labels"], 1.0)
        out = {"loss": rows.sum().view(1), "rows": rows, "dz": dz}
        for i, ly in enumerate(s["layers"]):
            w, x = ly["w_lp"].double(), ly["x"].double()
            dy = (dz if ly["top"] else ly["dy"].double())[:, ly["lo"]:ly["hi"]]
            y = x @ w.t() + ly["bias"].double()
            out["y%d" % i] = y if ly["top"] else y.clamp(min=0.0)
            out["dw%d" % i] = scale * (dy.t() @ x)
            out["db%d" % i] = scale * dy.sum(dim=0)
            if i > 0:
                out["dx%d" % i] = (dy @ w) * (x > 0)
            nw = ly["w"].double() - s["lr"] * out["dw%d" % i]
            out["w%d" % i] = nw
            if case["dtype"] == "bf16":
                out["w_lp%d" % i] = nw
        return out
    ws = [ly["w_lp"].double() for ly in s["layers"]]
    acts, L = [s["x"].double()], len(ws)
    for i, w in enumerate(ws):
        y = acts[-1] @ w.t()
        acts.append(y if i == L - 1 else y.clamp(min=0.0))
    rows, dy = _xent(acts[-1], s["labels"], 1.0 / case["batch"])
    out = {"loss": rows.mean().view(1), "logits": acts[-1]}
    for i in range(L - 1, -1, -1):
        dw, db = dy.t() @ acts[i], dy.sum(dim=0)
        if i > 0:
            dy = (dy @ ws[i]) * (acts[i] > 0)
        elif case.get("dx1"):
            out["dx1"] = dy @ ws[i]
        if case["kind"] == "grads":
            out["dw%d" % i], out["db%d" % i] = dw, db
        else:
            out["w%d" % i] = s["layers"][i]["w"].double() - s["lr"] * dw
            out["b%d" % i] = s["layers"][i]["b"].double() - s["lr"] * db
        if case["dtype"] == "f32" and i < L - 1:
            # the error of these is the few ReLU decisions that fp32 sums take the other way (see tolerance)
            out.update({k: None for k in ("dw%d" % i, "db%d" % i, "b%d" % i, "dx1") if k in out})
        if case["kind"] == "grads":
            continue
        if case["dtype"] == "bf16":
            out["w_lp%d" % i] = out["w%d" % i]
    return out
