"""The work that is timed when this library is made faster: training passes through the binding's entry points.

Six families, each a stretch of a mixed-precision training step as a program of the library's user runs it:

  mlp        one step of a two-layer perceptron: both layers forward, loss, both backward, one update of all weights
  layer      the three products of one dense layer, with or without its ReLU, and if asked the update of its weight
  recurrent  a projected-LSTM layer over T time steps, forward ("fwd") or back through time ("bwd")
  conv       a 3x3 convolution with batch normalisation and ReLU, forward and backward
  update     the optimizer's part of a step on a flat buffer or on many tensors: overflow test, clipping, update, loss scale
  loss       softmax cross-entropy with the loss scale in its gradient

`listed()` holds the sizes that stand for each family, `draw()` gives others of the same ranges.  Inputs are synthetic,
made on the GPU from the seed.  Splitting products get the workspace that the library asks for, as a program that
allocates once and keeps it would give them.
"""
import math

import torch

from paper_1710_03740_amd import binding as mpt

F16, F32 = torch.float16, torch.float32


# ---------------------------------------------------------------- cases
def listed():
    return [
        # The smallest training step the repository is run with: launches and latencies.
        {"name": "mlp 256x1024-1024-10", "family": "mlp", "batch": 256, "d_in": 1024, "d_hid": 1024, "d_out": 10, "momentum": False},
        # The same of a still smaller network whose rows are not whole 16-byte chunks, with momentum.
        {"name": "mlp 100x500-300-10", "family": "mlp", "batch": 100, "d_in": 500, "d_hid": 300, "d_out": 10, "momentum": True},
        # The benchmark's step: a large square layer, all three products, and the update of its weight.
        {"name": "layer 4096", "family": "layer", "M": 4096, "N": 4096, "K": 4096, "relu": False, "grad32": False, "update": True},
        # A middle-sized hidden layer with its ReLU; no size is a multiple of a tile.
        {"name": "layer 2000x3000x1000 relu", "family": "layer", "M": 2000, "N": 3000, "K": 1000, "relu": True, "grad32": False, "update": False},
        # Odd sizes in every direction (a vocabulary, a hand-picked width), weight gradient kept in FP32, with its update.
        {"name": "layer 1001x1999x1503 grad32", "family": "layer", "M": 1001, "N": 1999, "K": 1503, "relu": False, "grad32": True, "update": True},
        # The language model's recurrent layer, 20 time steps of batch 256, forward with all that the backward pass needs ...
        {"name": "recurrent fwd 20x256", "family": "recurrent", "direction": "fwd", "T": 20, "B": 256, "I": 1024, "H": 8192, "R": 1024},
        # ... and backward: per-step gradients, the projection's weight gradient summed in FP32 over the steps.
        {"name": "recurrent bwd 20x256", "family": "recurrent", "direction": "bwd", "T": 20, "B": 256, "I": 1024, "H": 8192, "R": 1024},
        # The middle stage of an image network: 256 channels at 14 x 14.
        {"name": "conv 256x14x14x256", "family": "conv", "Nb": 256, "H": 14, "W": 14, "C": 256, "Kf": 256},
        # Its first stage: few channels, many positions.
        {"name": "conv 64x56x56x64", "family": "conv", "Nb": 64, "H": 56, "W": 56, "C": 64, "Kf": 64},
        # Dynamic loss scaling and momentum over all weights of the speech model.
        {"name": "update 116M momentum", "family": "update", "kind": "momentum", "n": 116_000_000, "tensors": 1, "grad32": False, "clip": False, "overflow": False},
        # Adam with the gradient clipped by its norm; a length with a ragged end.
        {"name": "update 25M adam clip", "family": "update", "kind": "adam", "n": 25_000_003, "tensors": 1, "grad32": False, "clip": True, "overflow": False},
        # The language model's loss: 20 steps of batch 256 over a 32768-word vocabulary.
        {"name": "loss 5120x32768", "family": "loss", "B": 5120, "C": 32768},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _size(rng, lo, hi, grain=None):
    """A size between lo and hi, spread over the logarithm: a third multiples of 64 where the range has room for them, a
    third multiples of 8, a third anything (grain: the least multiple that the entry point takes)."""
    x = _log(rng, lo, hi)
    g = rng.choice((64, 8, 1))
    if grain is not None:
        g = max(g, grain)
    if g > lo:
        g = grain or 1
    return int(min(hi, max(lo, round(x / g) * g)))


def draw(rng):
    family = rng.choice(("mlp", "layer", "layer", "recurrent", "conv", "update", "loss"))
    if family == "mlp":
        return {"family": family, "batch": _size(rng, 32, 1024), "d_in": _size(rng, 128, 2048), "d_hid": _size(rng, 128, 2048),
                "d_out": _size(rng, 10, 1000), "momentum": rng.random() < 0.5}
    if family == "layer":
        return {"family": family, "M": _size(rng, 64, 4096), "N": _size(rng, 256, 4096), "K": _size(rng, 256, 4096), "relu": rng.random() < 0.5,
                "grad32": rng.random() < 0.25, "update": rng.random() < 0.5}
    if family == "recurrent":
        return {"family": family, "direction": rng.choice(("fwd", "bwd")), "T": rng.randint(2, 20), "B": _size(rng, 16, 256), "I": _size(rng, 128, 1024),
                "H": _size(rng, 256, 8192), "R": _size(rng, 128, 1024)}
    if family == "conv":
        hw = rng.choice((7, 13, 14, 28, 35, 56))
        C, Kf = _size(rng, 32, 512, 8), _size(rng, 32, 512, 8)
        most = 256 * 14 * 14 * 256 * 256 // (hw * hw * C * Kf)               # the work of the first listed one
        return {"family": family, "Nb": _size(rng, 1, max(1, min(256, most, 51_380_224 // (hw * hw * max(C, Kf))))), "H": hw, "W": hw, "C": C, "Kf": Kf}
    if family == "update":
        kind = rng.choice(("momentum", "momentum", "fused", "nesterov", "adagrad", "adam", "stats"))
        n = int(_log(rng, 20_000, 116_000_000 if kind != "adam" else 80_000_000))
        tensors = rng.choice((1, rng.randint(2, 60))) if kind == "momentum" else 1
        return {"family": family, "kind": kind, "n": n, "tensors": tensors, "grad32": kind != "stats" and rng.random() < 0.3,
                "clip": kind in ("nesterov", "adagrad", "adam") and rng.random() < 0.6, "overflow": rng.random() < 0.15}
    C = _size(rng, 10, 65536)
    return {"family": family, "B": _size(rng, 16, min(8192, 5120 * 32768 // C)), "C": C}


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std=1.0, dtype=F16):
    return torch.empty(shape, device="cuda", dtype=F32).normal_(0.0, std, generator=g).to(dtype)


def _uniform(g, shape, lo, hi, dtype=F16):
    return torch.empty(shape, device="cuda", dtype=F32).uniform_(lo, hi, generator=g).to(dtype)


def _log_uniform(g, shape, lo, hi, scale, dtype=F16):
    """scale * 2^u with u uniform in [lo, hi) and a random sign: the spread of magnitudes that gradients have."""
    u = torch.empty(shape, device="cuda", dtype=F32).uniform_(lo, hi, generator=g).exp2_().mul_(scale)
    u.copysign_(torch.empty(shape, device="cuda", dtype=F32).uniform_(-1.0, 1.0, generator=g))
    return u.to(dtype)


def _empty(*shape, dtype=F16):
    return torch.empty(shape, device="cuda", dtype=dtype)


def _workspace(*byte_counts):
    need = max(byte_counts)
    return torch.empty((need + 3) // 4, device="cuda", dtype=F32) if need else None


def _gemm_ws(M, N, K):
    return [mpt.mpt_gemm_workspace_bytes(op, M, N, K) for op in (mpt.OP_FWD, mpt.OP_DGRAD, mpt.OP_WGRAD)]


def _flag():
    return torch.zeros(1, device="cuda", dtype=torch.int32)


# ---------------------------------------------------------------- mlp
def _prepare_mlp(c, g):
    b, i, h, o = c["batch"], c["d_in"], c["d_hid"], c["d_out"]
    a1, a2 = math.sqrt(6.0 / (i + h)), math.sqrt(6.0 / (h + o))
    w1, w2 = _uniform(g, (i, h), -a1, a1, F32), _uniform(g, (h, o), -a2, a2, F32)
    m1, m2 = (torch.zeros_like(w1), torch.zeros_like(w2)) if c["momentum"] else (None, None)
    s = {"x": _normal(g, (b, i)), "labels": torch.randint(0, o, (b,), device="cuda", dtype=torch.int32, generator=g),
         "w1": w1.half(), "w2": w2.half(), "flag": _flag(), "loss": _empty(1, dtype=F32), "rows": _empty(b, dtype=F32),
         "h": _empty(b, h), "logits": _empty(b, o), "dlogits": _empty(b, o), "dy": _empty(b, h), "dw1": _empty(i, h), "dw2": _empty(h, o),
         "ws": _workspace(*_gemm_ws(b, h, i), *_gemm_ws(b, o, h))}
    s["weights"] = ((w1, m1, s["dw1"], s["w1"]), (w2, m2, s["dw2"], s["w2"]))
    s["momentum"] = 0.9 if c["momentum"] else 0.0
    return s


def _run_mlp(s):
    ws, flag = s["ws"], s["flag"]
    mpt.mpt_gemm_fwd_relu(s["x"], s["w1"], s["h"], ws)
    mpt.mpt_gemm_fwd(s["h"], s["w2"], s["logits"], ws)
    mpt.mpt_softmax_xent_scaled(s["logits"], s["labels"], 1024.0, s["dlogits"], s["loss"], s["rows"])
    mpt.mpt_gemm_wgrad(s["h"], s["dlogits"], s["dw2"], flag=flag, ws=ws)
    mpt.mpt_gemm_dgrad_relu(s["dlogits"], s["w2"], s["h"], s["dy"], ws)
    mpt.mpt_gemm_wgrad(s["x"], s["dy"], s["dw1"], flag=flag, ws=ws)
    mpt.mpt_master_update_multi(s["weights"], 1.0 / 1024.0, 0.01, s["momentum"], flag)
    (w1, m1, dw1, w1h), (w2, m2, dw2, w2h) = s["weights"]
    return {"loss": s["loss"], "logits": s["logits"], "dw1": dw1, "dw2": dw2, "w1": w1, "w2": w2, "m1": m1, "m2": m2, "w1h": w1h, "w2h": w2h, "flag": flag}


def _work_mlp(c):
    b, i, h, o = c["batch"], c["d_in"], c["d_hid"], c["d_out"]
    weights = i * h + h * o
    # x and the weights read, activations and gradients of both layers written and read back, the update's streams
    bytes_ = 2 * b * i * 2 + 2 * weights * 2 + b * (2 * h * 2 * 2 + 2 * o * 2 * 2) + weights * (2 + (20 if c["momentum"] else 12))
    return {"bytes": bytes_, "flops": 2.0 * b * (2 * i * h + 3 * h * o)}


# ---------------------------------------------------------------- layer
def _prepare_layer(c, g):
    M, N, K = c["M"], c["N"], c["K"]
    w32 = _normal(g, (K, N), 0.05, F32)
    s = {"x": _normal(g, (M, K), 0.05), "w": w32.half(), "g": _log_uniform(g, (M, N), -30.0, -5.0, 8192.0), "y": _empty(M, N), "dx": _empty(M, K),
         "dw": _empty(K, N, dtype=F32 if c["grad32"] else F16), "flag": _flag(), "ws": _workspace(*_gemm_ws(M, N, K)), "relu": c["relu"]}
    if c["relu"]:
        s["x"].relu_()                                                      # the output of the ReLU below, which is also the backward mask
    if c["update"]:
        s.update(w32=w32, m32=torch.zeros_like(w32), scaler=mpt.scaler_to_device(mpt.mpt_scaler_init(8192.0, 1000)))
    return s


def _run_layer(s):
    if s["relu"]:
        mpt.mpt_gemm_fwd_relu(s["x"], s["w"], s["y"], s["ws"])
        mpt.mpt_gemm_dgrad_relu(s["g"], s["w"], s["x"], s["dx"], s["ws"])
    else:
        mpt.mpt_gemm_fwd(s["x"], s["w"], s["y"], s["ws"])
        mpt.mpt_gemm_dgrad(s["g"], s["w"], s["dx"], s["ws"])
    mpt.mpt_gemm_wgrad(s["x"], s["g"], s["dw"], flag=s["flag"], ws=s["ws"])
    out = {"y": s["y"], "dx": s["dx"], "dw": s["dw"], "flag": s["flag"]}
    if "w32" in s:
        mpt.mpt_master_update(s["w32"], s["m32"], s["dw"], s["w"], 1.0, 1e-3, 0.9, s["flag"], scaler_dev=s["scaler"])
        mpt.mpt_loss_scale_update_dev(s["scaler"], s["flag"])
        out.update(w32=s["w32"], m32=s["m32"], w=s["w"], scaler=s["scaler"])
    return out


def _work_layer(c):
    M, N, K = c["M"], c["N"], c["K"]
    gsz = 4 if c["grad32"] else 2
    bytes_ = 3 * 2 * (M * K + K * N + M * N) - 2 * K * N + gsz * K * N + (2 * M * K if c["relu"] else 0)
    return {"bytes": bytes_ + (K * N * (18 + gsz) if c["update"] else 0), "flops": 6.0 * M * N * K}


# ---------------------------------------------------------------- recurrent
def _prepare_recurrent(c, g):
    T, B, I, H, R = c["T"], c["B"], c["I"], c["H"], c["R"]
    s = {"direction": c["direction"], "T": T, "x": _normal(g, (T * B, I)), "wx": _normal(g, (I, 4 * H), 1.0 / math.sqrt(I)),
         "wr": _normal(g, (R, 4 * H), 1.0 / math.sqrt(R)), "wp": _normal(g, (H, R), 1.0 / math.sqrt(H))}
    steps = lambda t, n=T: [t[k * B:(k + 1) * B] for k in range(n)]  # noqa: E731
    if c["direction"] == "fwd":
        gx, act = _empty(T * B, 4 * H), _empty(T * B, 4 * H)
        cell, out = torch.zeros((T + 1) * B, H, device="cuda", dtype=F16), torch.zeros((T + 1) * B, R, device="cuda", dtype=F16)
        h = _empty(T * B, H)
        s.update(gx=gx, gr=_empty(B, 4 * H), act=act, cell=cell, h=h, r=out, gx_t=steps(gx), act_t=steps(act), cell_t=steps(cell, T + 1), h_t=steps(h),
                 r_t=steps(out, T + 1), ws=_workspace(_gemm_ws(T * B, 4 * H, I)[0], _gemm_ws(B, 4 * H, R)[0], _gemm_ws(B, R, H)[0]))
        return s
    # what the forward pass stored: gates behind their sigmoid / tanh, states, outputs; and the gradient from above
    act = _uniform(g, (T * B, 4 * H), 0.02, 0.98)
    act[:, 2 * H:3 * H].mul_(2.0).sub_(1.0)
    cell, h, r = _normal(g, ((T + 1) * B, H)), _uniform(g, (T * B, H), -0.7, 0.7), _normal(g, ((T + 1) * B, R), 0.4)
    dr = _log_uniform(g, (T * B, R), -30.0, -5.0, 128.0)
    da, dr_all = _empty(T * B, 4 * H), _empty(T * B, R)
    s.update(act_t=steps(act), cell_t=steps(cell, T + 1), h_t=steps(h), r=r[:T * B], dr_t=steps(dr), da=da, da_t=steps(da), drall_t=steps(dr_all), dr_all=dr_all,
             dh=_empty(B, H), dc=_empty(B, H), drec=torch.zeros(B, R, device="cuda", dtype=F16), dx=_empty(T * B, I), dwx=_empty(I, 4 * H), dwr=_empty(R, 4 * H),
             dwp=torch.zeros(H, R, device="cuda", dtype=F32), flag=_flag(),
             ws=_workspace(_gemm_ws(B, R, H)[1], _gemm_ws(B, R, H)[2], _gemm_ws(B, 4 * H, R)[1], *_gemm_ws(T * B, 4 * H, I)[1:], _gemm_ws(T * B, 4 * H, R)[2]))
    return s


def _run_recurrent(s):
    T, ws = s["T"], s["ws"]
    if s["direction"] == "fwd":
        mpt.mpt_gemm_fwd(s["x"], s["wx"], s["gx"], ws)
        for t in range(T):
            mpt.mpt_gemm_fwd(s["r_t"][t], s["wr"], s["gr"], ws)
            mpt.mpt_lstm_cell_fwd(s["gx_t"][t], s["gr"], None, s["cell_t"][t], s["act_t"][t], s["cell_t"][t + 1], s["h_t"][t])
            mpt.mpt_gemm_fwd(s["h_t"][t], s["wp"], s["r_t"][t + 1], ws)
        return {"r": s["r"], "h": s["h"], "cell": s["cell"], "act": s["act"]}
    for t in range(T - 1, -1, -1):
        last = t == T - 1
        dr = s["dr_t"][t] if last else s["drall_t"][t]
        if not last:
            mpt.mpt_add_fp16(s["dr_t"][t], s["drec"], dr)                   # from above and from the next step
        mpt.mpt_gemm_dgrad(dr, s["wp"], s["dh"], ws)
        mpt.mpt_lstm_cell_bwd(s["dh"], None if last else s["dc"], s["act_t"][t], s["cell_t"][t + 1], s["cell_t"][t], s["da_t"][t], s["dc"])
        mpt.mpt_gemm_wgrad(s["h_t"][t], dr, s["dwp"], accumulate=not last, flag=s["flag"] if t == 0 else None, ws=ws)
        if t:
            mpt.mpt_gemm_dgrad(s["da_t"][t], s["wr"], s["drec"], ws)
    mpt.mpt_gemm_dgrad(s["da"], s["wx"], s["dx"], ws)
    mpt.mpt_gemm_wgrad(s["x"], s["da"], s["dwx"], flag=s["flag"], ws=ws)
    mpt.mpt_gemm_wgrad(s["r"], s["da"], s["dwr"], flag=s["flag"], ws=ws)
    return {"dx": s["dx"], "dwx": s["dwx"], "dwr": s["dwr"], "dwp": s["dwp"], "da": s["da"], "dc": s["dc"], "flag": s["flag"]}


def _work_recurrent(c):
    T, B, I, H, R = c["T"], c["B"], c["I"], c["H"], c["R"]
    products = 2.0 * T * B * (I * 4 * H + R * 4 * H + H * R)
    # Weights once per step they are used in (a step ends before the next begins), time-batched tensors once per call.
    if c["direction"] == "fwd":
        per_step = R * 4 * H + H * R + B * (4 * H * 4 + H * 3 + 2 * R)
        once = T * B * (I + 4 * H) + I * 4 * H
        return {"bytes": 2.0 * (T * per_step + once), "flops": products}
    per_step = R * 4 * H + H * R + B * (4 * H * 3 + H * 6 + 4 * R) + 4 * H * R
    once = T * B * (3 * 4 * H + 2 * I + R) + 2 * I * 4 * H + R * 4 * H
    return {"bytes": 2.0 * (T * per_step + once), "flops": 2.0 * products}


# ---------------------------------------------------------------- conv
def _prepare_conv(c, g):
    Nb, H, W, C, Kf = c["Nb"], c["H"], c["W"], c["C"], c["Kf"]
    P = Nb * H * W
    dz = _normal(g, (Nb, H, W, Kf), 2.0 ** -6)
    s = {"x": _normal(g, (Nb, H, W, C)).relu_(), "w": _normal(g, (Kf, 3, 3, C), math.sqrt(2.0 / (9 * C))), "dz": dz, "y": _empty(Nb, H, W, Kf),
         "z": _empty(Nb, H, W, Kf), "dzm": _empty(Nb, H, W, Kf), "dy": _empty(Nb, H, W, Kf), "dx": _empty(Nb, H, W, C), "dw": _empty(Kf, 3, 3, C), "flag": _flag(),
         "gamma": _uniform(g, (Kf,), 0.5, 1.5, F32), "beta": _uniform(g, (Kf,), -0.5, 0.5, F32), "mean": _empty(Kf, dtype=F32), "var": _empty(Kf, dtype=F32),
         "dgamma": _empty(Kf, dtype=F32), "dbeta": _empty(Kf, dtype=F32),
         "ws": _workspace(*[mpt.mpt_conv3x3_workspace_bytes(op, Nb, H, W, C, Kf) for op in (mpt.OP_FWD, mpt.OP_DGRAD, mpt.OP_WGRAD)]),
         "bn_ws": _workspace(mpt.mpt_bn_workspace_bytes(P, Kf))}
    for k in ("y", "z", "dzm", "dy"):
        s[k + "2"] = s[k].view(P, Kf)
    return s


def _run_conv(s):
    eps, ws = 1e-5, s["ws"]
    mpt.mpt_conv3x3_fwd(s["x"], s["w"], s["y"], ws)
    mpt.mpt_bn_stats(s["y2"], s["mean"], s["var"], s["bn_ws"])
    mpt.mpt_bn_apply(s["y2"], s["mean"], s["var"], s["gamma"], s["beta"], eps, s["z2"], relu=True)
    mpt.mpt_relu_bwd(s["dz"], s["z"], s["dzm"])
    mpt.mpt_bn_bwd_reduce(s["y2"], s["dzm2"], s["mean"], s["var"], eps, s["dgamma"], s["dbeta"], s["bn_ws"])
    mpt.mpt_bn_bwd_apply(s["y2"], s["dzm2"], s["mean"], s["var"], s["gamma"], eps, s["dgamma"], s["dbeta"], s["dy2"])
    mpt.mpt_conv3x3_dgrad(s["dy"], s["w"], s["dx"], ws)
    mpt.mpt_conv3x3_wgrad(s["x"], s["dy"], s["dw"], flag=s["flag"], ws=ws)
    return {"y": s["y"], "z": s["z"], "dx": s["dx"], "dw": s["dw"], "mean": s["mean"], "var": s["var"], "dgamma": s["dgamma"], "dbeta": s["dbeta"], "flag": s["flag"]}


def _work_conv(c):
    P, C, Kf = c["Nb"] * c["H"] * c["W"], c["C"], c["Kf"]
    # each call's tensors once: the three products, then statistics 1, apply 2, ReLU 3, reductions 2, gradient 3 of P x Kf
    return {"bytes": 2.0 * (3 * (P * C + P * Kf + 9 * C * Kf) + 11 * P * Kf), "flops": 6.0 * P * 9 * C * Kf}


# ---------------------------------------------------------------- update
def _prepare_update(c, g):
    n, kind = c["n"], c["kind"]
    gdt = F32 if c["grad32"] else F16
    if kind == "stats":
        grad = _log_uniform(g, (n,), -28.0, -2.0, 65536.0)
        if c["overflow"]:
            grad[n // 3] = math.inf
        return {"kind": kind, "grad": grad, "hist": torch.zeros(42, device="cuda", dtype=torch.int64), "absmax": torch.zeros(1, device="cuda", dtype=torch.int32)}
    s = {"kind": kind, "flag": _flag(), "scaler": mpt.scaler_to_device(mpt.mpt_scaler_init(65536.0, 1000)), "clip": c["clip"]}
    if kind == "momentum" and c["tensors"] > 1:
        cuts = [n * k * k // (c["tensors"] * c["tensors"]) for k in range(c["tensors"] + 1)]     # small tensors and large ones
        sizes = [b - a for a, b in zip(cuts, cuts[1:])]
    else:
        sizes = [n]
    s["items"] = []
    for k, size in enumerate(sizes):
        w = _uniform(g, (size,), -0.05, 0.05, F32)
        grad = _log_uniform(g, (size,), -28.0, -2.0, 65536.0, gdt)
        if c["overflow"] and k == 0:
            grad[size // 3] = math.inf
        s["items"].append((w, torch.zeros_like(w), grad, w.half()))
    w, m, grad, w16 = s["items"][0]
    if kind == "fused":
        s["sets"] = [(w, m, w16), (torch.empty_like(w), torch.empty_like(m), torch.empty_like(w16))]
    if kind in mpt.OPT_KINDS and kind != "momentum":
        s["second"] = torch.zeros_like(w) if kind == "adam" else None
        s["sumsq"], s["factor"], s["norm"] = _empty(1, dtype=torch.float64), _empty(1, dtype=F32), _empty(1, dtype=F32)
        s["norm_ws"] = torch.empty(mpt.mpt_grad_norm_workspace_bytes(), device="cuda", dtype=torch.uint8)
        mu, b2, step = 0.9, 0.999, 10
        s["hp"] = mpt.mpt_opt_params(1e-3, mu, b2, 1e-8, 0.0, 1.0 - mu, 1.0 - b2, 1.0 - mu ** step, 1.0 - b2 ** step,
                                     s["factor"].data_ptr() if c["clip"] else None)
    return s


def _run_update(s):
    kind = s["kind"]
    if kind == "stats":
        mpt.mpt_grad_stats(s["grad"], s["hist"], s["absmax"])
        return {"hist": s["hist"], "absmax": s["absmax"]}
    flag, scaler, items = s["flag"], s["scaler"], s["items"]
    w, m, grad, w16 = items[0]
    out = {"scaler": scaler}
    if kind == "fused":
        (w, m, w16), (w_new, m_new, w16_new) = s["sets"]
        mpt.mpt_master_update_fused(w, m, grad, w_new, m_new, w16_new, 1.0, 1e-3, 0.9, flag, scaler_dev=scaler)
        out["flag"] = flag.clone()                                          # what the program reads to adopt the new set or drop it
        mpt.mpt_loss_scale_update_dev(scaler, flag)
        out.update(w=w_new, m=m_new, w16=w16_new)
        return out
    if kind == "momentum":
        for _, _, gr, _ in items:
            mpt.mpt_unscale_check(gr, 2.0 ** -16, flag)
        if len(items) == 1:
            mpt.mpt_master_update(w, m, grad, w16, 1.0, 1e-3, 0.9, flag, scaler_dev=scaler)
        else:
            mpt.mpt_master_update_multi(items, 1.0, 1e-3, 0.9, flag, scaler_dev=scaler)
        out["items"] = [t for it in items[-16:] for t in (it[0], it[1], it[3])]
    else:
        if s["clip"]:
            mpt.mpt_grad_sumsq(grad, 1.0, s["sumsq"], s["norm_ws"], flag=flag, scaler_dev=scaler)
            mpt.mpt_clip_factor(s["sumsq"], 1.0, s["factor"], s["norm"])
            out.update(norm=s["norm"])
        else:
            mpt.mpt_unscale_check(grad, 2.0 ** -16, flag)
        mpt.mpt_optimizer_update(kind, s["hp"], w, m, s["second"], grad, w16, 1.0, flag, scaler_dev=scaler)
        out.update(w=w, m=m, second=s["second"], w16=w16)
    mpt.mpt_loss_scale_update_dev(scaler, flag)
    return out


def _work_update(c):
    n, gsz = c["n"], 4 if c["grad32"] else 2
    if c["kind"] == "stats":
        return {"bytes": n * gsz, "flops": n}
    if c["kind"] == "fused":
        return {"bytes": n * (18 + gsz), "flops": 6.0 * n}
    if c["overflow"]:                                                       # the test finds it and the update writes nothing
        return {"bytes": n * gsz, "flops": n}
    state = 26 if c["kind"] == "adam" else 18
    return {"bytes": n * (state + 2 * gsz), "flops": (14.0 if c["kind"] == "adam" else 6.0) * n}


# ---------------------------------------------------------------- loss
def _prepare_loss(c, g):
    B, C = c["B"], c["C"]
    return {"logits": _normal(g, (B, C), 3.0), "labels": torch.randint(0, C, (B,), device="cuda", dtype=torch.int32, generator=g), "dlogits": _empty(B, C),
            "loss": _empty(1, dtype=F32), "rows": _empty(B, dtype=F32)}


def _run_loss(s):
    mpt.mpt_softmax_xent_scaled(s["logits"], s["labels"], 128.0, s["dlogits"], s["loss"], s["rows"])
    return {"loss": s["loss"], "rows": s["rows"], "dlogits": s["dlogits"]}


def _work_loss(c):
    return {"bytes": c["B"] * (4.0 * c["C"] + 8), "flops": 5.0 * c["B"] * c["C"]}


# ---------------------------------------------------------------- the same results in 64 bits
# Plain torch in FP64 from the same inputs, nothing rounded on the way.  Flags, counters and the scaler's record have no such value.
_F64 = torch.float64


def _d(t):
    return t.to(_F64)


def _f32(x):
    return torch.tensor(x, dtype=F32).item()                                 # a parameter as the entry points take it


def _softmax_xent(z, labels, scale):
    p = torch.log_softmax(z, 1)
    rows = -p.gather(1, labels.long()[:, None])[:, 0]
    grad = p.exp_().scatter_add_(1, labels.long()[:, None], torch.full((z.shape[0], 1), -1.0, device="cuda", dtype=_F64))
    return rows, grad.mul_(scale / z.shape[0])


def _exact_mlp(s):
    x, (w1, _, _, h1), (w2, _, _, h2) = _d(s["x"]), *s["weights"]
    h1, h2 = _d(h1), _d(h2)
    h = torch.relu(x @ h1)
    logits = h @ h2
    rows, dlogits = _softmax_xent(logits, s["labels"], 1024.0)
    dw2, dw1 = h.t() @ dlogits, x.t() @ ((dlogits @ h2.t()) * (h > 0))
    m1, m2 = dw1 / 1024.0, dw2 / 1024.0                                     # momentum starts at zero
    w1, w2 = _d(w1) - _f32(0.01) * m1, _d(w2) - _f32(0.01) * m2
    mom = s["momentum"] != 0.0
    return {"loss": rows.mean().reshape(1), "logits": logits, "dw1": dw1, "dw2": dw2, "w1": w1, "w2": w2, "m1": m1 if mom else None,
            "m2": m2 if mom else None, "w1h": w1, "w2h": w2, "flag": None}


def _exact_layer(s):
    x, w, g = _d(s["x"]), _d(s["w"]), _d(s["g"])
    y, dx, dw = x @ w, g @ w.t(), x.t() @ g
    if s["relu"]:
        y, dx = torch.relu(y), dx * (x > 0)
    out = {"y": y, "dx": dx, "dw": dw, "flag": None}
    if "w32" in s:
        m = dw / 8192.0
        w = _d(s["w32"]) - _f32(1e-3) * m
        out.update(w32=w, m32=m, w=w, scaler=None)
    return out


def _exact_recurrent(s):
    T, (R, H4), wp = s["T"], s["wr"].shape, _d(s["wp"])
    x, wx, wr, H = _d(s["x"]), _d(s["wx"]), _d(s["wr"]), H4 // 4
    B = x.shape[0] // T
    if s["direction"] == "fwd":
        gx, c, r = x @ wx, torch.zeros(B, H, device="cuda", dtype=_F64), torch.zeros(B, R, device="cuda", dtype=_F64)
        rs, hs, cs, acts = [r], [], [c], []
        for t in range(T):
            i, f, g, o = (gx[t * B:(t + 1) * B] + r @ wr).split(H, 1)
            i, f, g, o = torch.sigmoid(i), torch.sigmoid(f), torch.tanh(g), torch.sigmoid(o)
            c = f * c + i * g
            h = o * torch.tanh(c)
            r = h @ wp
            rs.append(r), hs.append(h), cs.append(c), acts.append(torch.cat((i, f, g, o), 1))
        return {"r": torch.cat(rs), "h": torch.cat(hs), "cell": torch.cat(cs), "act": torch.cat(acts)}
    das, dwp, drec, dc = [None] * T, torch.zeros(H, R, device="cuda", dtype=_F64), 0.0, 0.0
    for t in range(T - 1, -1, -1):
        dr = _d(s["dr_t"][t]) + drec
        dh = dr @ wp.t()
        i, f, g, o = _d(s["act_t"][t]).split(H, 1)
        tc = torch.tanh(_d(s["cell_t"][t + 1]))
        d = dh * o * (1.0 - tc * tc) + dc
        das[t] = torch.cat((d * g * i * (1.0 - i), d * _d(s["cell_t"][t]) * f * (1.0 - f), d * i * (1.0 - g * g), dh * tc * o * (1.0 - o)), 1)
        dc = d * f
        dwp += _d(s["h_t"][t]).t() @ dr
        drec = das[t] @ wr.t()
    da = torch.cat(das)
    return {"dx": da @ wx.t(), "dwx": x.t() @ da, "dwr": _d(s["r"]).t() @ da, "dwp": dwp, "da": da, "dc": dc, "flag": None}


def _taps(t):
    """The nine shifted copies of an image tensor (zero outside), as matrices of its pixels."""
    Nb, H, W, C = t.shape
    p = torch.zeros(Nb, H + 2, W + 2, C, device="cuda", dtype=_F64)
    p[:, 1:-1, 1:-1] = t
    for k in range(9):
        yield k, p[:, k // 3:k // 3 + H, k % 3:k % 3 + W].reshape(-1, C)


def _exact_conv(s):
    w, gamma, eps = _d(s["w"]), _d(s["gamma"]), _f32(1e-5)
    Kf, _, _, C = w.shape
    w = w.reshape(Kf, 9, C)
    y = sum(x @ w[:, k].t() for k, x in _taps(s["x"]))
    mean, var = y.mean(0), y.var(0, unbiased=False)
    istd = 1.0 / torch.sqrt(var + eps)
    xh = (y - mean) * istd
    z = torch.relu(gamma * xh + _d(s["beta"]))
    dz = _d(s["dz"]).reshape(-1, Kf) * (z > 0)
    dgamma, dbeta = (dz * xh).sum(0), dz.sum(0)
    dy = (gamma * istd * (dz - dbeta / len(y) - xh * (dgamma / len(y)))).reshape(s["dz"].shape)
    dx = sum(g @ w[:, 8 - k] for k, g in _taps(dy))
    dy = dy.reshape(-1, Kf)
    dw = torch.stack([dy.t() @ x for _, x in _taps(s["x"])], 1)
    return {"y": y.reshape(s["y"].shape), "z": z.reshape(s["z"].shape), "dx": dx.reshape(s["dx"].shape), "dw": dw.reshape(s["dw"].shape), "mean": mean, "var": var,
            "dgamma": dgamma, "dbeta": dbeta, "flag": None}


def _exact_update(s):
    kind = s["kind"]
    if kind == "stats" or not all(torch.isfinite(it[2]).all() for it in s["items"]):
        return None                                                         # counts, or a step that is to be dropped
    lr, mu, inv, out = _f32(1e-3), _f32(0.9), 2.0 ** -16, {"scaler": None}
    if kind in ("momentum", "fused"):
        res = []
        for w, _, grad, _ in s["items"][-16:]:
            m = _d(grad) * inv
            w = _d(w) - lr * m
            res += [w, m, w]
        if kind == "fused":
            out.update(flag=None, w=res[0], m=res[1], w16=res[2])
        else:
            out["items"] = res
        return out
    w, _, grad, _ = s["items"][0]
    g = _d(grad) * inv
    if s["clip"]:
        norm = g.norm()
        g *= min(1.0, 1.0 / norm.item())
        out["norm"] = norm.reshape(1)
    second = None
    if kind == "nesterov":
        m, step = g, lr * (g + mu * g)
    elif kind == "adagrad":
        m = g * g
        step = lr * g / (m.sqrt() + _f32(1e-8))
    else:
        m, second = _f32(1.0 - 0.9) * g, _f32(1.0 - 0.999) * g * g
        step = lr * (m / _f32(1.0 - 0.9 ** 10)) / ((second / _f32(1.0 - 0.999 ** 10)).sqrt() + _f32(1e-8))
    w = _d(w) - step
    out.update(w=w, m=m, second=second, w16=w)
    return out


def _exact_loss(s):
    rows, grad = _softmax_xent(_d(s["logits"]), s["labels"], 128.0)
    return {"loss": rows.mean().reshape(1), "rows": rows, "dlogits": grad}


_EXACT = {"mlp": _exact_mlp, "layer": _exact_layer, "recurrent": _exact_recurrent, "conv": _exact_conv, "update": _exact_update, "loss": _exact_loss}


# ---------------------------------------------------------------- what the measuring program calls
_FAMILIES = {"mlp": (_prepare_mlp, _run_mlp, _work_mlp), "layer": (_prepare_layer, _run_layer, _work_layer),
             "recurrent": (_prepare_recurrent, _run_recurrent, _work_recurrent), "conv": (_prepare_conv, _run_conv, _work_conv),
             "update": (_prepare_update, _run_update, _work_update), "loss": (_prepare_loss, _run_loss, _work_loss)}


def prepare(case, seed):
    state = _FAMILIES[case["family"]][0](case, _gen(seed))
    state["family"] = case["family"]
    return state


def run(state):
    return _FAMILIES[state["family"]][1](state)


def exact(case, seed):
    return _EXACT[case["family"]](_FAMILIES[case["family"]][0](case, _gen(seed)))


def work(case):
    return _FAMILIES[case["family"]][2](case)


def tolerance(case):
    """About four times what the same pass differs by when its sums run in another order (split reductions against unsplit
    ones) or against products formed in FP64, over the listed cases and drawn ones.  An FP16 result moves by a whole step
    (2^-10 of its value at most) where the two sums fall on different sides of a rounding boundary, and moves what is computed from it."""
    family = case["family"]
    if family == "layer":                                                   # seen: 1.4e-5; one step
        return {"rel": 6e-5, "max": 4e-3}
    if family == "mlp":                                                     # seen: 1.2e-4, through two layers and the loss
        return {"rel": 5e-4, "max": 4e-3}
    if family == "recurrent":                                               # seen: 4e-4 and 1.2e-2 after 20 steps
        return {"rel": 1.6e-3, "max": 5e-2}
    if family == "conv":                                                    # seen: 6e-5 and 2.6e-3, through the statistics
        return {"rel": 3e-4, "max": 1e-2}
    if family == "loss":                                                    # seen: 6e-7 (the labels' elements outweigh the rest); one step
        return {"rel": 2.5e-6, "max": 4e-3}
    if case["clip"]:                                                        # the FP32 clip factor may round the other way: 6e-8; one FP16 step in the copy
        return {"rel": 1e-6, "max": 4e-3}
    return "exact"
