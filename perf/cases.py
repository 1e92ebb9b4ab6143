"""Performance cases of the streaming 1-D CNN library.

Each case is one call pattern of a user's program, through the public entry
points of ``paper_2108_12430_amd.gwstream`` (and ``autograd``):

  listed()            the cases that are always timed
  draw(rng)           one more case of the same ranges
  prepare(case, seed) what the program holds before the call (on the GPU)
  run(state)          one pass
  work(case)          the bytes and operations the pass cannot do without
  exact(case, seed)   the pass's outputs in 64 bits, written with plain torch

Paths (case["path"]):
  streams   n DeepClean streams send their new witness samples; the snapshot
            rings are updated and every window is cleaned (deepclean_update_forward)
  step      the serving mix: DeepClean streams as above, and BBHnet streams on
            a second HIP stream (snapshot_update, bbhnet_forward)
  windows   n dense witness windows (offline cleaning, or one window on its own)
  cached    DeepClean streams over activation caches with an aggregation delay
  bbh       n dense two-detector windows through BBHnet
  train     one DeepClean retraining step
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2108_12430_amd import autograd
from paper_2108_12430_amd import gwstream as gs

DEV = "cuda:0"
C_WIT = 21            # witness channels
PRECISION = {"fp32": gs.FP32, "bf16": gs.BF16, "fp16": gs.FP16}

# (type, C_in, C_out, k, stride, pad, out_pad, BN + tanh)
LAYERS = ([("conv", a, b, 7, 2, 3, 0, True) for a, b in ((21, 8), (8, 16), (16, 32), (32, 64))]
          + [("convT", a, b, 7, 2, 3, 1, True) for a, b in ((64, 32), (32, 16), (16, 8), (8, 8))]
          + [("conv", 8, 1, 7, 1, 3, 0, False)])
STAGES = [(2, 32), (32, 64), (64, 128)]


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # one online detector: a 1/16-s request of one stream, the smallest
        # call of the serving loop, where latency is everything
        {"name": "stream_1_bf16", "path": "streams", "n": 1, "W": 32768, "fs": 4096, "precision": "bf16",
         "strides": "sixteenth", "causal": False, "noise": True},
        # the same service at a site that samples at 4000 Hz and asks for
        # r requests per second, r not a divisor: strides of any size and
        # alignment (4 .. 1333 samples), 8-s windows of 32000 samples
        {"name": "streams_24_ragged_bf16", "path": "streams", "n": 24, "W": 32000, "fs": 4000, "precision": "bf16",
         "strides": "ragged", "causal": False, "noise": True},
        # the headline serving step: 179 DeepClean and 77 BBHnet streams
        {"name": "step_179_77_bf16", "path": "step", "n": 179, "W": 32768, "fs": 4096, "precision": "bf16",
         "strides": "mix", "causal": False, "noise": False, "n_bbh": 77, "W_bbh": 2048},
        # the same streams when only the newest outputs are computed
        {"name": "streams_179_causal_bf16", "path": "streams", "n": 179, "W": 32768, "fs": 4096, "precision": "bf16",
         "strides": "mix", "causal": True, "noise": False},
        # half precision, the format of the online study
        {"name": "streams_48_fp16", "path": "streams", "n": 48, "W": 32768, "fs": 4096, "precision": "fp16",
         "strides": "mix", "causal": False, "noise": True},
        # full precision: one 1-s window, and a small group of online streams
        {"name": "window_1_fp32", "path": "windows", "n": 1, "W": 4096, "precision": "fp32"},
        {"name": "streams_16_fp32", "path": "streams", "n": 16, "W": 32768, "fs": 4096, "precision": "fp32",
         "strides": "mix", "causal": False, "noise": True},
        # 0.75 s of aggregation latency over activation caches
        {"name": "cached_179_bf16", "path": "cached", "n": 179, "W": 32768, "fs": 4096, "precision": "bf16",
         "strides": "mix", "noise": False},
        # offline scoring of two-detector windows, in both precisions
        {"name": "bbh_1024_bf16", "path": "bbh", "n": 1024, "W": 2048, "precision": "bf16"},
        {"name": "bbh_64_fp32", "path": "bbh", "n": 64, "W": 2048, "precision": "fp32"},
        # retraining on recent data: batches of 8-s windows
        {"name": "train_32_fp32", "path": "train", "n": 32, "W": 32768, "fs": 4096, "precision": "fp32"},
        {"name": "train_32_bf16", "path": "train", "n": 32, "W": 32768, "fs": 4096, "precision": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _window(rng, fs, lo_s, hi_s):
    """A window of lo_s .. hi_s seconds, a multiple of the network's stride of 16."""
    return max(16, 16 * int(round(fs * math.exp(rng.uniform(math.log(lo_s), math.log(hi_s))) / 16)))


def draw(rng):
    path = rng.choice(["streams", "streams", "step", "windows", "cached", "bbh", "train"])
    fs = rng.choice([4096, 4096, 4000])
    case = {"path": path, "fs": fs, "precision": "bf16"}
    if path == "streams":
        case["precision"] = rng.choice(["bf16", "bf16", "fp16", "fp32"])
        case["n"] = _log_int(rng, 1, {"bf16": 179, "fp16": 96, "fp32": 24}[case["precision"]])
        case["W"] = _window(rng, fs, 1, 8)
        case["strides"] = rng.choice(["sixteenth", "mix", "ragged"])
        case["causal"] = rng.random() < 0.25
        case["noise"] = not case["causal"] and rng.random() < 0.5
    elif path == "step":
        case.update(n=_log_int(rng, 4, 179), W=_window(rng, fs, 2, 8), strides=rng.choice(["mix", "ragged"]),
                    causal=False, noise=False, n_bbh=_log_int(rng, 4, 77), W_bbh=rng.choice([1024, 2048, 4096]))
    elif path == "windows":
        case["precision"] = rng.choice(["fp32", "fp32", "bf16"])
        case["n"] = _log_int(rng, 1, 16)
        case["W"] = _window(rng, fs, 0.25, 8)
    elif path == "cached":
        case.update(n=_log_int(rng, 2, 179), W=_window(rng, fs, 2, 8), strides=rng.choice(["sixteenth", "mix"]),
                    noise=rng.random() < 0.5)
    elif path == "bbh":
        case["precision"] = rng.choice(["bf16", "fp32"])
        case["n"] = _log_int(rng, 1, 1024 if case["precision"] == "bf16" else 96)
        case["W"] = 8 * _log_int(rng, 64, 256)
    else:
        case["precision"] = rng.choice(["fp32", "bf16"])
        case["n"] = _log_int(rng, 2, 32)
        case["W"] = _window(rng, fs, 1, 8)
    return case


def _strides(case, n=None, fs=None, W=None):
    """New samples per request of every stream (a function of the case)."""
    n = case["n"] if n is None else n
    fs = case["fs"] if fs is None else fs
    W = case["W"] if W is None else W
    if case["strides"] == "sixteenth":
        s = np.full(n, fs // 16)
    elif case["strides"] == "mix":
        s = (np.random.default_rng(6).choice([1 / 16, 1 / 8, 1 / 4], n) * fs).astype(np.int64)
    else:  # floor(fs / r), request rates r from 3 to 1000 Hz
        s = np.floor(fs / np.exp(np.random.default_rng(6).uniform(math.log(3), math.log(1000), n)))
    if case["path"] == "cached":
        s = s // 16 * 16  # the cached path advances in units of the network's stride
    return np.clip(s, 1, W).astype(np.int64)


# ---------------------------------------------------------------------------
# Inputs and parameters (made from the seed alone)
# ---------------------------------------------------------------------------

def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + salt)


def _witness(n, W, fs, seed):
    """Witness windows [n][21][W] and strain [n][W]: unit noise, with 60 and
    120 Hz lines on the first four channels, which leak into the strain."""
    g = _gen(seed, 1)
    x = torch.randn(n, C_WIT, W, device=DEV, generator=g)
    strain = torch.randn(n, W, device=DEV, generator=g)
    t = torch.arange(W, device=DEV, dtype=torch.float32) / fs
    for c in range(4):
        for f in (60.0, 120.0):
            amp = 0.5 + 1.5 * torch.rand(n, 1, device=DEV, generator=g)
            ph = 2 * math.pi * torch.rand(n, 1, device=DEV, generator=g)
            line = amp * torch.sin(2 * math.pi * f * t + ph)
            x[:, c] += line
            strain += 0.3 * line
    return x, strain


def _bbh_windows(n, W, seed):
    """Whitened two-detector windows [n][2][W]; every other one holds a chirp."""
    g = _gen(seed, 2)
    x = torch.randn(n, 2, W, device=DEV, generator=g)
    t = torch.arange(W, device=DEV, dtype=torch.float32) / 2048.0
    tc = (0.5 + 0.45 * torch.rand(n, 1, device=DEV, generator=g)) * W / 2048.0
    tau = (tc - t).clamp_min(0.002)
    h = torch.sin(-2 * math.pi * 60.0 * tau.pow(0.625)) * tau.pow(-0.25) * (t < tc)
    h *= (6 + 14 * torch.rand(n, 1, device=DEV, generator=g)) / h.square().sum(1, keepdim=True).sqrt().clamp_min(1e-6)
    h[1::2] = 0
    return x + h[:, None] / math.sqrt(2.0)


def _uniform(shape, fan_in, g):
    return (2 * torch.rand(shape, device=DEV, generator=g) - 1) / math.sqrt(fan_in)


def _dc_params(seed):
    """Per layer: weight, bias, then gamma, beta, running mean and variance."""
    g, parts = _gen(seed, 3), []
    for typ, ci, co, k, _s, _p, _op, bn in LAYERS:
        fan = (ci if typ == "conv" else co) * k
        parts += [_uniform((co, ci, k) if typ == "conv" else (ci, co, k), fan, g), _uniform((co,), fan, g)]
        if bn:
            u = torch.rand(2, co, device=DEV, generator=g)
            v = torch.randn(2, co, device=DEV, generator=g)
            parts += [0.5 + u[0], 0.1 * v[0], 0.1 * v[1], 0.5 + u[1]]
    return parts


def _bb_params(seed):
    """Per stage: conv_a, conv_b and 1x1 shortcut (weight, bias); then the head."""
    g, parts = _gen(seed, 4), []
    for ci, co in STAGES:
        for cin, k in ((ci, 7), (co, 7), (ci, 1)):
            parts += [_uniform((co, cin, k), cin * k, g), _uniform((co,), cin * k, g)]
    return parts + [_uniform((1, 128), 128, g), _uniform((1,), 128, g)]


def _flat(parts):
    return torch.cat([p.reshape(-1) for p in parts])


def _samples(new, strides):
    """Each stream's newest samples packed back to back: blocks [C][s_i] and
    their offsets, from new [n][C][>= max s]."""
    blocks = [new[i, :, new.shape[2] - int(s):].reshape(-1) for i, s in enumerate(strides)]
    off = np.concatenate([[0], np.cumsum([b.numel() for b in blocks])[:-1]]).astype(np.int64)
    return torch.cat(blocks), off


def _tails(strain, strides, delay=0):
    W = strain.shape[1]
    return torch.cat([strain[i, W - int(s) - delay: W - delay] for i, s in enumerate(strides)])


def _stream_inputs(case, seed):
    """The windows held before the request, the windows after it, the strain
    of the latter, and the strides."""
    strides = _strides(case)
    smax = int(strides.max())
    x, strain = _witness(case["n"], case["W"] + smax, case["fs"], seed)
    W = case["W"]
    old = torch.stack([x[i, :, smax - int(s): smax - int(s) + W] for i, s in enumerate(strides)])
    return old, x[:, :, smax:], strain[:, smax:], strides


def _ring_bytes(c, w):
    up = lambda b: (b + 255) // 256 * 256
    return up(c * w * 4) + up(c * w * 2)


def _open(windows):
    """A pool whose n slots hold the given windows."""
    n, c, w = windows.shape
    pool = gs.Pool(n * _ring_bytes(c, w) + (8 << 20), max_slots=n, max_items=n)
    slots = [pool.open(c, w) for _ in range(n)]
    for i, s in enumerate(slots):
        pool.load(s, windows[i].contiguous(), w)
    return pool, slots


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------

def _prepare_streams(case, seed):
    old, new, strain, strides = _stream_inputs(case, seed)
    n, W, prec = case["n"], case["W"], PRECISION[case["precision"]]
    flags = gs.CAUSAL if case["causal"] else 0
    model = gs.DeepClean(_flat(_dc_params(seed)), LAYERS)
    pool, slots = _open(old)
    samples, offsets = _samples(new, strides)
    ws = torch.empty(max(256, model.workspace_bytes(n, W, prec, flags)), dtype=torch.uint8, device=DEV)
    return {"path": "streams", "model": model, "pool": pool,
            "call": dict(pool=pool, slots=slots, strides=strides, samples=samples, offsets=offsets, W=W,
                         strain=_tails(strain, strides), clean=torch.empty(int(strides.sum()), device=DEV),
                         noise=torch.empty(n, W, device=DEV) if case["noise"] else None, precision=prec,
                         flags=flags, ws=ws)}


_serving_streams = []


def _prepare_step(case, seed):
    state = _prepare_streams(case, seed)
    state["path"] = "step"
    n, W = case["n_bbh"], case["W_bbh"]
    strides = _strides({**case, "strides": "mix"}, n, W, W)  # 1-s BBHnet windows at W samples a second
    x = _bbh_windows(n, 2 * W, seed)
    old = torch.stack([x[i, :, W - int(s): 2 * W - int(s)] for i, s in enumerate(strides)])
    bbh = gs.BBHnet(_flat(_bb_params(seed)), STAGES)
    pool, slots = _open(old)
    samples, offsets = _samples(x, strides)
    ws = torch.empty(max(256, bbh.workspace_bytes(n, W, gs.BF16)), dtype=torch.uint8, device=DEV)
    if not _serving_streams:  # a server keeps one HIP stream per model group
        _serving_streams.extend(torch.cuda.Stream() for _ in range(2))
    state.update(bbh=bbh, bbh_pool=pool,
                 bbh_update=dict(slots=slots, strides=strides, samples=samples, offsets=offsets),
                 bbh_call=dict(pool=pool, slots=slots, W=W, logits=torch.empty(n, device=DEV), precision=gs.BF16,
                               ws=ws),
                 hip=list(_serving_streams))
    torch.cuda.synchronize()  # the groups' streams start on finished inputs
    return state


def _prepare_windows(case, seed):
    n, W, prec = case["n"], case["W"], PRECISION[case["precision"]]
    x, _ = _witness(n, W, 4096, seed)
    model = gs.DeepClean(_flat(_dc_params(seed)), LAYERS)
    ws = torch.empty(max(256, model.workspace_bytes(n, W, prec)), dtype=torch.uint8, device=DEV)
    return {"path": "windows", "model": model,
            "call": dict(x=x, noise=torch.empty(n, W, device=DEV), precision=prec, ws=ws)}


def _delay(case):
    return min(3 * case["fs"] // 4, case["W"] // 2)


def _prepare_cached(case, seed):
    old, new, strain, strides = _stream_inputs(case, seed)
    n, W = case["n"], case["W"]
    model = gs.DeepClean(_flat(_dc_params(seed)), LAYERS)
    pool, slots = _open(old)
    caches = [model.new_cache(W) for _ in slots]
    for s, c in zip(slots, caches):
        pool.attach_cache(s, c)
    samples, offsets = _samples(new, strides)
    delay = _delay(case)
    call = dict(pool=pool, slots=slots, W=W, strides=strides, strain=_tails(strain, strides, delay),
                clean=torch.empty(int(strides.sum()), device=DEV), delays=np.full(n, delay),
                noise=torch.empty(n, W, device=DEV) if case["noise"] else None)
    model.forward_cached(**call)  # the streams have been served before: their caches are current
    return {"path": "cached", "model": model, "pool": pool, "caches": caches,
            "update": dict(slots=slots, strides=strides, samples=samples, offsets=offsets), "call": call}


def _prepare_bbh(case, seed):
    n, W, prec = case["n"], case["W"], PRECISION[case["precision"]]
    model = gs.BBHnet(_flat(_bb_params(seed)), STAGES)
    ws = torch.empty(max(256, model.workspace_bytes(n, W, prec)), dtype=torch.uint8, device=DEV)
    return {"path": "bbh", "model": model,
            "call": dict(x=_bbh_windows(n, W, seed), logits=torch.empty(n, device=DEV), precision=prec, ws=ws)}


def _prepare_train(case, seed):
    n, W, prec = case["n"], case["W"], PRECISION[case["precision"]]
    x, strain = _witness(n, W, case["fs"], seed)
    params = _flat(_dc_params(seed))
    state = {"path": "train", "x": x, "strain": strain, "fs": float(case["fs"]), "precision": prec, "params": params}
    if prec == gs.FP32:  # through torch.autograd
        params.requires_grad_(True)
        state["model"] = gs.DeepClean(params.detach(), LAYERS)
    else:
        flags = gs.TRAIN | gs.RECOMPUTE
        model = gs.DeepClean(params, LAYERS)
        state.update(model=model, flags=flags, noise=torch.empty(n, W, device=DEV), grad=torch.empty_like(params),
                     ws=torch.empty(model.workspace_bytes(n, W, prec, flags), dtype=torch.uint8, device=DEV),
                     scratch=torch.empty(model.backward_scratch_bytes(n, W, flags), dtype=torch.uint8, device=DEV))
    return state


def prepare(case, seed):
    return {"streams": _prepare_streams, "step": _prepare_step, "windows": _prepare_windows,
            "cached": _prepare_cached, "bbh": _prepare_bbh, "train": _prepare_train}[case["path"]](case, seed)


def run(state):
    path = state["path"]
    if path == "streams":
        c = state["call"]
        state["model"].update_forward(**c)
        return {"clean": c["clean"]} if c["noise"] is None else {"clean": c["clean"], "noise": c["noise"]}
    if path == "step":
        c, b = state["call"], state["bbh_call"]
        s_dc, s_bb = state["hip"]
        state["model"].update_forward(**c, stream=s_dc)
        state["bbh_pool"].update(**state["bbh_update"], stream=s_bb)
        state["bbh"].forward(**b, stream=s_bb)
        return {"clean": c["clean"], "logits": b["logits"]}
    if path == "windows":
        state["model"].forward(**state["call"])
        return {"noise": state["call"]["noise"]}
    if path == "cached":
        c = state["call"]
        state["pool"].update(**state["update"])
        state["model"].forward_cached(**c)
        return {"clean": c["clean"]} if c["noise"] is None else {"clean": c["clean"], "noise": c["noise"]}
    if path == "bbh":
        return {"logits": state["model"].forward(**state["call"])}
    if state["precision"] == gs.FP32:
        params = state["params"]
        params.grad = None
        noise = autograd.DeepCleanFn.apply(params, state["x"], state["model"], True)
        loss = autograd.bandpass_mse_loss(state["strain"], noise, state["fs"])
        loss.backward()
        return {"noise": noise.detach(), "loss": loss.detach(), "grad": params.grad}
    m = state["model"]
    m.forward(x=state["x"], noise=state["noise"], flags=state["flags"], ws=state["ws"], precision=state["precision"])
    loss, dn = gs.bandpass_mse(state["strain"], state["noise"], state["fs"])
    m.backward(state["x"], dn, state["ws"], state["grad"], flags=state["flags"], scratch=state["scratch"],
               precision=state["precision"])
    return {"noise": state["noise"], "loss": loss, "grad": state["grad"]}


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------

def _dc_flops_per_sample():
    """Multiply-adds of the network times two, per window sample."""
    macs, f = 0.0, 1.0  # f: layer input positions per window sample
    for typ, ci, co, k, s, _p, _op, _bn in LAYERS:
        if typ == "conv":
            f /= s
            macs += f * ci * co * k
        else:
            macs += f * ci * co * k
            f *= s
    return 2.0 * macs


def _bbh_flops(W):
    macs = 128.0
    for ci, co in STAGES:
        W //= 2
        macs += W * co * (7 * ci + 7 * co + ci)
    return 2.0 * macs


_N_DC = sum(ci * co * k + co + (4 * co if bn else 0) for _t, ci, co, k, _s, _p, _o, bn in LAYERS)
_N_BB = sum(7 * ci * co + 7 * co * co + ci * co + 3 * co for ci, co in STAGES) + 129


def work(case):
    path, n, W = case["path"], case["n"], case["W"]
    esz = 4 if case["precision"] != "bf16" else 2  # the ring's FP32 samples, or its BF16 shadow
    if path in ("streams", "step", "cached"):
        s = _strides(case)
        new = C_WIT * float(s.sum()) * (4 + 4 + 2) + 8.0 * float(s.sum())  # update; strain in, clean out
        if path == "cached":  # what changed: the new samples and the receptive field on either side
            span = np.minimum(s + 2 * 93, W)
        elif case["causal"]:
            span = np.minimum(s + 93, W)
        else:
            span = np.full(n, W)
        b = new + C_WIT * float(span.sum()) * esz + 4.0 * _N_DC
        fl = _dc_flops_per_sample() * float(span.sum())
        if case["noise"]:
            b += 4.0 * n * W
        if path == "step":
            sb = _strides({**case, "strides": "mix"}, case["n_bbh"], case["W_bbh"], case["W_bbh"])
            b += 2 * float(sb.sum()) * (4 + 4 + 2) + case["n_bbh"] * (2.0 * case["W_bbh"] * 2 + 4) + 4.0 * _N_BB
            fl += case["n_bbh"] * _bbh_flops(case["W_bbh"])
        return {"bytes": b, "flops": fl}
    if path == "windows":
        return {"bytes": 4.0 * n * W * (C_WIT + 1) + 4.0 * _N_DC, "flops": _dc_flops_per_sample() * n * W}
    if path == "bbh":
        return {"bytes": 4.0 * n * (2 * W + 1) + 4.0 * _N_BB, "flops": n * _bbh_flops(W)}
    # forward, input gradients (all but the first layer's) and weight gradients
    first = 2.0 * LAYERS[0][1] * LAYERS[0][2] * 7 / 2
    return {"bytes": 4.0 * n * W * (C_WIT + 2) + 8.0 * _N_DC,
            "flops": n * W * (3 * _dc_flops_per_sample() - first)}


# ---------------------------------------------------------------------------
# exact: the same outputs in 64 bits
# ---------------------------------------------------------------------------

def _conv(x, w, b, stride, pad):
    xp = torch.nn.functional.pad(x, (pad, pad))
    L = (xp.shape[2] - w.shape[2]) // stride + 1
    y = sum(torch.matmul(w[:, :, j].contiguous(), xp[:, :, j: j + stride * (L - 1) + 1: stride].contiguous())
            for j in range(w.shape[2]))
    return y + b[:, None]


def _conv_t(x, w, b):
    """k7, stride 2, pad 3, output padding 1: y[2m + r] = sum over taps j = r + 3 - 2d of w[j] x[m + d]."""
    L = x.shape[2]
    xp = torch.nn.functional.pad(x, (2, 2))
    ph = []
    for r in (0, 1):
        y = 0
        for d in (-1, 0, 1, 2):
            j = r + 3 - 2 * d
            if 0 <= j < 7:
                y = y + torch.matmul(w[:, :, j].t().contiguous(), xp[:, :, 2 + d: 2 + d + L].contiguous())
        ph.append(y)
    return torch.stack(ph, 3).reshape(x.shape[0], w.shape[1], 2 * L) + b[:, None]


def _dc_exact(parts, x, train=False):
    a, it = x, iter(parts)
    for typ, _ci, _co, _k, s, p, _op, bn in LAYERS:
        w, b = next(it), next(it)
        a = _conv(a, w, b, s, p) if typ == "conv" else _conv_t(a, w, b)
        if bn:
            ga, be, mean, var = next(it), next(it), next(it), next(it)
            if train:
                mean, var = a.mean((0, 2)), a.var((0, 2), unbiased=False)
            a = torch.tanh((a - mean[:, None]) / torch.sqrt(var[:, None] + 1e-5) * ga[:, None] + be[:, None])
    return a[:, 0]


def _bbh_exact(parts, x):
    a, it = x, iter(parts)
    for _ in STAGES:
        wa, ba, wb, bb, ws, bs = (next(it) for _ in range(6))
        h = torch.relu(_conv(a, wa, ba, 2, 3))
        a = torch.relu(_conv(h, wb, bb, 1, 3) + _conv(a[:, :, ::2].contiguous(), ws, bs, 1, 0))
    w, b = next(it), next(it)
    return a.mean(2) @ w[0] + b[0]


def _in_parts(fn, x, size=16):
    return torch.cat([fn(x[i: i + size].double()) for i in range(0, x.shape[0], size)])


def exact(case, seed):
    path = case["path"]
    if path == "bbh":
        parts = [p.double() for p in _bb_params(seed)]
        return {"logits": _in_parts(lambda x: _bbh_exact(parts, x), _bbh_windows(case["n"], case["W"], seed), 64)}
    parts = [p.double() for p in _dc_params(seed)]
    if path == "windows":
        x, _ = _witness(case["n"], case["W"], 4096, seed)
        return {"noise": _in_parts(lambda v: _dc_exact(parts, v), x)}
    if path == "train":
        x, strain = _witness(case["n"], case["W"], case["fs"], seed)
        parts = [p.requires_grad_(True) for p in parts]
        noise = _dc_exact(parts, x.double(), train=True)
        r = torch.fft.rfft(strain.double() - noise)
        f = torch.arange(r.shape[1], device=DEV, dtype=torch.float64) * case["fs"] / case["W"]
        inside = ((f >= 55.0) & (f <= 65.0)).double()
        loss = torch.fft.irfft(r * inside, n=case["W"]).square().mean()
        grads = torch.autograd.grad(loss, parts, allow_unused=True)
        grad = _flat([torch.zeros_like(p) if g is None else g for p, g in zip(parts, grads)])
        out = loss.detach()
        return {"noise": noise.detach(), "loss": out if case["precision"] == "fp32" else out.reshape(1), "grad": grad}
    _, new, strain, strides = _stream_inputs(case, seed)
    noise = _in_parts(lambda v: _dc_exact(parts, v), new)
    delay = _delay(case) if path == "cached" else 0
    out = {"clean": _tails(strain.double(), strides, delay) - _tails(noise, strides, delay)}
    if case["noise"]:
        out["noise"] = noise
    if path == "step":
        W = case["W_bbh"]
        bb = [p.double() for p in _bb_params(seed)]
        x = _bbh_windows(case["n_bbh"], 2 * W, seed)[:, :, W:]
        out["logits"] = _in_parts(lambda v: _bbh_exact(bb, v.contiguous()), x, 64)
    return out
