"""The passes that this library is timed and checked on.

A case is one whole forward + reverse pass through ``Runner.run``: its inputs
already in HBM, a runner that the program keeps from pass to pass, gradient
buffers that it reuses.  The listed cases are the repository's own workloads
(the two longest cut in length, every width and batch kept) and, beside them,
ragged sizes, small batches and the tests' options; ``draw`` gives more of the
same ranges.

The checkpoint interval is part of a case: it is the one that
``Runner.calibrate`` measures for the workload, given here so that a pass does
the same work on every box.
"""
from __future__ import annotations

import math

import torch

import paper_1806_01117_amd as amb

# Bounds on the relative error of each output: about four times the largest
# seen when the listed cases (six seeds each) and 120 drawn ones were compared
# with their 64-bit evaluation (fp32 cells 2.3e-6, bf16 cells 3.5e-3, the
# residual MLP 6.7e-5 and, bf16, 3.7e-3, the fp32 MLP 6.1e-3).  A bf16 pass rounds the stored
# state after every step, and an entry that falls on the other side of a
# rounding boundary moves on through the steps that follow.  A ReLU whose
# pre-activation lies within rounding of zero may be decided either way, which
# changes one batch row's gradients by some percent without a residual path
# and by some tenths of a percent with one.
CELL = {"f32": {"rel": 1e-5}, "bf16": {"rel": 1.4e-2}}
RESMLP = {"f32": {"rel": 3e-4}, "bf16": {"rel": 1.5e-2}}
MLP = {"rel": 2.5e-2}


def _case(name, cell, dtype, loss, batch, input, hidden, n, s, slow, interval, **kw):
    c = {"name": name, "cell": cell, "dtype": dtype, "loss": loss, "batch": batch, "input": input,
         "hidden": hidden, "n": n, "fast_slots": s, "slow_slots": slow, "interval": interval,
         "forget_bias": 0.0, "online": False, "widths": ""}
    c.update(kw)
    return c


def listed():
    return [
        # the 128-step tanh RNN on 4 slots and no host tier: the smallest call,
        # a chain of some 650 tiny dependent steps (a loss over every step: that
        # of the last state alone has a dL/dh_0 below the range of fp32)
        _case("rnn_h64_t128", "rnn", "f32", "mean_sq_all", 4, 32, 64, 128, 4, 0, 0),
        # a small LSTM with ragged rows and columns whose length is not known
        # in advance (online checkpointing), over a bounded host tier
        _case("lstm_h80_online", "lstm", "f32", "mean_sq_all", 5, 208, 80, 61, 4, 12, 2, forget_bias=1.0,
              online=True),
        # the 512-LSTM over 1000 steps, 10 slots and a host tier
        _case("lstm_h512_t1000", "lstm", "f32", "mean_sq_all", 64, 256, 512, 1000, 10, 1000, 1, forget_bias=1.0),
        # an fp32 LSTM of ordinary width whose weights are too many for the
        # registers of the chip, small batch: one launch per step
        _case("lstm_h1024_b32", "lstm", "f32", "mean_sq_all", 32, 256, 1024, 48, 6, 48, 2, forget_bias=1.0),
        # a bf16 LSTM on a small batch, ragged rows, plain Revolve
        _case("lstm_h1024_bf16_b20", "lstm", "bf16", "half_sq_last", 20, 512, 1024, 48, 6, 0, 0, forget_bias=1.0),
        # a bf16 tanh RNN, wide batch with ragged rows
        _case("rnn_h1536_bf16_b100", "rnn", "bf16", "mean_sq_all", 100, 64, 1536, 40, 4, 40, 2),
        # the 2048-wide bf16 LSTM (10000 steps cut to 192)
        _case("lstm_h2048_bf16", "lstm", "bf16", "mean_sq_all", 128, 1024, 2048, 192, 16, 192, 3),
        # the bf16 residual MLP of width 4096, depth as the sequence (2000
        # layers cut to 24)
        _case("resmlp_w4096_bf16", "resmlp", "bf16", "half_sq_last", 256, 0, 4096, 24, 4, 24, 2),
        # an fp32 residual MLP, ragged batch and width
        _case("resmlp_w1040", "resmlp", "f32", "half_sq_last", 70, 0, 1040, 24, 4, 24, 2),
        # the MLP whose layers change width (2000 layers cut to 64: ReLU layers
        # without a residual path are chaotic over hundreds)
        _case("mlp_widths", "mlp", "f32", "half_sq_last", 256, 0, 1024, 64, 8, 64, 5,
              widths="1024,512,256,512"),
        # a large-batch fp32 LSTM with rows and inputs ragged against the tiles
        _case("lstm_h1024_b300", "lstm", "f32", "mean_sq_all", 300, 96, 1024, 24, 4, 24, 2),
        # the 4096-wide fp32 LSTM (20000 steps cut to 48): the largest
        _case("lstm_h4096", "lstm", "f32", "mean_sq_all", 512, 1024, 4096, 48, 8, 48, 6),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, step * round(v / step))))


def draw(rng):
    kind = rng.choice(("rnn", "lstm_small", "lstm_small", "lstm_bf16", "lstm_bf16", "rnn_bf16", "resmlp",
                       "resmlp_bf16", "mlp", "lstm_large", "lstm_large"))
    loss = rng.choice(("half_sq_last", "mean_sq_all"))
    if kind == "rnn":
        c = _case("", "rnn", "f32", "mean_sq_all", _log(rng, 1, 64), _log(rng, 16, 128, 16), _log(rng, 16, 256, 16),
                  _log(rng, 16, 160), rng.randint(2, 8), 0, 0)
    elif kind == "lstm_small":  # both sides of the line at which the weights fit the registers
        c = _case("", "lstm", "f32", loss, _log(rng, 1, 64), _log(rng, 16, 512, 16), _log(rng, 32, 1024, 16),
                  _log(rng, 16, 100), rng.randint(3, 10), 0, 0, forget_bias=1.0, online=rng.random() < 0.25)
    elif kind == "lstm_bf16":  # both sides of the wide batch
        c = _case("", "lstm", "bf16", "mean_sq_all", _log(rng, 8, 256), _log(rng, 32, 1024, 32),
                  _log(rng, 128, 2048, 32), _log(rng, 12, 96), rng.randint(3, 12), 0, 0, forget_bias=1.0)
    elif kind == "rnn_bf16":
        c = _case("", "rnn", "bf16", "mean_sq_all", _log(rng, 8, 256), _log(rng, 32, 512, 32),
                  _log(rng, 128, 2048, 32), _log(rng, 12, 64), rng.randint(3, 8), 0, 0)
    elif kind == "resmlp":
        c = _case("", "resmlp", "f32", loss, _log(rng, 8, 256), 0, _log(rng, 128, 2048, 16), _log(rng, 8, 24),
                  rng.randint(2, 5), 0, 0)
    elif kind == "resmlp_bf16":
        c = _case("", "resmlp", "bf16", loss, _log(rng, 16, 256), 0, _log(rng, 256, 4096, 32), _log(rng, 8, 20),
                  rng.randint(2, 5), 0, 0)
    elif kind == "mlp":
        # quarters of one width: the state sizes then have a large common
        # divisor, which keeps the sized schedule's tables within their limit
        top = _log(rng, 128, 1280, 64)
        ws = [top] + [rng.randint(1, 4) * top // 4 for _ in range(rng.randint(1, 3))]
        c = _case("", "mlp", "f32", "half_sq_last", _log(rng, 16, 256, 4), 0, top, _log(rng, 16, 64),
                  rng.randint(3, 10), 0, 0, widths=",".join(map(str, ws)))
    else:
        c = _case("", "lstm", "f32", loss, _log(rng, 200, 512),
                  _log(rng, 16, 1024, 16), _log(rng, 1024, 3072, 16), _log(rng, 8, 40), rng.randint(3, 8), 0, 0)
    if rng.random() < 0.7:  # a host tier as long as the sequence
        c["slow_slots"], c["interval"] = c["n"], rng.randint(1, 6)
    del c["name"]
    return c


def _widths(case):
    """w_0 .. w_n of the MLP whose layers change width."""
    pat = [int(v) for v in case["widths"].split(",")]
    return [pat[t % len(pat)] for t in range(case["n"] + 1)]


def _gates(case):
    return 4 if case["cell"] == "lstm" else 1


def _inputs(case, seed):
    """x, W, b, h0, c0 in HBM: standard normal step inputs, uniform
    +-1/sqrt(H) recurrent weights, He-scaled MLP weights (the residual MLP's
    scaled down with its depth, so that activations stay of order one), zero
    biases but the forget gate's."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dev = torch.device("cuda")
    op = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    B, D, H, n = case["batch"], case["input"], case["hidden"], case["n"]

    def normal(shape, std):
        return torch.empty(shape, dtype=torch.float32, device=dev).normal_(0.0, std, generator=g)

    if case["cell"] == "mlp":
        ws = _widths(case)
        W = torch.cat([normal((ws[l + 1] * ws[l],), math.sqrt(2.0 / ws[l])) for l in range(n)])
        return None, W, torch.zeros(sum(ws[1:]), device=dev), normal((B, ws[0]), 1.0), None
    if case["cell"] == "resmlp":
        W = torch.empty((n, H, H), dtype=op, device=dev)
        for l in range(n):
            W[l] = normal((H, H), 1.28 / math.sqrt(H * n)).to(op)
        return None, W, torch.zeros((n, H), device=dev), normal((B, H), 1.0).to(op), None
    G = _gates(case)
    k = 1.0 / math.sqrt(H)
    W = torch.empty((G * H, D + H), dtype=torch.float32, device=dev).uniform_(-k, k, generator=g).to(op)
    x = normal((n, B, D), 1.0).to(op)
    b = torch.zeros(G * H, device=dev)
    if case["cell"] == "lstm":
        b[H:2 * H] = case["forget_bias"]
    h0 = normal((B, H), math.sqrt(0.1)).to(op)
    c0 = normal((B, H), math.sqrt(0.1)) if case["cell"] == "lstm" else None
    return x, W, b, h0, c0


def prepare(case, seed):
    x, W, b, h0, c0 = _inputs(case, seed)
    spec = amb.ProblemSpec(cell=case["cell"], dtype=case["dtype"], loss=case["loss"], batch=case["batch"],
                           input=case["input"], hidden=case["hidden"], n_steps=case["n"],
                           fast_slots=case["fast_slots"], slow_slots=case["slow_slots"],
                           interval_min=case["interval"],
                           widths=tuple(_widths(case)) if case["cell"] == "mlp" else None)
    r = amb.Runner(spec)
    if case["online"]:
        r.set("online", 1)
    r.set("reserve", 1)  # the pinned host tier, before the first pass
    out = {"dW": torch.empty(W.shape, dtype=torch.float32, device="cuda"), "db": torch.empty_like(b),
           "dh0": torch.empty(h0.shape, dtype=torch.float32, device="cuda"),
           "dc0": torch.empty_like(c0) if c0 is not None else None}
    return {"runner": r, "inputs": (x, W, b, h0, c0), "out": out}


def run(state):
    res = state["runner"].run(*state["inputs"], out=state["out"])
    outs = {"loss": res["loss"], "dW": res["dW"], "db": res["db"], "dh0": res["dh0"]}
    if res["dc0"] is not None:
        outs["dc0"] = res["dc0"]
    return outs


def work(case):
    """Conventional backpropagation's products (forward, state adjoint, weight
    gradient), without any recomputation; every input read and every gradient
    written once."""
    B, D, H, n = case["batch"], case["input"], case["hidden"], case["n"]
    e = 4 if case["dtype"] == "f32" else 2
    if case["cell"] == "mlp":
        ws = _widths(case)
        m = sum(ws[l + 1] * ws[l] for l in range(n))
        return {"bytes": 8 * m + 8 * sum(ws[1:]) + 8 * B * ws[0], "flops": 6 * B * m}
    if case["cell"] == "resmlp":
        return {"bytes": n * (H * H * (e + 4) + 8 * H) + B * H * (e + 4), "flops": 6 * n * B * H * H}
    GH = _gates(case) * H
    c = 8 * B * H if case["cell"] == "lstm" else 0
    return {"bytes": n * B * D * e + GH * (D + H) * (e + 4) + 8 * GH + B * H * (e + 4) + c,
            "flops": 2 * n * B * GH * (2 * (D + H) + H)}


def tolerance(case):
    if case["cell"] == "mlp":
        return MLP
    return (RESMLP if case["cell"] == "resmlp" else CELL)[case["dtype"]]


def exact(case, seed):
    """The same pass by conventional backpropagation through time in 64 bits,
    every state kept; a bf16 workload's stored state is rounded to bf16 after
    every step, as its definition says."""
    x, W, b, h0, c0 = _inputs(case, seed)
    n, B, D, H, loss = case["n"], case["batch"], case["input"], case["hidden"], case["loss"]
    f64 = torch.float64
    rnd = (lambda h: h.to(torch.bfloat16).to(f64)) if case["dtype"] == "bf16" else (lambda h: h)

    def term(t, h):
        if loss == "mean_sq_all":
            return float((h * h).mean())
        if t < n:
            return 0.0
        return float(0.5 * (h * h).sum()) if loss == "half_sq_last" else float(h.mean())

    def seed_of(t, h):  # dL/dh_t
        if loss == "mean_sq_all":
            return 2.0 * h / h.numel()
        if t < n:
            return torch.zeros_like(h)
        return h.clone() if loss == "half_sq_last" else torch.full_like(h, 1.0 / h.numel())

    if case["cell"] in ("mlp", "resmlp"):
        res = case["cell"] == "resmlp"
        ws = [H] * (n + 1) if res else _widths(case)
        offs, boffs = [0], [0]
        for l in range(n):
            offs.append(offs[-1] + ws[l + 1] * ws[l])
            boffs.append(boffs[-1] + ws[l + 1])
        flat, bflat = W.reshape(-1), b.reshape(-1)

        def layer(l):
            return flat[offs[l]:offs[l + 1]].view(ws[l + 1], ws[l]).to(f64), bflat[boffs[l]:boffs[l + 1]].to(f64)

        ys, masks = [h0.to(f64)], []
        for l in range(n):
            Wl, bl = layer(l)
            z = ys[l] @ Wl.t() + bl
            masks.append(z > 0)
            ys.append(rnd(ys[l] + z.clamp(min=0.0) if res else z.clamp(min=0.0)))
        total = sum(term(t, ys[t]) for t in range(1, n + 1))
        dW = torch.empty(flat.numel(), dtype=torch.float32, device=W.device)
        db = torch.empty(bflat.numel(), dtype=torch.float32, device=W.device)
        bar = torch.zeros_like(ys[n])
        for l in range(n - 1, -1, -1):
            bar = bar + seed_of(l + 1, ys[l + 1])
            zb = bar * masks[l]
            dW[offs[l]:offs[l + 1]] = (zb.t() @ ys[l]).reshape(-1)
            db[boffs[l]:boffs[l + 1]] = zb.sum(dim=0)
            bar = zb @ layer(l)[0] + (bar if res else 0.0)
        return {"loss": total, "dW": dW.view(W.shape), "db": db.view(b.shape), "dh0": bar}

    W64, b64 = W.to(f64), b.to(f64)
    lstm = case["cell"] == "lstm"
    hs, cs = [h0.to(f64)], [c0.to(f64) if lstm else None]

    def gates(t):
        z = torch.cat([x[t].to(f64), hs[t]], dim=1) @ W64.t() + b64
        if not lstm:
            return (torch.tanh(z),)
        i, f, g, o = z.split(H, dim=1)
        return torch.sigmoid(i), torch.sigmoid(f), torch.tanh(g), torch.sigmoid(o)

    for t in range(n):
        a = gates(t)
        if lstm:
            cs.append(a[1] * cs[t] + a[0] * a[2])
            hs.append(rnd(a[3] * torch.tanh(cs[t + 1])))
        else:
            hs.append(rnd(a[0]))
    total = sum(term(t, hs[t]) for t in range(1, n + 1))
    dW, db = torch.zeros_like(W64), torch.zeros_like(b64)
    hb = torch.zeros_like(hs[n])
    cb = torch.zeros_like(hs[n])
    for t in range(n - 1, -1, -1):
        a = gates(t)
        hb = hb + seed_of(t + 1, hs[t + 1])
        if lstm:
            i, f, g, o = a
            tc = torch.tanh(cs[t + 1])
            cb = cb + hb * o * (1.0 - tc * tc)
            zb = torch.cat([cb * g * i * (1.0 - i), cb * cs[t] * f * (1.0 - f), cb * i * (1.0 - g * g),
                            hb * tc * o * (1.0 - o)], dim=1)
            cb = cb * f
        else:
            zb = hb * (1.0 - a[0] * a[0])
        dW += zb.t() @ torch.cat([x[t].to(f64), hs[t]], dim=1)
        db += zb.sum(dim=0)
        hb = zb @ W64[:, D:]
    outs = {"loss": total, "dW": dW, "db": db, "dh0": hb}
    if lstm:
        outs["dc0"] = cb
    return outs
