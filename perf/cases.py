"""The workloads that the mixed-precision training step is measured on.

A case is one model of the four step classes of `paper_1805_10387_amd.steps` at one size, and one pass is one whole
training iteration of it: forward, loss with the scaled seed gradient, backward, the fused unscale / check / update, and
the loss-scale update.  Sizes are the five configurations of `mp_inputs.py`, their reduced versions, and what lies
between them; the batch is in device memory before the pass, as a training loop has it.

`launch` is how the program drives the step: "eager" calls `step()`, "graph" replays a HIP graph of it that was captured
when the model was built (what `bench.py` does).  `tuned` is the configuration `bench.py` times: overflow inspection in
the gradient producers, one flat update descriptor, and (Transformer) the weight gradients on a second stream.
"""
import math

import numpy as np
import torch

import mp_inputs as I
from paper_1805_10387_amd import steps as St


def _mlp(name, rows, d_in, d_hidden, d_out, opt="sgd", launch="eager", tuned=False):
    return dict(name=name, kind="mlp", rows=rows, d_in=d_in, d_hidden=d_hidden, d_out=d_out, opt=opt, launch=launch, tuned=tuned)


def _transformer(name, layers, d_model, d_ff, seq_len, n_seq, opt="adam", launch="eager", tuned=False):
    return dict(name=name, kind="transformer", layers=layers, d_model=d_model, d_ff=d_ff, seq_len=seq_len, n_seq=n_seq, opt=opt,
                launch=launch, tuned=tuned)


def _xent(name, tokens, d_model, vocab, opt="adam", launch="eager", tuned=False):
    return dict(name=name, kind="xent", tokens=tokens, d_model=d_model, vocab=vocab, opt=opt, launch=launch, tuned=tuned)


def _lstm(name, layers, hidden, d_in, batch, seq_len, opt="adam", launch="eager", tuned=False):
    return dict(name=name, kind="lstm", layers=layers, hidden=hidden, d_in=d_in, batch=batch, seq_len=seq_len, opt=opt, launch=launch,
                tuned=tuned)


def listed():
    return [
        # configuration 1: the smallest step there is (launches and latency), SGD, driven call by call
        _mlp("mlp_64x256x1024x256", 64, 256, 1024, 256),
        # a feature front end with widths that are no multiple of 8 (161 spectrogram bins in, 29 characters out)
        _mlp("mlp_frames_161_to_29", 1500, 161, 1024, 29, opt="adam"),
        # configuration 2: one Transformer-base layer, 4096 tokens, as a graph replay
        _transformer("layer_base_4096", 1, 512, 2048, 64, 64, launch="graph"),
        # configuration 2 reduced: ragged in every dimension, per-tensor update with its inspection pass, call by call
        _transformer("layer_192_ragged", 1, 192, 328, 40, 5),
        # two base layers on sentences whose length is no multiple of 8 (the unfused attention chain)
        _transformer("stack_base_seq53", 2, 512, 2048, 53, 61, launch="graph"),
        # configuration 3: the Transformer-big stack that bench.py times, in its launch configuration
        _transformer("stack_big_8192", 6, 1024, 4096, 128, 64, launch="graph", tuned=True),
        # configuration 4: 32K vocabulary projection and cross-entropy
        _xent("vocab_8192x32768", 8192, 1024, 32768),
        # configuration 4 reduced
        _xent("vocab_520x3000", 520, 256, 3000),
        # a vocabulary as a tokenizer leaves it: odd
        _xent("vocab_1021x12001", 1021, 512, 12001, launch="graph", tuned=True),
        # configuration 5: the four-layer LSTM
        _lstm("lstm_4x1024_b32_t50", 4, 1024, 1024, 32, 50, launch="graph"),
        # configuration 5 reduced, call by call
        _lstm("lstm_2x128_b8_t6", 2, 128, 96, 8, 6),
        # a batch of 64 on a smaller stack (step-by-step recurrence)
        _lstm("lstm_2x512_b64_t25", 2, 512, 320, 64, 25, launch="graph"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _log8(rng, lo, hi, odd=0.0):
    """A multiple of 8, or with probability `odd` any number."""
    n = _log(rng, lo, hi)
    return n if rng.random() < odd else max(8, (n + 4) // 8 * 8)


def draw(rng):
    kind = rng.choice(["mlp", "transformer", "transformer", "xent", "xent", "lstm", "lstm"])
    how = dict(opt="adam" if rng.random() < 0.8 else "sgd", launch=rng.choice(["eager", "graph"]), tuned=rng.random() < 0.5)
    if kind == "mlp":
        c = _mlp("", _log(rng, 16, 4096), _log8(rng, 64, 1024, 0.3), _log8(rng, 128, 4096), _log8(rng, 24, 1024, 0.3), **how)
    elif kind == "transformer":
        d = 64 * rng.randint(2, 16)
        seq = _log8(rng, 8, 128, 0.4)
        n_seq = max(1, min(8192 // seq, _log(rng, 4, 512)))
        c = _transformer("", rng.randint(1, 4), d, _log8(rng, d, 4 * d) if rng.random() < 0.3 else 4 * d, seq, n_seq, **how)
    elif kind == "xent":
        c = _xent("", _log(rng, 64, 8192), 64 * rng.randint(2, 16), _log8(rng, 1000, 32768, 0.2), **how)
        if c["vocab"] % 8:      # an unpadded vocabulary comes with the smaller models
            c["tokens"] = min(c["tokens"], 1024)
            c["d_model"] = min(c["d_model"], 512)
            c["vocab"] = min(c["vocab"], 16001)
    else:
        c = _lstm("", rng.randint(1, 4), 64 * rng.randint(1, 16), _log8(rng, 32, 1024), _log(rng, 1, 64), _log(rng, 4, 50), **how)
        if c["batch"] > 32 or c["hidden"] % 128:
            c["seq_len"] = min(c["seq_len"], 25)
    del c["name"]
    return c


# ----------------------------------------------------------------------------------------------------------- inputs
def _scale_and_opt(case):
    # the learning rate of the first iterations of a warm-up schedule
    opt = I.OptCfg(kind=case["opt"], lr=1e-6 if case["opt"] == "adam" else 1e-3, weight_decay=1e-4 if case["tuned"] else 0.0)
    return opt, I.ScaleCfg(init_scale=2.0 ** 10 if case["kind"] == "mlp" else 2.0 ** 15, growth_interval=100)


def _draws(seed):
    g = np.random.Generator(np.random.SFC64(seed))

    def uniform(shape, a):
        w = g.random(size=shape, dtype=np.float32)
        w -= np.float32(0.5)
        w *= np.float32(2 * a)
        return w

    return (lambda *s: g.standard_normal(size=s, dtype=np.float32)), uniform, g


def prepare(case, seed):
    normal, uniform, g = _draws(seed)
    opt, scale = _scale_and_opt(case)
    xavier = lambda o, i, rows=None: uniform((rows or o, i), math.sqrt(6.0 / (o + i)))  # noqa: E731
    zeros = lambda n: np.zeros(n, np.float32)  # noqa: E731
    kw = dict(prechecked=True, flat_update=True) if case["tuned"] else {}
    if case["kind"] == "mlp":
        R, di, dh, do = case["rows"], case["d_in"], case["d_hidden"], case["d_out"]
        wl = I.MLPWorkload(rows=R, d_in=di, d_hidden=dh, d_out=do, opt=opt, scale=scale)
        masters = {"w1": normal(dh, di) * np.float32(0.02), "b1": zeros(dh), "w2": normal(do, dh) * np.float32(0.02), "b2": zeros(do)}
        batch = {"x": normal(R, di), "target": normal(R, do)}
        step = St.MLPStep(wl, masters=masters, **kw)
    elif case["kind"] == "transformer":
        d, f = case["d_model"], case["d_ff"]
        wl = I.TransformerWorkload(n_layers=case["layers"], d_model=d, n_heads=d // 64, d_ff=f, seq_len=case["seq_len"],
                                   n_seq=case["n_seq"], opt=opt, scale=scale)
        masters = {}
        for l in range(case["layers"]):
            masters.update({f"l{l}.wqkv": xavier(d, d, 3 * d), f"l{l}.bqkv": zeros(3 * d), f"l{l}.wo": xavier(d, d), f"l{l}.bo": zeros(d),
                            f"l{l}.ln1_g": np.ones(d, np.float32), f"l{l}.ln1_b": zeros(d), f"l{l}.w1": xavier(f, d), f"l{l}.b1": zeros(f),
                            f"l{l}.w2": xavier(d, f), f"l{l}.b2": zeros(d), f"l{l}.ln2_g": np.ones(d, np.float32), f"l{l}.ln2_b": zeros(d)})
        batch = {"x": normal(wl.tokens, d), "target": normal(wl.tokens, d)}
        step = St.TransformerStep(wl, masters=masters, two_streams=case["tuned"], **kw)
    elif case["kind"] == "xent":
        T, d, V = case["tokens"], case["d_model"], case["vocab"]
        wl = I.XentWorkload(tokens=T, d_model=d, vocab=V, opt=opt, scale=scale)
        masters = {"w": xavier(V, d), "b": zeros(V)}
        batch = {"h": normal(T, d), "targets": g.integers(0, V, size=T, dtype=np.int64).astype(np.int32)}
        step = St.XentStep(wl, masters=masters, **kw)
    else:
        H, di, T, b = case["hidden"], case["d_in"], case["seq_len"], case["batch"]
        wl = I.LSTMWorkload(n_layers=case["layers"], hidden=H, d_in=di, batch_size=b, seq_len=T, opt=opt, scale=scale)
        masters = {}
        for l in range(case["layers"]):
            masters[f"l{l}.w"] = uniform((4 * H, (di if l == 0 else H) + H), 0.1)
            masters[f"l{l}.b"] = zeros(4 * H)
        batch = {"x": normal(T, b, di), "target": normal(T, b, H)}
        step = St.LSTMStep(wl, masters=masters, **kw)
    step.set_batch(batch)
    call = step.step
    if case["launch"] == "graph":
        step.forward_backward()          # every kernel has run once call by call, then the step is captured
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step.step()
        call = graph.replay
    return {"case": case, "step": step, "call": call}


def run(state):
    state["call"]()
    step, P = state["step"], state["step"].P
    out = {"loss": step.loss, "gradients": P.g16_arena, "masters": P.w32_arena, "weights": P.w16_arena, "scale_state": step.st}
    if P.m_arena is not None:
        out["m"], out["v"] = P.m_arena, P.v_arena
    kind = state["case"]["kind"]
    if kind == "mlp":
        out["y"], out["dx"] = step.y, step.dx
    elif kind == "transformer":
        out["y"], out["dx"] = step.act[-1]["y2"], step.dx_input
    elif kind == "xent":
        out["dlogits"], out["dx"] = step.logits, step.dh
    else:
        T, b, di = state["case"]["seq_len"], state["case"]["batch"], state["case"]["d_in"]
        out["y"], out["dx"] = step.y, step.dx_input.view(T, b, -1)[:, :, :di]
    return out


# ------------------------------------------------------------------------------------------------------ least work
def work(case):
    """Products: 2 M N K each for forward, input gradient and weight gradient (all three are computed everywhere).
    Bytes: parameter state (fp16 weight read, fp16 gradient written, masters and moments read and written, fp16 copy
    written), the batch read, the outputs and the gradient of the input written."""
    if case["kind"] == "mlp":
        R, di, dh, do = case["rows"], case["d_in"], case["d_hidden"], case["d_out"]
        params = dh * di + dh + do * dh + do
        flops = 6.0 * R * dh * (di + do)
        io = 2.0 * R * (2 * di + 2 * do)
    elif case["kind"] == "transformer":
        d, f, S, L = case["d_model"], case["d_ff"], case["seq_len"], case["layers"]
        T = S * case["n_seq"]
        params = L * (4 * d * d + 2 * d * f + 3 * d + d + f + d + 4 * d)
        flops = 3.0 * L * (8.0 * T * d * d + 4.0 * T * d * f + 4.0 * T * S * d)
        io = 2.0 * T * d * 4
    elif case["kind"] == "xent":
        T, d, V = case["tokens"], case["d_model"], case["vocab"]
        params = V * d + V
        flops = 6.0 * T * d * V
        io = 2.0 * T * d * 2 + 4.0 * T + 2.0 * T * V
    else:
        H, T, L = case["hidden"], case["seq_len"] * case["batch"], case["layers"]
        params = flops = 0.0
        for l in range(L):
            i = case["d_in"] if l == 0 else H
            params += 4 * H * (i + H) + 4 * H
            flops += 6.0 * T * 4 * H * (i + H)
        io = 2.0 * T * (2 * case["d_in"] + 2 * H)
    per_param = 2 + 2 + (24 if case["opt"] == "adam" else 8) + 2
    return {"bytes": per_param * float(params) + io, "flops": flops}


def tolerance(case):
    """Outputs are fp16 (one ulp is up to 2^-10 of a value) of fp32 sums whose order is free.  Measured against the same
    model with its inner dimensions permuted, so that every sum runs in another order, over two iterations: a product and
    cross-entropy move by 1e-5 and single values by one ulp; an LSTM by 1.1e-3, single values of a long weight-gradient
    sum by 5e-2; behind a ReLU an activation that moves by an ulp can flip a mask bit, which is worth a whole term of a
    gradient: 5e-3 for one encoder layer, 2e-2 for six, single values by up to 0.6 of the root mean square."""
    if case["kind"] == "transformer":
        return {"rel": min(0.03, 0.015 * (1 + case["layers"]) / 2), "max": 0.95}
    return {"mlp": {"rel": 1e-3, "max": 0.3}, "xent": {"rel": 5e-5, "max": 4e-3}, "lstm": {"rel": 4.5e-3, "max": 0.2}}[case["kind"]]
