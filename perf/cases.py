"""The work that programs have this library do, as measurable cases.

Five kinds of call, over the model shapes of `synth/workloads.py` (the tests and
the benchmark run the same shapes):

  score      trace_forward_bits over streams x positions: code lengths, the mean
             per position, optionally the logits
  update     a training loop: keep-activations forward + trace_adapt_step for a
             few positions, then the last gradient is read out
  gated      trace_gated_run: Algorithm 1 with the back-prop controller
  roundtrip  trace_compress, then trace_decompress by a second model that starts
             from the same state

Inputs come from the case and a seed alone.  Weights are normal draws: std 0.02
(the random start of the online setting) where the model trains, 0.05 (spread
logits, as frozen weights have them) where it only scores.  Training starts from
a checkpoint in mid-run, moments included.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2203_16114_amd as P

# the shapes of synth/workloads.py
SHAPES = {
    "tiny": dict(W=16, e=16, g=4, H=1, F=256, k=2, dtype="fp32"),
    "small": dict(W=32, e=32, g=4, H=4, F=512, k=2, dtype="fp32"),
    "main": dict(W=64, e=32, g=8, H=8, F=1024, k=3, dtype="bf16"),
    "adapt": dict(W=32, e=32, g=4, H=4, F=512, k=2, dtype="bf16"),
    "large": dict(W=64, e=64, g=8, H=8, F=2048, k=3, dtype="bf16"),
}
LR, BETA1, BETA2, EPS = 1e-3, 0.9, 0.999, 1e-8
START_STEP = 500  # Adam steps behind a training case's checkpoint


def _case(name, kind, shape, streams, steps, pos=None, **more):
    c = {"kind": kind, "shape": shape, **SHAPES[shape], "streams": streams, "steps": steps,
         "pos": SHAPES[shape]["W"] if pos is None else pos,  # position of the first byte that is predicted
         "logits": False, "performer": False, "untied": False, **more}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest call: one byte of a few streams, with logits (an interactive decoder)
        _case("tiny_step", "score", "tiny", 16, 1, logits=True),
        # one byte of every stream of a coder's batch, with logits
        _case("adapt_step", "score", "adapt", 4096, 1, pos=1000, logits=True),
        # scoring in single precision
        _case("small_score", "score", "small", 512, 128),
        # bulk scoring, the benchmark's own launch: 2^20 windows
        _case("main_score", "score", "main", 4096, 256),
        # files whose lengths and starts are no round numbers
        _case("main_ragged", "score", "main", 1021, 203, pos=77),
        # the wide model's scoring
        _case("large_score", "score", "large", 2048, 64),
        # Performer attention (positive random features)
        _case("main_performer", "score", "main", 512, 64, performer=True),
        # training in single precision
        _case("small_update", "update", "small", 512, 4),
        # training at the adaptation workload's batch
        _case("adapt_update", "update", "adapt", 4096, 4),
        # training of the wide model
        _case("large_update", "update", "large", 8192, 4),
        # the online loop: a forced update per step at first, then speculative forwards
        _case("adapt_gated", "gated", "adapt", 4096, 128),
        # a compressor and its decompressor, online updates included
        _case("adapt_roundtrip", "roundtrip", "adapt", 1024, 64),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["score"] * 5 + ["update"] * 3 + ["gated", "roundtrip"])
    shape = rng.choice(sorted(SHAPES))
    W = SHAPES[shape]["W"]
    pos = W + rng.choice([0, rng.randrange(1, 64), rng.randrange(64, 1024)])
    untied = rng.random() < 0.15
    if kind == "score":
        # at most what the largest listed launch of that shape holds
        most = {"tiny": 65536, "small": 65536, "main": 1 << 20, "adapt": 1 << 19, "large": 1 << 17}[shape]
        steps = _log_int(rng, 1, 256)
        streams = _log_int(rng, 1, min(4096, most // steps))
        performer = shape != "tiny" and rng.random() < 0.15 and streams * steps <= 32768
        logits = rng.random() < 0.4 and streams * steps <= 65536
        return _case(None, kind, shape, streams, steps, pos, performer=performer, untied=untied and not performer,
                     logits=logits)
    if kind == "update":
        most = {"tiny": 1024, "small": 1024, "main": 4096, "adapt": 4096, "large": 8192}[shape]
        return _case(None, kind, shape, _log_int(rng, 16, most), rng.randrange(1, 5), pos, untied=untied)
    if kind == "gated":
        most = {"tiny": 512, "small": 512, "main": 1024, "adapt": 4096, "large": 512}[shape]
        return _case(None, kind, shape, _log_int(rng, 64, most), rng.randrange(20, 129), pos)
    most = {"tiny": 512, "small": 512, "main": 512, "adapt": 1024, "large": 256}[shape]
    return _case(None, kind, shape, _log_int(rng, 4, most), rng.randrange(8, 65))


# ---- inputs ----------------------------------------------------------------
def _model_args(c):
    return dict(W=c["W"], e=c["e"], g=c["g"], H=c["H"], F=c["F"], k=c["k"], dtype=c["dtype"], untied_ffn=c["untied"],
                lr=LR, beta1=BETA1, beta2=BETA2, eps=EPS)


def _layout(c):
    """(name, shape) of the flat parameter vector's tensors, in order."""
    T, d, F, r = c["W"] // c["g"], c["g"] * c["e"], c["F"], c["k"] if c["untied"] else 1
    return [("E", (256, c["e"])), ("P", (T, d)), ("Wq", (d, d)), ("Wk", (d, d)), ("Wv", (d, d)), ("Wo", (d, d)),
            ("W1", (r, d, F)), ("W2", (r, F, d)), ("Wout", (d, 256)), ("bout", (256,))]


def _split(c, flat):
    out, o = {}, 0
    for name, shape in _layout(c):
        n = math.prod(shape)
        out[name] = flat[o:o + n].reshape(shape)
        o += n
    return out


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _weights(c, gen):
    n = sum(math.prod(s) for _, s in _layout(c))
    flat = torch.randn(n, generator=gen, device="cuda") * (0.05 if c["kind"] == "score" else 0.02)
    flat[-256:] = 0  # bout
    return flat


def _streams(B, L, gen):
    """Bytes of three sources, by stream: an order-1 Markov chain with sparse
    rows, a Zipf distribution over a permutation, and uniform bytes with runs."""
    u = torch.rand(B, L, generator=gen, device="cuda")
    perm = torch.randperm(256, generator=gen, device="cuda")
    zipf = torch.cumsum(1.0 / torch.arange(1, 257, device="cuda", dtype=torch.float64) ** 1.2, 0)
    s = perm[torch.searchsorted((zipf / zipf[-1]).float(), u).clamp_(max=255)]
    rows = torch.cumsum(torch.rand(256, 256, generator=gen, device="cuda", dtype=torch.float64) ** 12, 1)
    rows = (rows / rows[:, -1:]).float()
    state = s[0::3, 0]
    for i in range(1, L):
        state = torch.searchsorted(rows[state], u[0::3, i:i + 1].contiguous()).clamp_(max=255)[:, 0]
        s[0::3, i] = state
    flat = (u[2::3] * 256).long().clamp_(max=255)
    start = torch.where(torch.rand(flat.shape, generator=gen, device="cuda") < 0.5,
                        torch.arange(L, device="cuda").expand_as(flat), torch.zeros_like(flat))
    s[2::3] = torch.gather(flat, 1, torch.cummax(start, 1).values)
    return s.to(torch.uint8)


def _features(c, gen):
    m, dh = (128, 32) if c["g"] * c["e"] // c["H"] <= 32 else (256, 64)
    return torch.randn(m, dh, generator=gen, device="cuda")


def _inputs(c, seed):
    """Everything that prepare() and exact() build from."""
    gen = _gen(seed)
    flat = _weights(c, gen)
    streams = _streams(c["streams"], c["pos"] + c["steps"], gen)
    extra = {}
    if c["performer"]:
        extra["omega"] = _features(c, gen)
    if c["kind"] != "score":  # Adam moments of a run under way
        extra["m"] = 3e-5 * torch.randn(flat.numel(), generator=gen, device="cuda")
        extra["v"] = 1e-8 * (0.5 + torch.rand(flat.numel(), generator=gen, device="cuda"))
    return flat, streams, extra


def prepare(case, seed):
    c = case
    flat, streams, extra = _inputs(c, seed)
    B, S = c["streams"], c["steps"]
    trains = c["kind"] != "score"
    args = _model_args(c)
    if c["performer"]:
        args["attention"] = "performer"
    # a scoring model is made for its bulk launches, a training one for its batch
    # (the online loop's speculative forwards run 64 positions at a time)
    windows = B * (S if c["kind"] == "score" else 64 if c["kind"] == "gated" else 1)

    def model():
        m = P.TraceModel(**args, max_windows=windows, max_keep=B if trains else 0)
        if trains:
            m.set_state(flat.cpu().numpy(), extra["m"].cpu().numpy(), extra["v"].cpu().numpy(), START_STEP)
        else:
            m.init_weights(0, flat=flat.cpu().numpy())
        if c["performer"]:
            m.set_features(extra["omega"].cpu().numpy())
        return m

    st = {"case": c, "model": model(), "streams": streams}
    if c["kind"] == "score":
        st["bits"] = torch.empty(B * S, dtype=torch.float32, device="cuda")
        st["step_ce"] = torch.empty(S, dtype=torch.float64, device="cuda")
        st["logits"] = torch.empty(B * S, 256, dtype=torch.float32, device="cuda") if c["logits"] else None
    if c["kind"] == "update":
        st["bits"] = torch.empty(B, dtype=torch.float32, device="cuda")
        st["grads"] = torch.empty(flat.numel(), dtype=torch.float32, pin_memory=True)
    if c["kind"] == "roundtrip":
        st["decoder"] = model()
        st["streams"] = streams.contiguous()
    torch.cuda.synchronize()
    return st


def run(state):
    c, m, s = state["case"], state["model"], state["streams"]
    if c["kind"] == "score":
        r = m.forward_bits(s, c["pos"], c["steps"], bits=state["bits"], logits=state["logits"], step_ce=state["step_ce"])
        return {k: v for k, v in r.items() if v is not None}
    if c["kind"] == "update":
        for i in range(c["steps"]):
            m.forward_bits(s, c["pos"] + i, 1, bits=state["bits"], keep=True)
            m.adapt_step()
        g = state["grads"]  # trace_get_grads into pinned memory: the C call behind TraceModel.grads()
        P.check(P.lib().trace_get_grads(m._h, g.data_ptr(), g.numel()))
        return {"bits": state["bits"], "grads": _split(c, g)}
    if c["kind"] == "gated":
        ce, decisions, _ = m.gated_run(s, c["pos"], c["steps"])
        theta, adam_m, adam_v, _ = m.get_state()
        return {"step_ce": ce, "theta": theta, "m": adam_m, "v": adam_v}
    codes, _ = m.compress(s, mode=P.MODE_GATED)
    back, _ = state["decoder"].decompress(codes, s.shape[1], mode=P.MODE_GATED)
    # the bytes of a code follow the last bit of the logits; its length does not
    return {"bytes": back, "code_lengths": np.array([len(x) for x in codes], np.float64)}


# ---- what a pass cannot do without ------------------------------------------
def _forward_flops(c, B, S):
    """Multiply-adds x 2 of B x S windows: keys and values once per distinct byte
    group of a stream (neighbouring windows share them), the rest per window."""
    T, d, F, k = c["W"] // c["g"], c["g"] * c["e"], c["F"], c["k"]
    groups = min(T * S, S + c["W"] - c["g"])
    f = B * groups * 4 * d * d + B * S * (4 * d * d + 4 * T * d + 4 * k * d * F + 512 * d)
    if c["performer"]:
        m, dh = (128, 32) if d // c["H"] <= 32 else (256, 64)
        f += B * S * (T + 1) * c["H"] * m * dh * 2
    return f


def _backward_flops(c, B):
    """Gradients of the FFN and the head (two products each), the four D x D
    projections' and their inputs' (last query row; rank-one keys and values)."""
    T, d, F, k = c["W"] // c["g"], c["g"] * c["e"], c["F"], c["k"]
    return B * (8 * k * d * F + 1024 * d + 16 * d * d + 8 * T * c["H"] * d)


def work(case):
    c = case
    n = sum(math.prod(s) for _, s in _layout(c))
    B, S = c["streams"], c["steps"]
    wb = 2 if c["dtype"] == "bf16" else 4
    one = B * c["W"] + n * wb + B * 4  # one position: window bytes, weights, code lengths
    adam = n * 28
    if c["kind"] == "score":
        return {"bytes": B * (S + c["W"]) + n * wb + B * S * 4 + S * 8 + (B * S * 1024 if c["logits"] else 0),
                "flops": _forward_flops(c, B, S)}
    if c["kind"] == "update":
        return {"bytes": S * (one + adam) + n * 4, "flops": S * (_forward_flops(c, B, 1) + _backward_flops(c, B))}
    if c["kind"] == "gated":
        u = min(S, 16)  # the updates of a cold controller
        return {"bytes": B * (S + c["W"]) + n * wb + S * 8 + u * (one + adam) + n * 12,
                "flops": _forward_flops(c, B, S) + u * (_forward_flops(c, B, 1) + _backward_flops(c, B))}
    u = min(S, 16)
    return {"bytes": 2 * (S * one + u * (one + adam)) + 2 * B * (S + c["W"]),
            "flops": 2 * (S * _forward_flops(c, B, 1) + u * (_forward_flops(c, B, 1) + _backward_flops(c, B)))}


def tolerance(case):
    """About four times the largest error against exact() that the listed cases
    showed: fp32 bits 5e-8, logits 6e-7, gradients 1.1e-6; bf16 bits 5e-4 (the
    wide model), logits 3.2e-3, gradients 5.2e-3 (the key weights')."""
    c = case
    if c["kind"] == "roundtrip":  # decoded bytes exactly; code lengths (floats) by the logits' rounding
        return {"rel": 2e-3, "max": 0.05, "differ": 0.0}
    if c["dtype"] == "fp32":
        return {"rel": 3e-6, "max": 1e-4} if c["kind"] == "score" else {"rel": 1e-5, "max": 1e-2}
    if c["kind"] == "score":
        return {"rel": 1.2e-2, "max": 0.2} if c["logits"] else {"rel": 2e-3, "max": 0.05}
    return {"rel": 2e-2, "max": 0.8}


# ---- the same in 64 bits ------------------------------------------------------
def _logits64(c, p, win, omega):
    """Head outputs of windows [n][W] (long), parameters p in float64."""
    n, T, d, H = win.shape[0], c["W"] // c["g"], c["g"] * c["e"], c["H"]
    dh = d // H
    x = p["E"][win].reshape(n, T, d) + p["P"]
    last = x[:, -1]
    q = (last @ p["Wq"]).reshape(n, H, dh)
    k = (x @ p["Wk"]).reshape(n, T, H, dh)
    v = (x @ p["Wv"]).reshape(n, T, H, dh)
    if omega is None:
        a = torch.softmax((q[:, None] * k).sum(-1) / math.sqrt(dh), 1)  # [n][T][H]
    else:
        qs, ks = q * dh ** -0.25, k * dh ** -0.25
        f = ((ks + qs[:, None]) @ omega.t()) - ((qs * qs).sum(-1)[:, None] + (ks * ks).sum(-1))[..., None] / 2
        a = torch.softmax(torch.logsumexp(f, -1), 1)
    y = (a[..., None] * v).sum(1).reshape(n, d) @ p["Wo"] + last
    for r in range(c["k"]):
        w = r if c["untied"] else 0
        u = y @ p["W1"][w]
        y = y + (u * 0.5 * (1 + torch.erf(u / math.sqrt(2)))) @ p["W2"][w]
    return y @ p["Wout"] + p["bout"]


def _nats(z, target):
    return torch.logsumexp(z, 1) - z.gather(1, target[:, None])[:, 0]


def _windows(c, streams, pos, S):
    """Windows [B][S][W] and targets [B][S] of positions pos .. pos + S."""
    s = streams.long()
    return s[:, pos - c["W"]:pos + S - 1].unfold(1, c["W"], 1), s[:, pos:pos + S]


def exact(case, seed):
    c = case
    if c["kind"] == "roundtrip":
        return {"bytes": _inputs(c, seed)[1], "code_lengths": None}
    if c["kind"] == "gated":
        return None  # the decisions hang on the last bit of the means
    flat, streams, extra = _inputs(c, seed)
    B, S, ln2 = c["streams"], c["steps"], math.log(2)
    if c["kind"] == "score":
        p = _split(c, flat.double())
        omega = extra["omega"].double() if c["performer"] else None
        win, tgt = _windows(c, streams, c["pos"], S)
        win, tgt = win.reshape(-1, c["W"]), tgt.reshape(-1)
        bits, logits, chunk = [], [], 4096 if c["performer"] else 16384
        for i in range(0, B * S, chunk):
            z = _logits64(c, p, win[i:i + chunk], omega)
            bits.append(_nats(z, tgt[i:i + chunk]) / ln2)
            if c["logits"]:
                logits.append(z)
        bits = torch.cat(bits)
        out = {"bits": bits, "step_ce": bits.view(B, S).mean(0)}
        if c["logits"]:
            out["logits"] = torch.cat(logits)
        return out
    th, m, v = (t.double() for t in (flat, extra["m"], extra["v"]))
    for i in range(S):
        win, tgt = _windows(c, streams, c["pos"] + i, 1)
        win, tgt = win[:, 0], tgt[:, 0]
        leaf = th.clone().requires_grad_(True)
        grad, bits = torch.zeros_like(th), []
        for j in range(0, B, 4096):
            nats = _nats(_logits64(c, _split(c, leaf), win[j:j + 4096], None), tgt[j:j + 4096])
            grad += torch.autograd.grad(nats.sum() / B, leaf)[0]
            bits.append(nats.detach() / ln2)
        t = START_STEP + i + 1
        m = BETA1 * m + (1 - BETA1) * grad
        v = BETA2 * v + (1 - BETA2) * grad * grad
        th = th - LR * (m / (1 - BETA1 ** t)) / ((v / (1 - BETA2 ** t)).sqrt() + EPS)
    return {"bits": torch.cat(bits), "grads": {k: g for k, g in _split(c, grad).items()}}
