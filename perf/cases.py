"""Performance cases of the RLA / RDN sequence-mixing layer: the calls that a
serving engine and a training loop make through the package's entry points,
each with its inputs, its work and a 64-bit reference.

A case is a dict of plain values:
  kind      "decode" (a few tokens from resident states), "forward" (prefill,
            scoring) or "train" (forward, then every gradient)
  op        "rdn" or "rla"
  dtype, out  element types of q, k, v, dO and of o, dq, dk, dv
  H, dk, dv   heads and head dimensions
  B, T      dense [B, T, H, d] inputs; or, packed (cu_seqlens),
  tokens, lo, hi, pack  sequences of lo..hi tokens drawn with the seed `pack`
            until they fill `tokens` (the last one is cut)
  raw       q, k before SiLU and L2 normalisation, gates as pre-activations
  states    initial states given (a continued sequence)
  own       the caller keeps the workspace and the outputs; otherwise each call
            allocates them
  static    (forward) the allocation-free entry point
  saved     (train) the forward saves for the backward; otherwise the backward
            recomputes it (activation checkpointing)
"""
import math
import random

import torch

import paper_2509_25223_amd as rla

CLIP = 1.0
PREPROC = rla.RLA_FLAG_QK_SILU_L2NORM | rla.RLA_FLAG_GATE_PREACT
GATES = ("alpha_s", "beta", "alpha_r", "gamma")


def _case(name, kind, op="rdn", dtype="bf16", out="bf16", H=16, dk=128, dv=128, B=0, T=0, tokens=0,
          lo=0, hi=0, pack=0, raw=False, states=False, own=True, static=False, saved=False):
    c = dict(kind=kind, op=op, dtype=dtype, out=out, H=H, dk=dk, dv=dv, B=B, T=T, tokens=tokens, lo=lo,
             hi=hi, pack=pack, raw=raw, states=states, own=own, static=static, saved=saved)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one user's next token: the smallest call, latency and launch
        _case("decode_b1", "decode", B=1, T=1, states=True),
        # a full serving batch, one token each: the states are read and written once (HBM)
        _case("decode_b256", "decode", out="f32", B=256, T=1, states=True),
        # verification of a drafted continuation: several tokens a call, pre-processing fused
        _case("decode_verify", "decode", op="rla", B=48, T=5, states=True, raw=True),
        # one more turn of a conversation: a short ragged prompt onto given states
        _case("prefill_turn", "forward", B=1, T=777, states=True, static=True),
        # one long prompt: few sequences, a long chain of chunks
        _case("prefill_long", "forward", B=1, T=16384, out="f32"),
        # a batch of prompts of all lengths, packed, raw projections
        _case("prefill_packed", "forward", tokens=20011, lo=30, hi=4000, pack=3, raw=True),
        # a dense evaluation batch of the additive model, plain calls that allocate
        _case("forward_rla", "forward", op="rla", out="f32", B=4, T=2048, own=False),
        # scoring of a long-document corpus: the largest call
        _case("forward_corpus", "forward", out="f32", tokens=262144, lo=512, hi=32768, pack=4),
        # the training step of the language-model layer
        _case("train", "train", out="f32", B=4, T=4096, saved=True),
        # a training step on packed documents from the raw projections
        _case("train_packed", "train", tokens=16000, lo=100, hi=6000, pack=5, raw=True, saved=True),
        # a small model with head dimension 64 under activation checkpointing
        _case("train_d64", "train", op="rla", H=8, dk=64, dv=64, B=4, T=1000, raw=True),
        # the fp32 path, for checks of a model against its reference
        _case("train_f32", "train", dtype="f32", out="f32", H=4, dk=64, dv=64, B=2, T=500, states=True,
              saved=True),
    ]


def _between(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "forward", "forward", "train", "train"])
    op = rng.choice(["rdn", "rdn", "rla"])
    out = rng.choice(["bf16", "f32"])
    raw, states = rng.random() < 0.4, rng.random() < 0.4
    if kind == "decode":
        return _case("", kind, op=op, out=out, H=rng.choice([8, 16, 16, 32]), B=_between(rng, 1, 300),
                     T=rng.choice([1, 1, 1, 2, 3, 4, 6, 8]), states=True, raw=raw)
    H, dk, dv, dtype = rng.choice([4, 8, 16, 16, 32]), 128, 128, "bf16"
    shape = rng.random()
    if shape < 0.15:
        dk = dv = 64
    elif shape < 0.22:
        dk, dv = rng.choice([(64, 128), (128, 64)])
    elif shape < 0.3:
        H, dk, dv, dtype, out = rng.choice([2, 4, 8]), 64, 64, "f32", "f32"
    most = (4096 if dtype == "f32" else 131072 if kind == "forward" else 24000) * 16 // max(H, 16)
    if rng.random() < 0.4:
        tokens = _between(rng, 1000, most)
        return _case("", kind, op=op, dtype=dtype, out=out, H=H, dk=dk, dv=dv, tokens=tokens,
                     lo=rng.randint(1, 200), hi=_between(rng, 400, max(500, tokens // 2)),
                     pack=rng.randrange(1 << 20), raw=raw, states=states, saved=rng.random() < 0.7)
    T = _between(rng, 100, min(most, 16384))
    return _case("", kind, op=op, dtype=dtype, out=out, H=H, dk=dk, dv=dv,
                 B=_between(rng, 1, max(1, min(16, most // T))), T=T, raw=raw, states=states,
                 own=rng.random() < 0.7, saved=rng.random() < 0.7)


def _lengths(c):
    if not c["tokens"]:
        return [c["T"]] * c["B"]
    r, got = random.Random(c["pack"]), []
    while sum(got) < c["tokens"]:
        got.append(min(r.randint(c["lo"], c["hi"]), c["tokens"] - sum(got)))
    return got


def _type(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _inputs(c, seed):
    """The tensors of one call, on the GPU (packed [T, H, d] or dense [B, T, H, d])."""
    dev = torch.device("cuda")
    g = torch.Generator(dev).manual_seed(seed)
    lens = _lengths(c)
    lead = (sum(lens),) if c["tokens"] else (c["B"], c["T"])
    H, dk, dv, dt = c["H"], c["dk"], c["dv"], _type(c["dtype"])

    def normal(*shape):
        return torch.randn(*shape, device=dev, generator=g)

    x = {}
    for n in ("q", "k"):
        y = normal(*lead, H, dk)
        x[n] = (y if c["raw"] else y / y.norm(dim=-1, keepdim=True)).to(dt)
    x["v"] = normal(*lead, H, dv).to(dt)
    mu = {"rdn": 2.0, "rla": 3.0}[c["op"]]
    for n in GATES:
        z = normal(*lead, H) + (mu if n.startswith("alpha") and not c["raw"] else 0.0)
        x[n] = z if c["raw"] else torch.sigmoid(z)
    # Mamba-2 decay parameters per head: a > 0, b (decays of about the same range as the plain gates')
    x["decay_param"] = None
    if c["raw"]:
        x["decay_param"] = torch.stack([0.05 + 0.3 * torch.rand(H, device=dev, generator=g), 0.5 * normal(H)])
    N = len(lens)
    for n in ("S0", "R0"):
        x[n] = normal(N, H, dk, dv) / math.sqrt(dk) if c["states"] else None
    x["cu"] = None
    if c["tokens"]:
        x["cu"] = torch.tensor([0] + lens, device=dev).cumsum(0).to(torch.int32)
    if c["kind"] == "train":
        x["dO"] = normal(*lead, H, dv).to(dt)
        x["v"] = _off_the_kink(c, x)
    return x


def _transform(c, x):
    """(q, k, alpha_s, beta, alpha_r, gamma) as the recurrence takes them."""
    q, k = x["q"], x["k"]
    if not c["raw"]:
        return q, k, x["alpha_s"], x["beta"], x["alpha_r"], x["gamma"]

    def rows(y):
        y = torch.nn.functional.silu(y)
        return y / y.norm(dim=-1, keepdim=True).clamp_min(1e-12)

    a, b = x["decay_param"][0], x["decay_param"][1]

    def decay(z):
        return torch.exp(-a * torch.nn.functional.softplus(z + b))

    return (rows(q), rows(k), decay(x["alpha_s"]), torch.sigmoid(x["beta"]), decay(x["alpha_r"]),
            torch.sigmoid(x["gamma"]))


def _rows(c):
    """[N, longest] token of each sequence's t-th place and whether it is one (dense inputs: all are)."""
    lens = torch.tensor(_lengths(c), device="cuda")
    t = torch.arange(int(lens.max()), device="cuda")
    there = t[None] < lens[:, None]
    return torch.where(there, lens.cumsum(0)[:, None] - lens[:, None] + t[None], 0), there


def _pairs(c, y, fill=None):
    """[..., H] or [..., H, d] inputs as [N * H, longest(, d)]; `fill`: the value past a sequence's end."""
    at, there = _rows(c)
    H = c["H"]
    y = y.reshape(-1, *y.shape[-(1 if fill is not None else 2):])[at]   # [N, longest, H(, d)]
    if fill is not None:
        y = torch.where(there[..., None], y, torch.full_like(y[:1, :1], fill))
    y = y.transpose(1, 2)
    return y.reshape(y.shape[0] * H, *y.shape[2:])


def _tokens(c, y, like):
    """_pairs undone, in the shape of `like`."""
    _, there = _rows(c)
    y = y.reshape(there.shape[0], c["H"], *y.shape[1:]).transpose(1, 2)
    return y[there].reshape(like.shape)


def _recurrence_inputs(c, x):
    """What the token recurrence reads, as [N * H, longest(, d)]; past a sequence's end the gates leave
    the states as they are."""
    q, k, a_s, b, a_r, g = _transform(c, x)
    return [_pairs(c, q), _pairs(c, k), _pairs(c, x["v"]), _pairs(c, a_s, 1.0), _pairs(c, b, 0.0),
            _pairs(c, a_r, 1.0), _pairs(c, g, 0.0)]


def _states(c, x, like):
    n = like.shape[0]
    return [torch.zeros(n, c["dk"], c["dv"], device=like.device, dtype=like.dtype) if x[s] is None
            else x[s].to(like.dtype).reshape(n, c["dk"], c["dv"]) for s in ("S0", "R0")]


def _off_the_kink(c, x):
    """v with no residual v - S k within 0.01 of the clip bound, where its derivative jumps: the
    gradients of two correct implementations then agree element by element.  About 1 % of the elements
    move, by up to 0.03."""
    wide = {n: t if t is None else t.float() if t.is_floating_point() else t for n, t in x.items()}
    _, k, v, a_s, b, _, _ = _recurrence_inputs(c, wide)
    S, _ = _states(c, wide, v)
    for t in range(v.shape[1]):
        kt, vt, at, bt = k[:, t, None], v[:, t, None], a_s[:, t, None, None], b[:, t, None, None]
        p = torch.bmm(kt, S)
        r = vt - p
        far = torch.where(r.abs() < CLIP, CLIP - 0.03, CLIP + 0.03)
        vt.copy_(torch.where((r.abs() - CLIP).abs() < 0.015, p + torch.copysign(far, r), vt).to(_type(c["dtype"])))
        S = torch.baddbmm(at * S, kt.transpose(1, 2), bt * (vt - at * p if c["op"] == "rdn" else vt))
    return _tokens(c, v, x["v"]).to(x["v"].dtype)


def prepare(case, seed):
    c = dict(case)
    x = _inputs(c, seed)
    dev, out = x["q"].device, _type(c["out"])
    # entry points, arguments and the buffers that a caller keeps
    x["variants"] = PREPROC if c["raw"] else 0
    x["case"] = c
    shape = (len(_lengths(c)), c["H"], c["dk"], c["dv"])
    new = lambda s, t=torch.float32: torch.empty(s, dtype=t, device=dev)   # noqa: E731
    x["buffers"], x["workspace"] = {}, None
    if c["kind"] == "decode":
        x["buffers"] = dict(out=new(x["v"].shape, out), S_out=new(shape), R_out=new(shape))
    elif c["static"]:
        x["buffers"] = dict(out=new(x["v"].shape, out), S_final=new(shape), R_final=new(shape))
    elif c["own"]:
        x["buffers"] = dict(out=new(x["v"].shape, out))
    if c["kind"] != "decode" and not c["static"] and (c["own"] or c["saved"]):
        problem = rla.make_problem(x["q"], x["v"], x["cu"], CLIP, out, x["variants"], x["decay_param"])
        fwd, bwd = ((rla.RLA_OP_RDN_FORWARD, rla.RLA_OP_RDN_BACKWARD) if c["op"] == "rdn" else
                    (rla.RLA_OP_RLA_FORWARD, rla.RLA_OP_RLA_BACKWARD))
        x["workspace"] = new(rla.rla_workspace_size(problem, bwd if c["kind"] == "train" else fwd), torch.uint8)
    x["grads"] = None
    if c["kind"] == "train" and c["own"]:
        x["grads"] = {"d" + n: new(x[n].shape, out) for n in ("q", "k", "v")}
        x["grads"].update({"d" + n: new(x[n].shape) for n in GATES}, dS0=new(shape), dR0=new(shape))
        if c["raw"]:
            x["grads"]["ddecay_param"] = new(x["decay_param"].shape)
    return x


def run(x):
    c = x["case"]
    inputs = [x[n] for n in ("q", "k", "v") + GATES]
    how = dict(clip=CLIP, out_dtype=_type(c["out"]), variants=x["variants"], decay_param=x["decay_param"])
    if c["kind"] == "decode":
        step = rla.rdn_decode if c["op"] == "rdn" else rla.rla_decode
        o, S, R = step(*inputs, S_in=x["S0"], R_in=x["R0"], **x["buffers"], **how)
        return {"o": o, "S": S, "R": R}
    how.update(S0=x["S0"], R0=x["R0"], cu_seqlens=x["cu"])
    if c["static"]:
        o, S, R = rla.rdn_forward_noalloc(*inputs, **x["buffers"], **how)
        return {"o": o, "S": S, "R": R}
    how["workspace"] = x["workspace"]
    forward = rla.rdn_forward if c["op"] == "rdn" else rla.rla_forward
    if c["kind"] == "forward":
        o, S, R = forward(*inputs, **x["buffers"], **how)
        return {"o": o, "S": S, "R": R}
    o, _, _ = forward(*inputs, return_states=False, save_for_backward=c["saved"], **x["buffers"], **how)
    backward = rla.rdn_backward if c["op"] == "rdn" else rla.rla_backward
    grads = backward(*inputs, x["dO"], grads=x["grads"], use_saved=c["saved"], **how)
    return {"o": o, **grads}


def work(case):
    """Each input read once and each output written once; the products of the token recurrence
    (S k, S q, R k, R q and two rank-one updates a token), twice as many again for the gradients."""
    c = case
    rows, N = sum(_lengths(c)) * c["H"], len(_lengths(c)) * c["H"]
    el, oel = (2 if c["dtype"] == "bf16" else 4), (2 if c["out"] == "bf16" else 4)
    state = 2 * 4 * c["dk"] * c["dv"] * N
    b = rows * ((2 * c["dk"] + c["dv"]) * el + c["dv"] * oel + 16)
    f = rows * 12 * c["dk"] * c["dv"]
    if c["states"]:
        b += state
    if c["kind"] != "train":
        return {"bytes": b + state, "flops": f}
    b += rows * (c["dv"] * el + (2 * c["dk"] + c["dv"]) * oel + 16) + state
    return {"bytes": b, "flops": 3 * f}


def tolerance(case):
    """About four times the largest relative error against 64 bits over the listed cases: outputs rounded
    to bf16 1.7e-3; fp32 outputs of the bf16 path 4.5e-4; the fp32 path 6.4e-7; decoding (fp32 arithmetic
    throughout) 1.0e-7."""
    if case["out"] == "bf16":
        return {"rel": 7e-3}
    if case["kind"] == "decode":
        return {"rel": 5e-7}
    return {"rel": 3e-6 if case["dtype"] == "f32" else 2e-3}


def _token(op, q, k, v, a_s, b, a_r, g, S, R):
    """One token of the recurrence; the states as [pairs, dk, dv]."""
    Sk, Rk = torch.bmm(k, S), torch.bmm(k, R)
    r = (v - Sk).clamp(-CLIP, CLIP)
    u, w = (v - a_s * Sk, r - a_r * Rk) if op == "rdn" else (v, r)
    kT = k.transpose(1, 2)
    R = torch.baddbmm(a_r * R, kT, g * w)
    o = a_s * torch.bmm(q, S) + g * torch.bmm(q, R)
    return o, torch.baddbmm(a_s * S, kT, b * u), R


def _span(op, x, S, R):
    """A stretch of tokens ([pairs, tokens(, d)] inputs): its outputs and the states after it."""
    outs = []
    for t in range(x[0].shape[1]):
        rows = [y[:, t, None] for y in x[:3]] + [y[:, t, None, None] for y in x[3:]]
        o, S, R = _token(op, *rows, S, R)
        outs.append(o)
    return torch.cat(outs, 1), S, R


SPAN = 64


def exact(case, seed):
    c = dict(case)
    lens = _lengths(c)
    longest, pairs = max(lens), len(lens) * c["H"]
    # about 20 s: launches of the token loop, or the states' traffic in it
    if longest * max(1.0, pairs * c["dk"] * c["dv"] / 2 ** 20) * (4 if c["kind"] == "train" else 1) > 70000:
        return None
    x = _inputs(c, seed)
    wide = {n: t.double() if t is not None and t.is_floating_point() else t for n, t in x.items()}
    raw = [n for n in ("q", "k", "v") + GATES + ("decay_param",) if wide[n] is not None]
    train = c["kind"] == "train"
    if train:
        for n in raw:
            wide[n].requires_grad_(True)
    with torch.set_grad_enabled(train):
        y = _recurrence_inputs(c, wide)
    S, R = _states(c, wide, y[0])
    starts, outs = [], []
    with torch.no_grad():
        for t in range(0, longest, SPAN):
            starts.append((S, R))
            o, S, R = _span(c["op"], [z[:, t:t + SPAN] for z in y], S, R)
            outs.append(o)
    o = _tokens(c, torch.cat(outs, 1), x["v"])
    shape = (len(lens), c["H"], c["dk"], c["dv"])
    if not train:
        return {"o": o, "S": S.reshape(shape), "R": R.reshape(shape)}
    dO = _pairs(c, wide["dO"]) * (_pairs(c, torch.ones_like(wide["gamma"]), 0.0)[..., None])
    dS, dR = torch.zeros_like(S), torch.zeros_like(R)
    parts = []
    for i in reversed(range(len(starts))):
        t = i * SPAN
        leaves = [z[:, t:t + SPAN].detach().requires_grad_(True) for z in y]
        s, r = (z.detach().requires_grad_(True) for z in starts[i])
        got = _span(c["op"], leaves, s, r)
        *d, dS, dR = torch.autograd.grad(got, leaves + [s, r], [dO[:, t:t + SPAN], dS, dR])
        parts.append(d)
    dy = [torch.cat([p[j] for p in reversed(parts)], 1) for j in range(len(y))]
    grads = torch.autograd.grad(y, [wide[n] for n in raw], dy)
    out = {"o": o.detach(), **{"d" + n: d for n, d in zip(raw, grads)}}
    return dict(out, dS0=dS.reshape(shape), dR0=dR.reshape(shape))
