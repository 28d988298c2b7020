"""The workloads this framework's speed is judged on, through its public entry
points: packed variable-length attention (forward and backward) from a tiny
pack to a long Ulysses shard, and the transformer layer around it.

``listed()`` names the fixed cases, ``draw(rng)`` gives another case of the
same ranges; ``prepare`` / ``run`` execute one, ``work`` states what it cannot
do without, ``exact`` computes its outputs in float64 with plain torch and
``tolerance`` bounds the difference.

A case is a dict of plain values.  Common keys: ``kind`` ("attn" or
"layer"), ``heads``, ``dim``, ``causal``, and the sequence lengths of the
packed batch by ``mix``:
  "list"      the lengths in ``lens`` (a comma-separated text);
  "uniform"   ``n`` sequences drawn uniformly from ``lens``;
  "lognormal" documents, log-normal (``median``, ``sigma``) clipped to [lo, hi],
              packed in order into at most ``tokens``;
  "temporal"  Transformer-2D temporal attention: clips of 1/16/32/51 frames x
              256/1620/3600 tokens give one sequence per token position, packed
              in order into at most ``tokens``.
The lengths are drawn from ``mix_seed`` (they are part of the case); ``prepare``'s
seed makes the tensors only.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_07524_amd as dcp
from paper_2608_07524_amd import inputs

LAYER_EPS = 1e-6


# ---------------------------------------------------------------------------
# the cases

def listed():
    return [
        # The smallest call: four short sequences through the per-call API, as an
        # interactive or smoke run makes it; launches and host work dominate.
        dict(name="tiny", kind="attn", api="call", bwd=True, heads=4, dim=64, causal=False, mix="list",
             lens="37,64,128,200"),
        # One video frame (3,600 tokens at 720p) of a Transformer-2D model, per call.
        dict(name="frame", kind="attn", api="call", bwd=True, heads=16, dim=72, causal=False, mix="list", lens="3600"),
        # Validation or scoring: the forward alone, one document of odd length.
        dict(name="doc_fwd", kind="attn", api="call", bwd=False, heads=32, dim=128, causal=True, mix="list",
             lens="3001"),
        # One device's Ulysses shard (SP = 8 of 16 heads) of a short, a middling
        # and a long sequence; the batch is prepared once, as every layer of the
        # model reuses it.
        dict(name="shard_4k", kind="attn", api="batch", bwd=True, heads=2, dim=128, causal=False, mix="list",
             lens="4096"),
        dict(name="shard_16k", kind="attn", api="batch", bwd=True, heads=2, dim=128, causal=False, mix="list",
             lens="16384"),
        dict(name="shard_128k", kind="attn", api="batch", bwd=True, heads=2, dim=128, causal=False, mix="list",
             lens="131072"),
        # A language-model pack of log-normal documents, causal.
        dict(name="text_pack", kind="attn", api="batch", bwd=True, heads=32, dim=128, causal=True, mix="lognormal",
             median=2048, sigma=1.0, lo=128, hi=131072, tokens=131072, mix_seed=0),
        # The Transformer-1D model's attention (48 heads of width 64) over many
        # short documents and a few long ones.
        dict(name="docs_1d", kind="attn", api="batch", bwd=True, heads=48, dim=64, causal=True, mix="lognormal",
             median=128, sigma=1.5, lo=8, hi=131072, tokens=65536, mix_seed=3),
        # 32 video clips of 1k-8k tokens (Transformer-2D heads).
        dict(name="video_mix", kind="attn", api="batch", bwd=True, heads=16, dim=72, causal=False, mix="uniform", n=32,
             lens="1024,2048,4096,8192", mix_seed=0),
        # Transformer-2D temporal attention: thousands of sequences of 1-51 tokens.
        dict(name="temporal", kind="attn", api="batch", bwd=True, heads=16, dim=72, causal=False, mix="temporal",
             tokens=131072, mix_seed=0),
        # One Transformer-2D layer's training step on a ragged batch of clips,
        # activations kept.
        dict(name="layer_2d", kind="layer", recompute=False, heads=16, dim=72, causal=False, mix="list",
             lens="6400,4096,3600,1620,409,256"),
        # One Transformer-1D layer's training step on a causal pack, recomputing
        # its forward in the backward.
        dict(name="layer_1d", kind="layer", recompute=True, heads=48, dim=64, causal=True, mix="list",
             lens="4001,2048,1500,643"),
    ]


# No drawn case does more matrix work than the largest listed one (the 128k
# shard) or holds more tokens than the largest pack.
_MAX_FLOPS = 14 * 131072 ** 2 * 2 * 128
_MAX_TOKENS = 131072


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges (no name)."""
    while True:
        case = _draw(rng)
        lens = lengths(case)
        if lens and sum(lens) <= _MAX_TOKENS and work(case)["flops"] <= _MAX_FLOPS:
            return case


def _draw(rng):
    what = rng.choice(["shard", "shard", "small", "text", "clips", "temporal", "layer_2d", "layer_1d"])
    seed = rng.randrange(1 << 30)
    dim = rng.choice([64, 72, 128])
    if what == "shard":  # one sequence, a few local heads
        return dict(kind="attn", api=rng.choice(["batch", "call"]), bwd=rng.random() < 0.8,
                    heads=rng.choice([1, 2, 3, 4, 6]), dim=dim, causal=rng.random() < 0.3, mix="list",
                    lens=str(_log_int(rng, 500, 100000)))
    if what == "small":  # a handful of short sequences
        n = rng.randint(1, 6)
        return dict(kind="attn", api="call", bwd=True, heads=rng.choice([2, 4, 7, 16]), dim=dim,
                    causal=rng.random() < 0.5, mix="list", lens=",".join(str(_log_int(rng, 20, 1500)) for _ in range(n)))
    if what == "text":  # causal documents
        return dict(kind="attn", api="batch", bwd=True, heads=rng.choice([8, 32, 48]), dim=rng.choice([64, 128]),
                    causal=True, mix="lognormal", median=_log_int(rng, 128, 4096), sigma=rng.choice([0.7, 1.0, 1.5]),
                    lo=8, hi=131072, tokens=_log_int(rng, 8000, 100000), mix_seed=seed)
    if what == "clips":  # video clips, ragged lengths
        sizes = ",".join(str(_log_int(rng, 256, 9000)) for _ in range(4))
        return dict(kind="attn", api="batch", bwd=True, heads=rng.choice([8, 16]), dim=rng.choice([64, 72]), causal=False,
                    mix="uniform", n=rng.randint(2, 32), lens=sizes, mix_seed=seed)
    if what == "temporal":
        return dict(kind="attn", api="batch", bwd=True, heads=16, dim=rng.choice([64, 72, 128]), causal=False,
                    mix="temporal", tokens=_log_int(rng, 20000, 131072), mix_seed=seed)
    n = rng.randint(1, 6)
    if what == "layer_2d":
        lens = ",".join(str(_log_int(rng, 200, 6000)) for _ in range(n))
        return dict(kind="layer", recompute=rng.random() < 0.5, heads=16, dim=72, causal=False, mix="list", lens=lens)
    lens = ",".join(str(_log_int(rng, 100, 3000)) for _ in range(n))
    return dict(kind="layer", recompute=rng.random() < 0.5, heads=48, dim=64, causal=True, mix="list", lens=lens)


def lengths(case):
    """Sequence lengths of the case's packed batch."""
    mix = case["mix"]
    if mix == "list":
        return [int(x) for x in case["lens"].split(",")]
    rng = np.random.default_rng(case["mix_seed"])
    if mix == "uniform":
        return rng.choice([int(x) for x in case["lens"].split(",")], case["n"]).tolist()
    if mix == "lognormal":
        pool = inputs.text_lengths(rng, 4096, case["median"], case["sigma"], case["lo"], case["hi"])
        pool = pool[pool <= case["tokens"]].tolist()
        return inputs.greedy_pack(pool, case["tokens"])[0]
    if mix == "temporal":
        out = []
        for frames, tokens in inputs.video_clips(rng, case["tokens"]):
            out += [frames] * tokens
        return inputs.greedy_pack(out, case["tokens"])[0]
    raise ValueError(mix)


# ---------------------------------------------------------------------------
# inputs and one pass

def _randn(gen, *shape, scale=1.0):
    return (torch.randn(*shape, generator=gen, device="cuda") * scale).to(torch.bfloat16)


def _attn_tensors(case, seed):
    """q, k, v, dO: bf16 N(0, 1), as projections of normalised activations are."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    shape = (sum(lengths(case)), case["heads"], case["dim"])
    return [_randn(gen, *shape) for _ in range(4)]


def _layer_tensors(case, seed):
    """Weights at 1/sqrt(fan-in), gains near one, unit activations."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    hidden = case["heads"] * case["dim"]
    weights = {}
    for name, shape in dcp.layer_param_shapes(hidden).items():
        if name.startswith("norm"):
            weights[name] = (1.0 + 0.2 * torch.randn(shape, generator=gen, device="cuda")).to(torch.bfloat16)
        else:
            weights[name] = _randn(gen, *shape, scale=1.0 / math.sqrt(shape[0]))
    tokens = sum(lengths(case))
    return weights, _randn(gen, tokens, hidden), _randn(gen, tokens, hidden)


def prepare(case, seed):
    cu = inputs.cu_from_lengths(lengths(case))
    if case["kind"] == "layer":
        weights, x, dout = _layer_tensors(case, seed)
        grads = {n: torch.zeros(w.shape, dtype=torch.float32, device="cuda") for n, w in weights.items()}
        layer = dcp.Layer(weights, grads, cu, case["heads"], case["dim"], case["causal"], None, LAYER_EPS)
        return dict(case=case, layer=layer, x=x, dout=dout, out=torch.empty_like(x), dx=torch.empty_like(x),
                    stash=torch.empty(layer.stash_bytes, dtype=torch.uint8, device="cuda"))
    q, k, v, dout = _attn_tensors(case, seed)
    state = dict(case=case, cu=cu, q=q, k=k, v=v, dout=dout)
    if case["api"] == "batch":
        state["batch"] = dcp.PreparedAttention(q, k, v, dout, cu, None, case["causal"])
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "layer":
        layer = state["layer"]
        torch._foreach_zero_(list(layer.grads.values()))  # a step starts from zero gradients
        out = layer.fwd(state["x"], keep=not case["recompute"], out=state["out"], stash=state["stash"])
        dx = layer.bwd(state["x"], state["dout"], dx=state["dx"])
        return dict(out=out, dx=dx, **{"d_" + n: g for n, g in layer.grads.items()})
    if case["api"] == "batch":
        b = state["batch"]
        b.fwd()
        if not case["bwd"]:
            return dict(o=b.o, lse=b.lse)
        b.bwd()
        return dict(o=b.o, lse=b.lse, dq=b.dq, dk=b.dk, dv=b.dv)
    q, k, v, cu = state["q"], state["k"], state["v"], state["cu"]
    o, lse = dcp.varlen_attn_fwd(q, k, v, cu, None, case["causal"])
    if not case["bwd"]:
        return dict(o=o, lse=lse)
    dq, dk, dv = dcp.varlen_attn_bwd(state["dout"], o, lse, q, k, v, cu, None, case["causal"])
    return dict(o=o, lse=lse, dq=dq, dk=dk, dv=dv)


# ---------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    """Valid (query, key) pairs only: forward 4 and backward 10 flops per pair,
    head and column; each input read once and each output written once."""
    lens = lengths(case)
    heads, dim = case["heads"], case["dim"]
    pairs = sum(s * (s + 1) // 2 if case["causal"] else s * s for s in lens)
    tokens, hidden = sum(lens), heads * dim
    if case["kind"] == "layer":
        passes = 4 if case["recompute"] else 3  # forward, backward (twice a forward), recomputed forward
        flops = passes * 24 * tokens * hidden ** 2 + pairs * hidden * (18 if case["recompute"] else 14)
        params = 12 * hidden ** 2 + 2 * hidden
        return dict(bytes=4 * 2 * tokens * hidden + (2 + 4) * params, flops=flops)
    tensors = 8 if case["bwd"] else 4  # q, k, v, dO, o, dq, dk, dv
    return dict(bytes=tensors * 2 * tokens * hidden + 4 * heads * tokens, flops=pairs * hidden * (14 if case["bwd"] else 4))


def tolerance(case):
    """About four times the error against float64 seen over these ranges (2.6e-3
    for attention, 6.2e-3 for a layer: the roundings of its bf16 intermediates)."""
    return {"rel": 2.5e-2 if case["kind"] == "layer" else 1e-2}


# ---------------------------------------------------------------------------
# float64 reference (plain torch)

_CHUNK = 1 << 27  # score elements held at once


def _blocks(lens):
    """Sequences grouped by length: (length, first rows), so that equal short
    sequences go through one batched product."""
    first = np.concatenate([[0], np.cumsum(lens)])
    groups = {}
    for s, r in zip(lens, first):
        if s:
            groups.setdefault(int(s), []).append(int(r))
    return sorted(groups.items())


def _each(lens, heads):
    """Yields (rows [n, s], head slice): batches of equal sequences whose full
    score matrices fit the chunk, or one (sequence, head) at a time."""
    for s, starts in _blocks(lens):
        fit = max(1, _CHUNK // (s * s * heads))
        hstep = heads if s * s * heads <= _CHUNK else max(1, _CHUNK // (s * s))
        for i in range(0, len(starts), fit):
            rows = torch.tensor(starts[i:i + fit], device="cuda")[:, None] + torch.arange(s, device="cuda")
            for h in range(0, heads, hstep):
                yield rows, slice(h, min(heads, h + hstep))


def _take(t, rows, hs):
    """[n * heads, s, D] float64, contiguous."""
    x = t[rows.reshape(-1), hs].double().reshape(*rows.shape, -1, t.shape[-1])
    return x.permute(0, 2, 1, 3).reshape(-1, rows.shape[1], t.shape[-1]).contiguous()


def _put(out, rows, hs, x):
    n, s = rows.shape
    out[rows.reshape(-1), hs] = x.reshape(n, -1, s, x.shape[-1]).permute(0, 2, 1, 3).reshape(n * s, -1, x.shape[-1])


def _scores(q, k, r0, scale, causal):
    """Scaled scores of query rows r0 .. r0 + len(q) - 1 against every key."""
    s = torch.matmul(q, k.transpose(1, 2).contiguous()).mul_(scale)
    if causal:
        keys = torch.arange(k.shape[1], device=s.device)
        s.masked_fill_(keys[None, :] > (r0 + torch.arange(q.shape[1], device=s.device))[:, None], -math.inf)
    return s


def _exact_attn(q, k, v, lens, scale, causal, dout=None):
    """O, LSE (and dQ, dK, dV of <dout, O>) in float64; q, k, v [T, H, D]."""
    tokens, heads, _ = q.shape
    new = lambda: torch.zeros(q.shape, dtype=torch.float64, device=q.device)
    o, lse = new(), torch.zeros(heads, tokens, dtype=torch.float64, device=q.device)
    grads = [new() for _ in range(3)] if dout is not None else []
    for rows, hs in _each(lens, heads):
        Q, K, V = (_take(t, rows, hs) for t in (q, k, v))
        dO = _take(dout, rows, hs) if grads else None
        O, L = torch.empty_like(Q), torch.empty(Q.shape[:2], dtype=torch.float64, device=q.device)
        if grads:
            dQ, dK, dV = torch.empty_like(Q), torch.zeros_like(K), torch.zeros_like(V)
        step = max(1, min(rows.shape[1], _CHUNK // (Q.shape[0] * rows.shape[1])))
        for r0 in range(0, rows.shape[1], step):
            r = slice(r0, r0 + step)
            S = _scores(Q[:, r].contiguous(), K, r0, scale, causal)
            L[:, r] = torch.logsumexp(S, -1)
            P = S.sub_(L[:, r, None]).exp_()
            O[:, r] = torch.matmul(P, V)
            if grads:
                g = dO[:, r].contiguous()
                dV += torch.matmul(P.transpose(1, 2).contiguous(), g)
                dS = torch.matmul(g, V.transpose(1, 2).contiguous())
                dS.sub_((g * O[:, r]).sum(-1, keepdim=True)).mul_(P).mul_(scale)
                dQ[:, r] = torch.matmul(dS, K)
                dK += torch.matmul(dS.transpose(1, 2).contiguous(), Q[:, r].contiguous())
        _put(o, rows, hs, O)
        n, s = rows.shape
        lse[hs, rows.reshape(-1)] = L.reshape(n, -1, s).permute(1, 0, 2).reshape(-1, n * s)
        if grads:
            for out, x in zip(grads, (dQ, dK, dV)):
                _put(out, rows, hs, x)
    return o, lse, grads


class _Attention(torch.autograd.Function):
    @staticmethod
    def forward(ctx, q, k, v, lens, scale, causal):
        ctx.save_for_backward(q, k, v)
        ctx.args = (lens, scale, causal)
        return _exact_attn(q, k, v, lens, scale, causal)[0]

    @staticmethod
    def backward(ctx, dout):
        return (*_exact_attn(*ctx.saved_tensors, *ctx.args, dout=dout)[2], None, None, None)


def _rmsnorm(x, g):
    return x * g * torch.rsqrt(x.square().mean(-1, keepdim=True) + LAYER_EPS)


def exact(case, seed):
    lens = lengths(case)
    scale = 1.0 / math.sqrt(case["dim"])
    if case["kind"] == "layer":
        weights, x, dout = _layer_tensors(case, seed)
        w = {n: t.double().requires_grad_() for n, t in weights.items()}
        x = x.double().requires_grad_()
        y = _rmsnorm(x, w["norm1"])
        q, k, v = ((y @ w[n]).reshape(-1, case["heads"], case["dim"]) for n in ("wq", "wk", "wv"))
        o = _Attention.apply(q, k, v, lens, scale, case["causal"]).reshape(x.shape)
        h = x + o @ w["wo"]
        u = _rmsnorm(h, w["norm2"]) @ w["w_up"]
        out = h + torch.nn.functional.gelu(u, approximate="tanh") @ w["w_down"]
        out.backward(dout.double())
        return dict(out=out.detach(), dx=x.grad, **{"d_" + n: t.grad for n, t in w.items()})
    q, k, v, dout = _attn_tensors(case, seed)
    o, lse, grads = _exact_attn(q, k, v, lens, scale, case["causal"], dout if case["bwd"] else None)
    return dict(o=o, lse=lse, **dict(zip(("dq", "dk", "dv"), grads)))
