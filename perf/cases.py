"""Timed workloads of the decoder-layer forward.

A case is one forward step of a batch through a layer (or a small stack of layers), called the way
a serving loop calls it: a handle on resident weights, a paged KV cache, a workspace, a schedule,
and `DynLayer.forward` on the program's one compute stream.  Decode steps repeat with the same batch
structure and replay a captured graph; steps with a prompt in them change shape from one to the
next and are issued eagerly.
"""
from __future__ import annotations

import functools
import math
import random

import numpy as np
import torch

from paper_2605_21603_amd import binding as B
from paper_2605_21603_amd import placement

EPS, ROPE_BASE = 1e-6, 10000.0

# Layer shapes.  "8b" is the full-size dense layer of the benchmark and "moe" its eight-expert form;
# "hd64" is a smaller layer with 64-wide heads, "f32" a layer kept in 32 bits throughout and "tiny"
# the benchmark's smallest configuration.
SHAPES = {
    "8b": dict(dtype="bf16", hidden=4096, n_q=32, n_kv=8, head_dim=128, inter=14336, n_experts=0, top_k=0),
    "moe": dict(dtype="bf16", hidden=4096, n_q=32, n_kv=8, head_dim=128, inter=14336, n_experts=8, top_k=2),
    "hd64": dict(dtype="bf16", hidden=2048, n_q=32, n_kv=8, head_dim=64, inter=8192, n_experts=0, top_k=0),
    "f32": dict(dtype="f32", hidden=1024, n_q=16, n_kv=4, head_dim=64, inter=4096, n_experts=0, top_k=0),
    "tiny": dict(dtype="f32", hidden=256, n_q=4, n_kv=4, head_dim=64, inter=1024, n_experts=0, top_k=0),
}


def _case(shape, *, prompt=0, cached=0, n_decode=0, ctx_lo=1, ctx_hi=1, layers=1, page=16, schedule="sequential", graph=False, name=None):
    """prompt tokens of one sequence behind `cached` positions, and n_decode single-token sequences
    with contexts spread over ctx_lo..ctx_hi (the step's own token included)."""
    c = dict(shape=shape, prompt=prompt, cached=cached, n_decode=n_decode, ctx_lo=ctx_lo, ctx_hi=ctx_hi, layers=layers, page=page,
             schedule=schedule, graph=graph)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest benchmark configuration: 32-bit, four tokens; what a step costs when nothing in it is large
        _case("tiny", n_decode=4, ctx_lo=128, ctx_hi=128, graph=True, name="tiny_f32_decode_4"),
        # a 32-bit layer as one runs it to check a model: a prompt of a few hundred tokens beside decodes
        _case("f32", prompt=201, n_decode=24, ctx_lo=17, ctx_hi=900, name="f32_prompt_201_decode_24"),
        # one user's chat: a single sequence, the weights are all there is to read
        _case("8b", n_decode=1, ctx_lo=2900, ctx_hi=2900, graph=True, name="decode_1"),
        # a lightly loaded server, cache pages of 32 positions
        _case("8b", n_decode=13, ctx_lo=200, ctx_hi=3000, page=32, graph=True, name="decode_13_pages_32"),
        # the benchmark's decode batch
        _case("8b", n_decode=128, ctx_lo=512, ctx_hi=4096, graph=True, name="decode_128"),
        # the benchmark's many-layer decode step, three of its layers: where a loaded server spends its time
        _case("8b", n_decode=256, ctx_lo=1024, ctx_hi=8192, layers=3, graph=True, name="decode_256_3_layers"),
        # a short prompt joins running decodes; the built-in policy chooses the schedule (two micro-batches side by side here)
        _case("8b", prompt=512, n_decode=64, ctx_lo=2048, ctx_hi=2048, schedule="policy", name="prompt_512_decode_64_policy"),
        # the benchmark's mixed step
        _case("8b", prompt=2048, n_decode=64, ctx_lo=2048, ctx_hi=2048, name="prompt_2048_decode_64"),
        # a long document is read in pieces: a 4096-token piece behind 8192 cached positions
        _case("8b", prompt=4096, cached=8192, name="prompt_4096_after_8192"),
        # the benchmark's mixture-of-experts decode batch
        _case("moe", n_decode=256, ctx_lo=1024, ctx_hi=1024, graph=True, name="moe_decode_256"),
        # a prompt through the mixture of experts, beside a few decodes
        _case("moe", prompt=1100, n_decode=20, ctx_lo=100, ctx_hi=2000, name="moe_prompt_1100_decode_20"),
        # 64-wide heads: a small model's mixed step
        _case("hd64", prompt=300, n_decode=40, ctx_lo=64, ctx_hi=2048, name="hd64_prompt_300_decode_40"),
    ]


def _spread(rng, lo, hi):
    """An integer of lo..hi, uniform over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    kind = rng.choice(["decode", "decode", "prompt", "prompt", "mixed", "moe_decode", "moe_mixed", "hd64", "f32", "tiny"])
    lo = _spread(rng, 16, 2048)
    hi = _spread(rng, lo, 4096)
    if kind == "decode":
        page = rng.choice([16, 16, 32])
        n = _spread(rng, 1, 300 if page == 16 else 16)
        return _case("8b", n_decode=n, ctx_lo=lo, ctx_hi=hi, layers=rng.choice([1, 1, 2]), page=page, graph=True)
    if kind == "prompt":
        return _case("8b", prompt=_spread(rng, 33, 4096), cached=rng.choice([0, 0, _spread(rng, 16, 8192)]))
    if kind == "mixed":
        return _case("8b", prompt=_spread(rng, 33, 2500), n_decode=_spread(rng, 1, 128), ctx_lo=lo, ctx_hi=hi,
                     schedule=rng.choice(["sequential", "policy"]))
    if kind == "moe_decode":
        return _case("moe", n_decode=_spread(rng, 1, 300), ctx_lo=lo, ctx_hi=hi, graph=True)
    if kind == "moe_mixed":
        return _case("moe", prompt=_spread(rng, 33, 1500), n_decode=_spread(rng, 1, 64), ctx_lo=lo, ctx_hi=hi)
    if kind == "hd64":
        return _case("hd64", prompt=rng.choice([0, _spread(rng, 2, 400)]), n_decode=_spread(rng, 1, 64), ctx_lo=min(lo, 512), ctx_hi=min(hi, 2048))
    if kind == "f32":
        return _case("f32", prompt=rng.choice([0, _spread(rng, 2, 300)]), n_decode=_spread(rng, 1, 48), ctx_lo=min(lo, 256), ctx_hi=min(hi, 1024))
    return _case("tiny", n_decode=_spread(rng, 1, 32), ctx_lo=min(lo, 128), ctx_hi=min(hi, 512), graph=True)


# ---------------------------------------------------------------------------------- inputs

@functools.lru_cache(maxsize=None)
def _stream():
    """The program's compute stream (graph replays need one that is not the null stream)."""
    return torch.cuda.Stream()


def _seqs(c):
    """(new tokens, context) of every sequence; decode contexts cover ctx_lo..ctx_hi evenly, in no order."""
    out = [(c["prompt"], c["cached"] + c["prompt"])] if c["prompt"] else []
    span = c["ctx_hi"] - c["ctx_lo"] + 1
    out += [(1, c["ctx_lo"] + int(span * ((i * 0.6180339887498949 + 0.5) % 1.0))) for i in range(c["n_decode"])]
    return out


def _inputs(c, seed, device="cuda:0"):
    """Weights, caches, activations and the batch's index arrays of one step."""
    sh = SHAPES[c["shape"]]
    dt = torch.float32 if sh["dtype"] == "f32" else torch.bfloat16
    H, I, E, d = sh["hidden"], sh["inter"], sh["n_experts"], sh["head_dim"]
    n_q, n_kv, L, ps = sh["n_q"], sh["n_kv"], c["layers"], c["page"]
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)

    def normal(shape, std, dtype=dt):
        return torch.randn(shape, generator=gen, device=device, dtype=dtype).mul_(std)

    def gains():
        return (1.0 + 0.1 * torch.randn(H, generator=gen, device=device)).to(dt)

    weights = []
    for _ in range(L):
        w = dict(w_qkv=normal(((n_q + 2 * n_kv) * d, H), 0.02), w_o=normal((H, n_q * d), 0.02), g_norm1=gains(), g_norm2=gains())
        if E:
            w.update(w_gate_up=normal((E, 2 * I, H), 0.02), w_down=normal((E, H, I), 0.02), w_router=normal((E, H), H ** -0.5, torch.float32))
        else:
            w.update(w_gate_up=normal((2 * I, H), 0.02), w_down=normal((H, I), 0.02))
        weights.append(w)

    seqs = _seqs(c)
    T = sum(q for q, _ in seqs)
    x = torch.randn((T, H), generator=gen, device=device)
    if E:
        # a trained router is sure of its choice and does not use all experts alike: every token
        # leans towards two experts, the popular ones more often
        popularity = 1.0 / torch.arange(1, E + 1, device=device, dtype=torch.float32).sqrt()
        pick = torch.multinomial(popularity.expand(T, E), 2, generator=gen)
        x += 6.0 * weights[0]["w_router"][pick[:, 0]] + 4.0 * weights[0]["w_router"][pick[:, 1]]
    pages = [(ctx + ps - 1) // ps for _, ctx in seqs]
    n_pages = sum(pages)
    perm = np.random.RandomState(seed % (1 << 31)).permutation(n_pages).astype(np.int32)
    table = np.zeros((len(seqs), max(pages)), dtype=np.int32)
    at = np.concatenate([[0], np.cumsum(pages)])
    for s, n in enumerate(pages):
        table[s, :n] = perm[at[s]:at[s] + n]
    q_len = np.array([q for q, _ in seqs], dtype=np.int32)
    ctx_len = np.array([ctx for _, ctx in seqs], dtype=np.int32)
    return dict(
        weights=weights, x=x.to(dt),
        k_cache=normal((L, n_pages, n_kv, ps, d), 1.0), v_cache=normal((L, n_pages, n_kv, d, ps), 1.0), block_table=table,
        seq_of_token=np.repeat(np.arange(len(seqs), dtype=np.int32), q_len),
        pos_of_token=np.concatenate([np.arange(ctx - q, ctx, dtype=np.int32) for q, ctx in seqs]),
        q_start=np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32), q_len=q_len, ctx_len=ctx_len)


def _config(c, data):
    sh = SHAPES[c["shape"]]
    chunk = placement.rule_chunk(data["ctx_len"].tolist(), data["q_len"].tolist(), sh["n_kv"])
    return B.dyn_layer_config(B.DYN_F32 if sh["dtype"] == "f32" else B.DYN_BF16, c["layers"], sh["hidden"], sh["n_q"], sh["n_kv"],
                              sh["head_dim"], sh["inter"], sh["n_experts"], sh["top_k"], EPS, ROPE_BASE, c["page"], chunk)


def prepare(c, seed):
    """A handle on the weights, the batch with its caches and workspace in device memory, and the schedule."""
    data = _inputs(c, seed)
    cfg = _config(c, data)
    layer = B.DynLayer(cfg, data["weights"])
    step = B.DeviceStep(layer, data)
    if c["schedule"] == "policy":
        sched, _ = B.Scheduler(cfg, data["q_start"]).auto(data["ctx_len"], use_graph=c["graph"])
    else:
        sched = B.sequential(use_graph=c["graph"])
    layer.prepare(sched)
    return dict(layer=layer, step=step, sched=sched, stream=_stream())


def run(state):
    """One forward: the layer's output, and the caches with this step's keys and values appended."""
    step = state["step"]
    state["layer"].forward(step.batch, state["sched"], state["stream"])
    return dict(y=step.y, k_cache=step.k_cache, v_cache=step.v_cache)


# ---------------------------------------------------------------------------------- what a pass needs, and what it should give

def work(c):
    sh = SHAPES[c["shape"]]
    e = 4 if sh["dtype"] == "f32" else 2
    H, I, E, d, n_q, n_kv = sh["hidden"], sh["inter"], sh["n_experts"], sh["head_dim"], sh["n_q"], sh["n_kv"]
    seqs = _seqs(c)
    T = sum(q for q, _ in seqs)
    attn_w = (n_q + 2 * n_kv) * d * H + H * n_q * d
    mlp_w = 3 * I * H
    weight_bytes = (attn_w + mlp_w * (min(E, T * sh["top_k"]) if E else 1)) * e + 2 * H * e + E * H * 4
    kv_bytes = sum(ctx for _, ctx in seqs) * 2 * n_kv * d * e         # read by the attention, this step's positions among them
    kv_written = T * 2 * n_kv * d * e
    keys = sum(q * (ctx - q) + q * (q + 1) // 2 for q, ctx in seqs)   # (query, key) pairs under the causal mask
    flops = 2 * T * (attn_w + mlp_w * (sh["top_k"] if E else 1) + E * H) + 4 * n_q * d * keys
    return {"bytes": c["layers"] * (weight_bytes + kv_bytes + kv_written) + 2 * T * H * e, "flops": c["layers"] * flops}


def tolerance(c):
    """About four times the error against exact(): 4.3e-7 in 32 bits; in bf16 3.6e-3 to 5.7e-3 for
    one layer (the rounding of a row that is large next to what the layer adds sets it), 7.4e-3
    behind three."""
    if SHAPES[c["shape"]]["dtype"] == "f32":
        return {"rel": 2e-6}
    return {"rel": 2e-2 if c["layers"] == 1 else 3e-2}


def exact(c, seed):
    """The step in 64 bits from the definition of the layer: RMSNorm, rotary (i, i + d/2) pairs, causal
    attention over the paged cache, gated MLP or weighted experts, residuals."""
    sh = SHAPES[c["shape"]]
    data = _inputs(c, seed)
    f = torch.float64
    E, d, n_q, n_kv, I, ps = sh["n_experts"], sh["head_dim"], sh["n_q"], sh["n_kv"], sh["inter"], c["page"]
    G, dev = n_q // n_kv, data["x"].device
    x = data["x"].to(f)
    T = x.shape[0]
    pos = torch.from_numpy(data["pos_of_token"]).to(dev).long()
    seq = torch.from_numpy(data["seq_of_token"]).to(dev).long()
    table = torch.from_numpy(data["block_table"]).to(dev).long()
    angle = pos.to(f)[:, None] * ROPE_BASE ** (-torch.arange(0, d, 2, device=dev, dtype=f) / d)
    cos, sin = angle.cos()[:, None], angle.sin()[:, None]
    page, slot = table[seq, pos // ps], pos % ps
    k_all, v_all = [], []

    def rotate(t):
        a, b = t[..., : d // 2], t[..., d // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    def norm(t, g):
        return t * g.to(f) / torch.sqrt((t * t).mean(-1, keepdim=True) + EPS)

    def mlp(h, gate_up, down):
        gu = h @ gate_up.to(f).t()
        return (torch.nn.functional.silu(gu[:, :I]) * gu[:, I:]) @ down.to(f).t()

    for layer, w in enumerate(data["weights"]):
        qkv = (norm(x, w["g_norm1"]) @ w["w_qkv"].to(f).t()).view(T, n_q + 2 * n_kv, d)
        q = rotate(qkv[:, :n_q])
        k_cache, v_cache = data["k_cache"][layer].to(f), data["v_cache"][layer].to(f)
        k_cache[page, :, slot] = rotate(qkv[:, n_q:n_q + n_kv])
        v_cache[page, :, :, slot] = qkv[:, n_q + n_kv:]
        out = torch.empty_like(q)
        row = 0
        for s, (n, ctx) in enumerate(_seqs(c)):
            pg = table[s, : (ctx + ps - 1) // ps]
            K = k_cache[pg].permute(1, 0, 2, 3).reshape(n_kv, -1, d)[:, :ctx]
            V = v_cache[pg].permute(1, 0, 3, 2).reshape(n_kv, -1, d)[:, :ctx]
            for r0 in range(row, row + n, 512):
                r1 = min(r0 + 512, row + n)
                qb = q[r0:r1].view(r1 - r0, n_kv, G, d).permute(1, 0, 2, 3).reshape(n_kv, -1, d)
                score = (qb @ K.transpose(1, 2)).view(n_kv, r1 - r0, G, ctx) / math.sqrt(d)
                ahead = torch.arange(ctx, device=dev)[None, :] > pos[r0:r1, None]
                p = score.masked_fill_(ahead[None, :, None], -math.inf).softmax(-1)
                out[r0:r1] = (p.view(n_kv, -1, ctx) @ V).view(n_kv, r1 - r0, G, d).permute(1, 0, 2, 3).reshape(r1 - r0, n_q, d)
                del score, p
            row += n
        x2 = x + out.view(T, n_q * d) @ w["w_o"].to(f).t()
        h = norm(x2, w["g_norm2"])
        if E:
            logits, choice = (h @ w["w_router"].to(f).t()).topk(sh["top_k"], -1)
            share = logits.softmax(-1)
            x = x2.clone()
            for e in range(E):
                t, j = (choice == e).nonzero(as_tuple=True)
                if len(t):
                    x.index_add_(0, t, share[t, j, None] * mlp(h[t], w["w_gate_up"][e], w["w_down"][e]))
        else:
            x = x2 + mlp(h, w["w_gate_up"], w["w_down"])
        k_all.append(k_cache)
        v_all.append(v_cache)
    return dict(y=x, k_cache=torch.stack(k_all), v_cache=torch.stack(v_all))
