"""Performance cases: the calls a serving program makes, over the sizes this framework is used at.

A case is a dict of plain values: ``op`` (what is called), ``model`` (a shape of MODELS), ``layers``, ``kv_heads``,
``prompt`` (context tokens) and the draft shape.  The models are random-normal decoders whose output embedding holds
one strong successor per token, so that greedy tokens have the margins a trained model gives them and do not hang on the
last bit of a logit; generated text runs through cycles of 16 tokens, so the context matcher finds repeats.

Outputs: a single-token call, a prefill and a generation return logits; a verify call of a wide block returns the final
hidden state of every block token (the whole grid of logits would cost more to copy than the call) beside its integer
results.  The draft builders return token ids, which are exact.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2411_03786_amd as ngg

# n_layers, d_model, n_heads, head_dim, d_ffn, vocab, dtype: the shapes of the benchmark's workloads, and a generic fp32 one
MODELS = {
    "tiny": (2, 128, 4, 32, 512, 512, "f32"),
    "mid32": (4, 512, 8, 64, 1408, 8192, "f32"),
    "small": (12, 768, 12, 64, 3072, 32000, "bf16"),
    "7b": (32, 4096, 32, 128, 14336, 32000, "bf16"),
    "3b": (28, 3072, 24, 128, 8192, 128256, "bf16"),
}
EPS, THETA = 1e-5, 10000.0


def _case(op, model, prompt, k=1, w=0, layers=0, kv_heads=0, **more):
    m = MODELS[model]
    return dict(op=op, model=model, layers=layers or m[0], kv_heads=kv_heads or m[2], prompt=prompt, k=k, w=w, **more)


def listed():
    """The benchmark's five workloads in their parts (draft building, block verification, single-token step, prefill),
    the corner of wide blocks, the allocation-free matcher, and one whole generation."""
    return [
        # the smallest call: two fp32 layers, a block of 13 tokens; launches and latency
        dict(_case("verify", "tiny", 128, 4, 3), name="verify_tiny_f32"),
        # a small model's serving loop: its single-token step and its block of 33 tokens
        dict(_case("decode", "small", 1024), name="decode_small"),
        dict(_case("verify", "small", 1024, 8, 4), name="verify_small"),
        # the headline: 7B shape at a 2K prompt, one token at a time and a block of 51 tokens
        dict(_case("decode", "7b", 2048), name="decode_7b"),
        dict(_case("verify", "7b", 2048, 10, 5), name="verify_7b"),
        # long context (16K cached positions), the block of 97 tokens; eight layers of the same widths
        dict(_case("verify", "7b", 16384, 16, 6, layers=8), name="verify_7b_16k"),
        # a wide block (241 tokens), where the call leaves the memory-bound regime; eight layers
        dict(_case("verify", "7b", 2048, 24, 10, layers=8), name="verify_7b_wide"),
        # large vocabulary: 3B shape, 128256 tokens, a 4K prompt; the block, and the drafts with their vocabulary sweep
        dict(_case("verify", "3b", 4096, 10, 5), name="verify_3b"),
        dict(_case("drafts", "3b", 4096, 10, 5, layers=1, k_ctx=10, q_min=2, q_max=2), name="drafts_3b"),
        # a ragged prompt on the small model, and the 2K prompt on the 7B shape
        dict(_case("prefill", "small", 777), name="prefill_small_ragged"),
        dict(_case("prefill", "7b", 2048, layers=16), name="prefill_7b"),
        # a whole answer: prompt of 1024, 64 tokens in blocks of 33
        dict(_case("generate", "small", 1024, 8, 4, k_ctx=8, q_min=2, q_max=2, n_gen=64), name="generate_small"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    op = rng.choice(("verify", "verify", "verify", "verify", "decode", "decode", "prefill", "prefill", "drafts", "match", "generate"))
    if op == "match":                       # the matcher alone, device tokens in, device rows out
        q_min = rng.randint(1, 2)
        return dict(op="match", prompt=_log(rng, 64, 32768), vocab=rng.choice((512, 32000, 128256)), k=1, w=rng.randint(1, 10),
                    k_ctx=rng.randint(1, 32), q_min=q_min, q_max=rng.randint(q_min, 3))
    model = rng.choice(("tiny", "mid32", "small", "7b", "7b", "3b"))
    wide = model in ("7b", "3b")
    layers = rng.randint(1, 6) if wide else rng.randint(1, MODELS[model][0])
    kv = MODELS[model][2] // rng.choice((1, 1, 4))
    prompt = _log(rng, 33, 4096 if model != "tiny" else 512)
    if op == "decode" or op == "prefill":
        return _case(op, model, prompt, layers=layers, kv_heads=kv)
    w = rng.randint(1, 10)
    k = min(32, max(1, _log(rng, 1, 288) // w))
    if op == "verify":
        return _case(op, model, prompt, k, w, layers=layers, kv_heads=kv)
    q_min = rng.randint(1, 2)
    more = dict(k_ctx=rng.randint(1, k), q_min=q_min, q_max=rng.randint(q_min, 3))
    if op == "drafts":
        return _case(op, model, prompt, k, w, layers=1, kv_heads=kv, **more)
    return _case(op, model, min(prompt, 1500), min(k, 12), min(w, 6), layers=min(layers, 4), kv_heads=kv,
                 **dict(more, k_ctx=min(more["k_ctx"], min(k, 12))), n_gen=rng.randint(8, 48))


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _desc(case):
    _, d, H, hd, f, V, dt = MODELS[case["model"]]
    return dict(n_layers=case["layers"], d_model=d, n_heads=H, n_kv_heads=case["kv_heads"], head_dim=hd, d_ffn=f, vocab=V,
                dtype=dt, rms_eps=EPS, rope_theta=THETA)


def _succ(x):
    """The token a model of these cases predicts after x: cycles of 16."""
    return (x // 16) * 16 + (x + 1) % 16


def _weights(m, seed):
    """Device weights in the storage type, from the seed alone."""
    dt = torch.bfloat16 if m["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * (seed % (1 << 30)) + 17)
    mat = lambda *shape: torch.randn(shape, generator=gen, device="cuda", dtype=dt).mul_(0.02)
    gain = lambda n: (1.0 + 0.1 * torch.randn(n, generator=gen, device="cuda")).to(dt)
    d, f, V = m["d_model"], m["d_ffn"], m["vocab"]
    dq, dkv = m["n_heads"] * m["head_dim"], m["n_kv_heads"] * m["head_dim"]
    # embeddings as large as the sum of what the layers add, so that the successor's logit stands out
    emb = torch.randn(V, d, generator=gen, device="cuda", dtype=dt)
    emb.mul_(0.5 * math.sqrt(m["n_layers"] * max(1.0, (0.02 * 0.02 * d * math.sqrt(f) * 0.02) ** 2)))
    unemb = torch.empty(V, d, device="cuda", dtype=dt)
    ids = torch.arange(V, device="cuda")
    unemb[_succ(ids)] = (emb.float() / emb.float().square().mean().sqrt() * 0.03).to(dt)
    unemb += mat(V, d)
    w = dict(tok_emb=emb, unemb=unemb, final_norm=gain(d), layers=[])
    for _ in range(m["n_layers"]):
        w["layers"].append(dict(attn_norm=gain(d), wq=mat(dq, d), wk=mat(dkv, d), wv=mat(dkv, d), wo=mat(d, dq), mlp_norm=gain(d),
                                w_gate=mat(f, d), w_up=mat(f, d), w_down=mat(d, f)))
    return w


def _prompt(V, n, seed):
    """A Zipf stream in which about 30 % of the tokens belong to spans copied from earlier ones."""
    rng = np.random.default_rng([seed % (1 << 30), 0x52])
    p = 1.0 / np.arange(1, V + 1) ** 1.1
    cdf = np.cumsum(p) / p.sum()
    x = np.minimum(np.searchsorted(cdf, rng.random(n)), V - 1).astype(np.int32)
    i = 16
    while i < n:
        if rng.random() < 0.041:
            ln, src = int(rng.integers(4, 17)), int(rng.integers(0, i))
            for t in range(min(ln, n - i)):
                x[i + t] = x[src + t]
            i += ln
        else:
            i += 1
    return x


def _drafts(case, prompt, V, seed):
    """k rows of w tokens: the likely continuation, cut off by another token at a place of its own in every row."""
    rng = np.random.default_rng([seed % (1 << 30), 0x53])
    k, w = case["k"], case["w"]
    out = np.zeros((k, w), dtype=np.int32)
    for r in range(k):
        t = _succ(int(prompt[-1]))
        cut = int(rng.integers(0, w + 1))
        for j in range(w):
            t = _succ(t) if j != cut else int(rng.integers(0, V))
            out[r, j] = t
    return out


def _cfg(case):
    return dict(k=case["k"], w=case["w"], k_ctx_max=case["k_ctx"], q_min=case["q_min"], q_max=case["q_max"])


def prepare(case, seed):
    op = case["op"]
    if op == "match":
        tokens = torch.from_numpy(_prompt(case["vocab"], case["prompt"], seed)).cuda()
        return dict(case=case, tokens=tokens, rows=torch.full((case["k_ctx"], case["w"]), -1, dtype=torch.int32, device="cuda"),
                    n_rows=torch.zeros(1, dtype=torch.int32, device="cuda"))
    m = _desc(case)
    prompt = _prompt(m["vocab"], case["prompt"], seed)
    room = case.get("n_gen", 0) + case["w"] + 16
    ctx = ngg.Context(m, _weights(m, seed), max_seq=len(prompt) + room, max_k=case["k"], max_w=max(1, case["w"]))
    s = dict(case=case, ctx=ctx, prompt=prompt, d=m["d_model"])
    if op in ("decode", "verify", "drafts"):
        ctx.prefill(prompt)
    if op == "verify":
        s["drafts"] = _drafts(case, prompt, m["vocab"], seed)
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "match":
        ngg.context_drafts_static(s["tokens"], case["w"], case["k_ctx"], case["q_min"], case["q_max"], s["rows"], s["n_rows"])
        return dict(rows=s["rows"], n_rows=s["n_rows"])
    ctx = s["ctx"]
    if op == "drafts":
        drafts, src, n_ctx = ctx.build_drafts(_cfg(case))
        return dict(drafts=drafts, row_src=src, n_ctx=n_ctx)
    if op == "verify":
        r = ctx.verify_step(s["drafts"])
        hidden, _ = ctx.debug_peek("h", np.float32, (1 + case["k"] * case["w"]) * s["d"])
        new = np.full(case["w"] + 1, -1, dtype=np.int32)
        new[:r["n_new"]] = r["new_tokens"]
        return dict(hidden=hidden, greedy=r["greedy"], accept_len=r["accept_len"], new_tokens=new, winner=r["winner"])
    out = {}
    if op == "prefill":
        ctx.prefill(s["prompt"])
    elif op == "generate":
        out["tokens"], stats = ctx.greedy_decode(s["prompt"], case["n_gen"], _cfg(case))
        out["calls"] = stats["calls"]
    r = ctx.verify_step(None, 1, 0, want_logits=True)
    out.update(logits=r["logits"], greedy=r["greedy"])
    return out


# ---- what a pass cannot do without ------------------------------------------------------------------------------------

def _model_call(m, tokens, cached, unembed_rows):
    """(bytes, flops) of one model call on `tokens` positions over `cached` ones."""
    e = 2 if m["dtype"] == "bf16" else 4
    d, f, V, L = m["d_model"], m["d_ffn"], m["vocab"], m["n_layers"]
    dq, dkv = m["n_heads"] * m["head_dim"], m["n_kv_heads"] * m["head_dim"]
    params = L * (2 * d * dq + 2 * d * dkv + 3 * d * f)
    byts = (params + (V * d if unembed_rows else 0)) * e + 2 * L * (cached + tokens) * dkv * e
    pairs = tokens * cached + tokens * (tokens + 1) / 2
    return byts, 2.0 * params * tokens + 4.0 * L * dq * pairs + 2.0 * V * d * unembed_rows


def work(case):
    op, P = case["op"], case["prompt"]
    if op == "match":
        return dict(bytes=4.0 * P + 4.0 * case["k_ctx"] * case["w"], flops=0.0)
    m = _desc(case)
    e = 2 if m["dtype"] == "bf16" else 4
    V, d, k, w = m["vocab"], m["d_model"], case["k"], case["w"]
    if op == "drafts":
        return dict(bytes=float(V * d * e + 4 * P + 4 * k * w), flops=2.0 * V * d)
    if op == "verify":
        M = 1 + k * w
        b, f = _model_call(dict(m), M, P, M)
        pairs = M * P + k * w * (w + 1) / 2 + M                         # a row sees the context, the shared token and itself
        f += 4.0 * m["n_layers"] * m["n_heads"] * m["head_dim"] * (pairs - (M * P + M * (M + 1) / 2))
        return dict(bytes=b + 4.0 * M * d, flops=f)
    b, f = _model_call(m, 1, P, 1)                                      # the call whose logits are returned
    if op == "prefill":
        b2, f2 = _model_call(m, P, 0, 1)
        b, f = b + b2, f + f2
    elif op == "generate":
        b2, f2 = _model_call(m, P, 0, 1)
        calls = math.ceil((case["n_gen"] - 1) / (w + 1))
        b3, f3 = _model_call(m, 1 + k * w, P, 1 + k * w)
        b, f = b + b2 + calls * (b3 + V * d * e), f + f2 + calls * (f3 + 2.0 * V * d)
    return dict(bytes=float(b + 4 * V), flops=float(f))


def tolerance(case):
    if case["op"] in ("drafts", "match"):
        return "exact"
    # about four times the distance from 64 bits that was measured: up to 3.5e-7 in fp32, 4e-4 to 5e-4 with fp16 operands (1 to 32 layers)
    return {"rel": 1.5e-6 if MODELS[case["model"]][6] == "f32" else 2e-3}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------------

def _norm(x, g):
    return x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * g


def _rope(x, pos, hd):
    half = hd // 2
    inv = THETA ** (-torch.arange(half, dtype=torch.float64, device=x.device) * 2.0 / hd)
    ang = pos.double()[:, None] * inv[None, :]
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _forward(m, w, tokens, pos, visible, past, keep):
    """Hidden states [T, d] of `tokens` at `pos`, over `past` (a list of (K, V) per layer, [Hkv, P, hd]); visible: [T, T] mask of
    the tokens' own keys, or None for causal.  keep: return the tokens' keys and values too."""
    H, Hkv, hd = m["n_heads"], m["n_kv_heads"], m["head_dim"]
    T, dev = len(tokens), "cuda"
    h = w["tok_emb"][tokens].double()
    kept = []
    for li, lw in enumerate(w["layers"]):
        lw = {n: t.double() for n, t in lw.items()}
        x = _norm(h, lw["attn_norm"])
        q = _rope((x @ lw["wq"].T).view(T, H, hd), pos, hd).transpose(0, 1)
        k = _rope((x @ lw["wk"].T).view(T, Hkv, hd), pos, hd).transpose(0, 1)
        v = (x @ lw["wv"].T).view(T, Hkv, hd).transpose(0, 1)
        if keep:
            kept.append((k.contiguous(), v.contiguous()))
        P = 0
        if past is not None:
            P = past[li][0].shape[1]
            k, v = torch.cat([past[li][0], k], 1), torch.cat([past[li][1], v], 1)
        out = torch.empty(T, H, hd, dtype=torch.float64, device=dev)
        step = max(16, min(1024, (1 << 28) // (k.shape[1] * (H // Hkv))))
        own = torch.arange(T, device=dev)
        for hk in range(Hkv):
            kt = k[hk].T.contiguous()
            for t0 in range(0, T, step):
                t1 = min(T, t0 + step)
                last = P + (t1 if visible is None else T)               # later keys are invisible to this piece
                qq = q[hk * (H // Hkv):(hk + 1) * (H // Hkv), t0:t1].reshape(-1, hd)
                s = (qq @ kt[:, :last] / math.sqrt(hd)).view(H // Hkv, t1 - t0, last)
                see = (own[None, :last - P] <= own[t0:t1, None]) if visible is None else visible[t0:t1]
                s[:, :, P:].masked_fill_(~see[None], -math.inf)
                p = torch.softmax(s, -1).view(-1, last)
                out[t0:t1, hk * (H // Hkv):(hk + 1) * (H // Hkv)] = (p @ v[hk, :last]).view(H // Hkv, t1 - t0, hd).transpose(0, 1)
        h = h + out.reshape(T, H * hd) @ lw["wo"].T
        x = _norm(h, lw["mlp_norm"])
        g = x @ lw["w_gate"].T
        h = h + (g * torch.sigmoid(g) * (x @ lw["w_up"].T)) @ lw["w_down"].T
    return h, kept


def _logits(w, h):
    return _norm(h, w["final_norm"].double()) @ w["unemb"].double().T


def exact(case, seed):
    op = case["op"]
    if op in ("match", "drafts"):
        return None
    m = _desc(case)
    w = _weights(m, seed)
    prompt = _prompt(m["vocab"], case["prompt"], seed)
    seq = torch.from_numpy(prompt.astype(np.int64)).cuda()
    if op == "generate":                    # the likely text, checked by the model itself
        more = [_succ(int(prompt[-1]))]
        while len(more) < case["n_gen"] - 1:
            more.append(_succ(more[-1]))
        seq = torch.cat([seq, torch.tensor(more, device="cuda")])
    P = len(seq)
    h, past = _forward(m, w, seq, torch.arange(P, device="cuda"), None, None, True)
    last = int(_logits(w, h[-1:]).argmax())                             # the last token, not cached yet
    if op == "generate":
        said = _logits(w, h[len(prompt) - 1:-1]).argmax(-1)
        if not torch.equal(said, seq[len(prompt):]):
            return None
    if op == "verify":
        k, c = case["k"], case["w"]
        block = torch.cat([torch.tensor([last]), torch.from_numpy(_drafts(case, prompt, m["vocab"], seed)).reshape(-1).long()]).cuda()
        at = torch.arange(k * c, device="cuda")
        row, col = at // c, at % c
        see = torch.zeros(1 + k * c, 1 + k * c, dtype=torch.bool, device="cuda")
        see[:, 0] = True
        see[1:, 1:] = (row[:, None] == row[None]) & (col[None] <= col[:, None])
        pos = torch.cat([torch.zeros(1, dtype=torch.long, device="cuda"), 1 + col]) + P
        h, _ = _forward(m, w, block, pos, see, past, False)
        return dict(hidden=h.reshape(-1).cpu().numpy(), greedy=None, accept_len=None, new_tokens=None, winner=None)
    h, _ = _forward(m, w, torch.tensor([last], device="cuda"), torch.tensor([P], device="cuda"),
                    torch.ones(1, 1, dtype=torch.bool, device="cuda"), past, False)
    out = dict(logits=_logits(w, h).view(1, 1, -1).cpu().numpy(), greedy=None)
    if op == "generate":
        out.update(tokens=None, calls=None)
    return out
