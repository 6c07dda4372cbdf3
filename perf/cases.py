"""The workloads this repository is measured on, one dict of plain values per case.

A case has a "kind":
  step       one verify pass (chain or draft tree) of a decoder over B sequences x (k+1) rows: the public
             sssd_verify_step / sssd_verify_step_tree.  "layers" layers of a model shape, so that a few-layer
             case is the decoder layer as a serving step runs it; outputs are the logits and the residual stream
             after the last layer (sssd_debug_outputs).  The tokens a step returns are the arg-max of those logits.
  attention  sssd_op_attention: the new rows' attention over the cached context of one layer.
  sample     sssd_op_sample_wide: one token per row of logits (temperature, top-k, top-p).
  kv_move    a prefilled prompt's K/V into the cache of every layer and out again (sssd_kv_import / export),
             what admitting a sequence and saving a prefix do.

Inputs come from the seed alone; `exact` restates every kind with plain torch in 64 bits.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import torch

from paper_2411_05894_amd import binding as sv

DEV = "cuda:0"

SHAPES = {
    "tiny": dict(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=688, rope_base=10000.0),
    "8b": dict(hidden=4096, n_q_heads=32, n_kv_heads=8, head_dim=128, ffn=14336, rope_base=500000.0),
    "70b": dict(hidden=8192, n_q_heads=64, n_kv_heads=8, head_dim=128, ffn=28672, rope_base=500000.0),
}
EPS = 1e-5


def _step(name, shape, layers, vocab, B, k, ctx, ctx_max=0, tree=False, room=0):
    """room: cache rows per sequence beyond the longest context and the new rows (a server reserves for growth)."""
    c = dict(kind="step", shape=shape, layers=layers, vocab=vocab, B=B, k=k, ctx=ctx, ctx_max=ctx_max or ctx, tree=tree, room=room)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest model of the test configurations: launches and latency, nothing else
        _step("tiny_b1_k4", "tiny", 2, 1024, 1, 4, 128),
        # the headline: one user's chat on the whole 8B-shaped model, eight drafts
        _step("8b_whole_b1_k8", "8b", 32, 128256, 1, 8, 2048),
        # plain decoding (no drafts) of a batch on the 70B shape: one layer, 16 rows
        _step("70b_layer_b16_k0", "70b", 1, 1024, 16, 0, 2048),
        # the same batch with eight drafts each, in a cache that has room for 8192 positions a sequence: 144 rows
        _step("70b_layer_b16_k8", "70b", 1, 1024, 16, 8, 2048, room=6135),
        # long context, few sequences: attention over 32768 cached positions and 36-row matrices
        _step("8b_layers_b4_k8_long", "8b", 2, 1024, 4, 8, 32768),
        # a serving batch of ragged sequences: 160 rows
        _step("8b_layers_b32_k4_ragged", "8b", 2, 1024, 32, 4, 1024, 4096),
        # prompts prefilled through the verify step in chunks of 32 tokens, room for 4096 positions: 512 rows
        _step("8b_layers_prefill_b16_k31", "8b", 2, 1024, 16, 31, 479, room=3585),
        # draft trees of 13 nodes on seven sequences with the real vocabulary: 91 rows, LM head and arg-max
        _step("8b_layer_head_tree_b7_k12", "8b", 1, 128256, 7, 12, 700, 1500, True),
        # attention alone, an odd context, a wide tree of drafts (five row tiles)
        dict(name="attn_8b_b2_k17", kind="attention", shape="8b", B=2, k=17, ctx=12345, ctx_max=12345),
        # sampling the k+1 rows of one sequence: T 0.6, top-p 0.95
        dict(name="sample_rows9", kind="sample", rows=9, vocab=128256, temperature=0.6, top_k=0, top_p=0.95),
        # sampling a whole serving batch: T 0.7, top-k 20, top-p 0.8
        dict(name="sample_rows160", kind="sample", rows=160, vocab=128256, temperature=0.7, top_k=20, top_p=0.8),
        # admitting a prompt of 4001 tokens into eight layers and saving it again
        dict(name="kv_move_4001", kind="kv_move", shape="8b", layers=8, t0=0, rows=4001),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["attention"] + ["sample"] * 2 + ["kv_move"])
    if kind == "sample":
        top_k, top_p = rng.choice([(0, 0.95), (20, 0.8), (50, 1.0), (0, 1.0), (0, 0.9)])
        return dict(kind=kind, rows=_log(rng, 1, 192), vocab=_log(rng, 1000, 131072), temperature=rng.choice([0.6, 0.7, 1.0]),
                    top_k=top_k, top_p=top_p)
    if kind == "kv_move":
        return dict(kind=kind, shape=rng.choice(["tiny", "8b", "70b"]), layers=rng.choice([1, 2, 4, 8]), t0=_log(rng, 1, 64) - 1,
                    rows=_log(rng, 9, 8192))
    shape = rng.choice(["tiny", "8b", "8b", "70b"])
    B = _log(rng, 1, 48)
    k = rng.randint(0, 31)
    while B * (k + 1) > 512:
        k = rng.randint(0, k)
    ctx = _log(rng, 33, max(64, min(32768, 131072 // B)))
    lo = rng.choice([ctx, max(17, ctx // 3)])
    if kind == "attention":
        return dict(kind=kind, shape=shape, B=B, k=k, ctx=lo, ctx_max=ctx)
    layers = 1 if shape == "70b" else rng.choice([1, 2])
    room = rng.choice([0, 0, 1, 3]) * ctx
    vocab = rng.choice([1024, 1024, 32000, 128256])
    return _step("", shape, layers, vocab, B, k, lo, ctx, rng.random() < 0.4, room)


# ---------------------------------------------------------------- inputs ----
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _normal(g, shape, std):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=g)


def _gains(g, n):
    return (1.0 + 0.1 * torch.randn(n, generator=g, device=DEV)).to(torch.bfloat16)


def _shape(name, layers, vocab):
    return SimpleNamespace(**SHAPES[name], n_layers=layers, vocab=vocab, rms_eps=EPS)


def _weights(g, s):
    """One decoder layer after another, then the globals; matrices N(0, 0.02) as the test models have them."""
    qd, kd = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    layers = []
    for _ in range(s.n_layers):
        layers.append(dict(wq=_normal(g, (qd, s.hidden), 0.02), wk=_normal(g, (kd, s.hidden), 0.02), wv=_normal(g, (kd, s.hidden), 0.02),
                           wo=_normal(g, (s.hidden, qd), 0.02), w_gate=_normal(g, (s.ffn, s.hidden), 0.02),
                           w_up=_normal(g, (s.ffn, s.hidden), 0.02), w_down=_normal(g, (s.hidden, s.ffn), 0.02),
                           attn_norm=_gains(g, s.hidden), mlp_norm=_gains(g, s.hidden)))
    top = dict(embed=_normal(g, (s.vocab, s.hidden), 0.02), lm_head=_normal(g, (s.vocab, s.hidden), 0.02),
               final_norm=_gains(g, s.hidden))
    return layers, top


def _lens(case):
    """Valid cache rows per sequence, spread evenly over [ctx, ctx_max]: part of the case, so that its work is fixed."""
    lo, hi = case["ctx"], case["ctx_max"]
    return [hi - (hi - lo) * (b * 11 % 31) // 30 for b in range(case["B"])]


def _kv(g, s, lens):
    """Cached K and V of one layer, N(0, 1), per sequence [kv heads][rows][head_dim]."""
    return [(_normal(g, (s.n_kv_heads, n, s.head_dim), 1.0), _normal(g, (s.n_kv_heads, n, s.head_dim), 1.0)) for n in lens]


def _step_inputs(case, seed):
    g = _gen(seed)
    s = _shape(case["shape"], case["layers"], case["vocab"])
    B, sq = case["B"], case["k"] + 1
    tokens = torch.randint(0, s.vocab, (B, sq), generator=g, device=DEV, dtype=torch.int32)
    parents = None
    if case["tree"]:
        u = torch.rand((B, sq), generator=g, device=DEV)
        parents = (u * torch.arange(sq, device=DEV)).to(torch.int32)      # in [0, i): parents come before children
    layers, top = _weights(g, s)
    return s, tokens, parents, layers, top, g


def _sample_inputs(case, seed):
    """Logits as a language model's: a broad floor and, per row, a few dozen likely tokens above it."""
    g = _gen(seed)
    rows, vocab = case["rows"], case["vocab"]
    logits = torch.randn(rows, vocab, generator=g, device=DEV) * 2.0
    n = min(64, vocab)
    at = torch.randint(0, vocab, (rows, n), generator=g, device=DEV)
    lift = 14.0 - 0.15 * torch.arange(n, device=DEV, dtype=torch.float32) + torch.randn(rows, n, generator=g, device=DEV)
    logits.scatter_(1, at, lift)
    uniforms = torch.rand(rows, generator=g, device=DEV)
    return logits, uniforms


def _cache_context(g, name, layers, B, k, max_seq):
    """A context whose cache has the shape's geometry; the matrices (unused by the call measured) are small."""
    s = _shape(name, layers, 64)
    s.hidden, s.ffn = 64, 64
    w, top = _weights(g, s)
    return s, sv.VerifyContext(sv.make_config(s, B, k, max_seq), w, top)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sample":
        logits, uniforms = _sample_inputs(case, seed)
        return dict(kind=kind, logits=logits, uniforms=uniforms,
                    params=sv.SamplingParams(case["temperature"], case["top_k"], case["top_p"]))
    if kind == "kv_move":
        g = _gen(seed)
        t0, n = case["t0"], case["rows"]
        s, ctx = _cache_context(g, case["shape"], case["layers"], 2, 0, t0 + n + 1)
        src = [_kv(g, s, [n])[0] for _ in range(case["layers"])]
        dst = [(torch.zeros_like(K), torch.zeros_like(V)) for K, V in src]
        return dict(kind=kind, ctx=ctx, t0=t0, src=src, dst=dst)
    lens = _lens(case)
    B, k = case["B"], case["k"]
    if kind == "attention":
        g = _gen(seed)
        s, ctx = _cache_context(g, case["shape"], 1, B, k, max(lens) + k + 1)
        q = torch.randn(B, k + 1, s.n_q_heads, s.head_dim, generator=g, device=DEV)
        for b, (K, V) in enumerate(_kv(g, s, [n + k + 1 for n in lens])):
            ctx.sssd_kv_import(0, b, 0, K, V)
        out = torch.zeros(B, k + 1, s.n_q_heads * s.head_dim, device=DEV)
        return dict(kind=kind, ctx=ctx, q=q, lens=torch.tensor(lens, dtype=torch.int32, device=DEV), out=out)
    s, tokens, parents, layers, top, g = _step_inputs(case, seed)
    ctx = sv.VerifyContext(sv.make_config(s, B, k, max(lens) + k + 1 + case["room"]), layers, top, in_place=case["shape"] == "70b")
    for l in range(s.n_layers):
        for b, (K, V) in enumerate(_kv(g, s, lens)):
            ctx.sssd_kv_import(l, b, 0, K, V)
    M = B * (k + 1)
    logits, hidden = torch.zeros(M, s.vocab, device=DEV), torch.zeros(M, s.hidden, device=DEV)
    ctx.sssd_debug_outputs(logits, hidden)
    ints = [torch.zeros(B, dtype=torch.int32, device=DEV) for _ in range(2)]
    return dict(kind=kind, ctx=ctx, tokens=tokens, parents=parents, lens=torch.tensor(lens, dtype=torch.int32, device=DEV),
                accepted=ints[0], following=ints[1], path=torch.zeros(B, k + 1, dtype=torch.int32, device=DEV),
                logits=logits, hidden=hidden)


def run(state):
    kind = state["kind"]
    if kind == "sample":
        return sv.sssd_op_sample_wide(state["logits"], state["params"], state["uniforms"])
    ctx = state["ctx"]
    if kind == "kv_move":
        for l, ((K, V), (Ko, Vo)) in enumerate(zip(state["src"], state["dst"])):
            ctx.sssd_kv_import(l, 1, state["t0"], K, V)
            ctx.sssd_kv_export(l, 1, state["t0"], Ko, Vo)
        return state["dst"]
    if kind == "attention":
        ctx.sssd_op_attention(0, state["q"], state["lens"], state["out"])
        return state["out"]
    if state["parents"] is None:
        ctx.sssd_verify_step(state["tokens"], state["lens"], state["accepted"], state["following"])
    else:
        ctx.sssd_verify_step_tree(state["tokens"], state["parents"], state["lens"], state["accepted"], state["following"], state["path"])
    return [state["logits"], state["hidden"]]


# ------------------------------------------------------------------ work ----
def work(case):
    kind = case["kind"]
    if kind == "sample":
        n = case["rows"] * case["vocab"]
        return dict(bytes=4.0 * n + 8.0 * case["rows"], flops=4.0 * n)
    s = SHAPES[case["shape"]]
    h, d, nq, nkv, f = s["hidden"], s["head_dim"], s["n_q_heads"], s["n_kv_heads"], s["ffn"]
    if kind == "kv_move":   # in: read and written once; out: the same
        return dict(bytes=4.0 * case["layers"] * 2 * nkv * case["rows"] * d * 2, flops=0.0)
    lens, B, sq = _lens(case), case["B"], case["k"] + 1
    M = B * sq
    attended = sum(sq * (n + (sq + 1) / 2) for n in lens)       # (row, position) pairs
    attn_flops = 4.0 * attended * nq * d
    kv_read = 2.0 * 2 * nkv * d * sum(n + sq for n in lens)
    if kind == "attention":
        return dict(bytes=kv_read + 8.0 * M * nq * d, flops=attn_flops)
    per_layer = h * d * (2 * nq + 2 * nkv) + 3 * h * f
    params = case["layers"] * per_layer + case["vocab"] * h
    kv_new = 2.0 * 2 * nkv * d * M
    return dict(bytes=2.0 * params + case["layers"] * (kv_read + kv_new) + 2.0 * M * h + 4.0 * M * (case["vocab"] + h),
                flops=2.0 * M * params + case["layers"] * attn_flops)


def tolerance(case):
    if case["kind"] in ("sample", "kv_move"):
        return "exact"
    if case["kind"] == "attention":
        return dict(rel=2e-5, max=8e-4)   # measured: 4e-6
    # measured against `exact` at the start: 6e-6 .. 8e-5 (a bf16 rounding of a new K or V element falls the other way now and then)
    return dict(rel=4e-4, max=1.6e-2)


# ----------------------------------------------------------------- exact ----
def _attend(q, K, V, visible):
    """q [rows][nq][d], K/V [nkv][n][d], visible [rows][n] -> [rows][nq*d], all in 64 bits."""
    rows, nq, d = q.shape
    nkv = K.shape[0]
    out = torch.empty(rows, nq, d, dtype=torch.float64, device=DEV)
    for kv in range(nkv):
        heads = slice(kv * nq // nkv, (kv + 1) * nq // nkv)
        g = nq // nkv
        qq = q[:, heads].reshape(rows * g, d).contiguous()
        s = qq @ K[kv].t().contiguous() / math.sqrt(d)
        s = s.view(rows, g, -1).masked_fill(~visible[:, None, :], -math.inf).view(rows * g, -1)
        out[:, heads] = (torch.softmax(s, -1) @ V[kv]).view(rows, g, d)
    return out.view(rows, nq * d)


def _chain_rows(sq, n):
    at = torch.arange(n + sq, device=DEV)
    return at[None, :] <= n + torch.arange(sq, device=DEV)[:, None]


def _exact_step(case, seed):
    s, tokens, parents, layers, top, g = _step_inputs(case, seed)
    lens, B, sq = _lens(case), case["B"], case["k"] + 1
    d, half = s.head_dim, s.head_dim // 2
    # depth and visible new rows of every node
    depth = torch.arange(sq).repeat(B, 1)
    sees = torch.ones(sq, sq, dtype=torch.bool).tril().repeat(B, 1, 1)
    if parents is not None:
        par = parents.cpu().tolist()
        for b in range(B):
            for i in range(sq):
                sees[b, i] = False
                sees[b, i, i] = True
                depth[b, i] = 0
                if i:
                    sees[b, i] |= sees[b, par[b][i]]
                    depth[b, i] = depth[b, par[b][i]] + 1
    pos = (torch.tensor(lens)[:, None] + depth).reshape(-1).to(DEV).double()
    ang = pos[:, None] * (s.rope_base ** (-2.0 * torch.arange(half, device=DEV, dtype=torch.float64) / d))[None, :]
    cos, sin = ang.cos()[:, None, :], ang.sin()[:, None, :]

    def rope(x):
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * cos - b * sin, a * sin + b * cos], -1)

    def norm(x, gain):
        return x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * gain.double()

    def mul(x, w):
        return x @ w.double().t().contiguous()

    def stored(x):      # the cache holds bf16
        return x.to(torch.bfloat16).double()

    x = top["embed"][tokens.reshape(-1).long()].double()
    M = B * sq
    for l in range(s.n_layers):
        w = layers[l]
        xn = norm(x, w["attn_norm"])
        q = rope(mul(xn, w["wq"]).view(M, s.n_q_heads, d))
        k = stored(rope(mul(xn, w["wk"]).view(M, s.n_kv_heads, d)))
        v = stored(mul(xn, w["wv"]).view(M, s.n_kv_heads, d))
        att = []
        for b, (K, V) in enumerate(_kv(g, s, lens)):
            r = slice(b * sq, (b + 1) * sq)
            Kf = torch.cat([K.double(), k[r].transpose(0, 1)], 1)
            Vf = torch.cat([V.double(), v[r].transpose(0, 1)], 1)
            visible = torch.cat([torch.ones(sq, lens[b], dtype=torch.bool, device=DEV), sees[b].to(DEV)], 1)
            att.append(_attend(q[r], Kf, Vf, visible))
        x = x + mul(torch.cat(att), w["wo"])
        xn = norm(x, w["mlp_norm"])
        gate, up = mul(xn, w["w_gate"]), mul(xn, w["w_up"])
        x = x + mul(gate * torch.sigmoid(gate) * up, w["w_down"])
    return [mul(norm(x, top["final_norm"]), top["lm_head"]), x]


def exact(case, seed):
    kind = case["kind"]
    if kind == "sample":
        return None
    if kind == "step":
        return _exact_step(case, seed)
    g = _gen(seed)
    if kind == "kv_move":
        s = _shape(case["shape"], case["layers"], 64)
        s.hidden, s.ffn = 64, 64
        _weights(g, s)
        return [(K.double(), V.double()) for K, V in (_kv(g, s, [case["rows"]])[0] for _ in range(case["layers"]))]
    s = _shape(case["shape"], 1, 64)
    s.hidden, s.ffn = 64, 64
    _weights(g, s)
    lens, B, sq = _lens(case), case["B"], case["k"] + 1
    q = torch.randn(B, sq, s.n_q_heads, s.head_dim, generator=g, device=DEV)
    return torch.stack([_attend(q[b].double(), K.double(), V.double(), _chain_rows(sq, lens[b]))
                        for b, (K, V) in enumerate(_kv(g, s, [n + sq for n in lens]))])
