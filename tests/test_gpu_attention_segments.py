"""Attention over segments cut from the device's own lens: ragged batches in caches with room to grow, more sequences than a
wave has lanes, sequences of one segment (finished without a merge) beside long ones, several passes over the row tiles, and
sequences that the step rejects.  Reference: softmax in 64 bits.  A sequence's results are the same bits whatever the others
hold."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

from harness import Pair
from paper_2411_05894_amd import binding as sv
from sssd_synth import MODEL_SHAPES, global_weight_specs, layer_weight_specs, normal_bf16, uniform_int

DEV = "cuda:0"
CASES = [  # shape, k, lens, max_seq
    ("8b", 8, [5000, 17, 1200], 20000),            # three row tiles
    ("8b", 4, [9000], 9100),                       # one sequence, segments of nine blocks: a partial round of the waves
    ("8b", 31, [479] * 16, 1024),                  # eight row tiles in two passes, one segment per sequence
    ("8b", 12, [0, 700, 31, 32, 1500], 4096),      # four row tiles
    ("70b", 8, [2048, 40], 8192),                  # five row tiles
    ("70b", 10, [700, 3000], 3100),                # six row tiles
    ("70b", 12, [64, 640], 1000),                  # seven row tiles: two passes of four, one tile to spare
    ("8b", 0, [100 * i for i in range(40)], 4200),
    ("tiny", 1, [(37 * i) % 301 for i in range(130)], 400),   # more than 64 sequences, head size 64
]


def reference(q, K, V, n_old, g):
    sq, nq, d = q.shape
    out = torch.empty(sq, nq, d, dtype=torch.float64, device=DEV)
    seen = torch.arange(n_old + sq, device=DEV)[None, :] <= n_old + torch.arange(sq, device=DEV)[:, None]
    for h in range(nq):
        s = q[:, h].double().contiguous() @ K[h // g].double().t().contiguous() / math.sqrt(d)
        out[:, h] = torch.softmax(s.masked_fill(~seen, -math.inf), -1) @ V[h // g].double()
    return out


def attention_context(shape_name, B, k, max_seq):
    """A context of which only the cache matters: the matrices are small and zero."""
    s = MODEL_SHAPES[shape_name]
    s = type(s)(**{**s.__dict__, "n_layers": 1, "vocab": 1024, "hidden": 64, "ffn": 64})
    layers = [{n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in layer_weight_specs(s)}]
    g = {n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in global_weight_specs(s)}
    return s, sv.VerifyContext(sv.make_config(s, B, k, max_seq), layers, g)


@pytest.mark.parametrize("shape_name,k,lens,max_seq", CASES)
def test_ragged_batches(shape_name, k, lens, max_seq):
    B = len(lens)
    s, ctx = attention_context(shape_name, B, k, max_seq)
    sq, d, grp = k + 1, s.head_dim, s.n_q_heads // s.n_kv_heads
    q = (normal_bf16(41, 1, (B, sq, s.n_q_heads, d), 1.0, device=DEV).float() * 1.28).contiguous()
    kv = []
    for b, n in enumerate(lens):
        kv.append([normal_bf16(42, 2 * b + i, (s.n_kv_heads, n + sq, d), 1.0, device=DEV) for i in range(2)])
        ctx.sssd_kv_import(0, b, 0, *kv[b])
    out = torch.empty(B, sq, s.n_q_heads * d, dtype=torch.float32, device=DEV)
    print(f"attention segments {shape_name} k={k} B={B}", flush=True)

    def run(ls):
        ctx.sssd_op_attention(0, q, torch.tensor(ls, dtype=torch.int32, device=DEV), out)
        return ctx.sssd_verify_sync(), out.view(B, sq, s.n_q_heads, d).clone()

    rc, got = run(lens)
    assert rc == 0
    for b in range(B):
        # q and the probabilities enter the MFMAs as bf16 hi+lo pairs (~2^-17 relative); outputs are O(1)
        assert (got[b] - reference(q[b], *kv[b], lens[b], grp)).abs().max().item() <= 1e-4, b
    if B > 2:      # a length that does not fit: that sequence alone is rejected
        bad = list(lens)
        bad[1] = max_seq
        rc, other = run(bad)
        assert rc == sv.SSSD_ENOSPACE
        for b in (0, 2):
            assert (other[b] - reference(q[b], *kv[b], lens[b], grp)).abs().max().item() <= 1e-4, b


@pytest.mark.parametrize("shape_name,k", [("8b", 8), ("8b", 0), ("8b", 31), ("70b", 8), ("tiny", 4)])
def test_the_other_sequences_change_no_bit(shape_name, k):
    """One sequence's rows are cut, summed and merged alike whatever its neighbours hold, and wherever it stands in the batch."""
    max_seq, mine = 20000, 3000
    s, ctx = attention_context(shape_name, 4, k, max_seq)
    sq = k + 1
    q = (normal_bf16(43, 1, (4, sq, s.n_q_heads, s.head_dim), 1.0, device=DEV).float() * 1.28).contiguous()
    q[2] = q[0]
    kv = [normal_bf16(44, i, (s.n_kv_heads, max_seq, s.head_dim), 1.0, device=DEV) for i in range(2)]
    for b in range(4):
        ctx.sssd_kv_import(0, b, 0, *kv)
    out = torch.empty(4, sq, s.n_q_heads * s.head_dim, dtype=torch.float32, device=DEV)
    seen = []
    for lens in ([mine, 10, mine, 0], [mine, 15000, mine, max_seq - sq], [mine, mine, mine, mine], [mine, 700, mine, 9000], [mine, max_seq, mine, 5]):
        print(f"attention beside others {shape_name} k={k} lens={lens}", flush=True)
        ctx.sssd_op_attention(0, q, torch.tensor(lens, dtype=torch.int32, device=DEV), out)
        assert ctx.sssd_verify_sync() == (0 if max(lens) + sq <= max_seq else sv.SSSD_ENOSPACE)
        seen += [out[0].clone(), out[2].clone()]
    assert all(torch.equal(o, seen[0]) for o in seen)


def test_a_long_sequence_with_a_bad_page_is_read_as_empty():
    """A sequence of several segments whose table names a page outside the pool, beside healthy ones: the error is reported,
    the others' logits and every cached row keep their bits."""
    s = MODEL_SHAPES["tiny"]
    B, k, max_seq = 3, 4, 1700
    p = Pair(s, seed=91, max_batch=B, max_k=k, max_seq=max_seq)
    _, bps, n_pages = sv.sssd_kv_geometry(p.cfg)
    table = torch.arange(n_pages, dtype=torch.int32).flip(0).view(B, bps).contiguous()
    good, bad = table.to(DEV), table.clone()
    bad[1, 30] = n_pages + 5
    p.ctx.sssd_kv_set_block_table(good)
    ctxs = [300, 1600, 45]
    for b in range(B):
        p.prefill_random_kv(92, b, ctxs[b])
    lens = torch.tensor(ctxs, dtype=torch.int32)
    tokens = uniform_int(93, 1, (B, k + 1), 0, s.vocab - 1)

    def cache():
        got = []
        for l in range(s.n_layers):
            for b in range(B):
                kv = [torch.empty(s.n_kv_heads, max_seq, s.head_dim, dtype=torch.bfloat16, device=DEV) for _ in range(2)]
                p.ctx.sssd_kv_export(l, b, 0, *kv)
                got += [x.view(torch.int16) for x in kv]
        return got

    healthy = p.step(tokens, lens)["logits"]
    before = cache()
    p.ctx.sssd_kv_set_block_table(bad.to(DEV))
    dev = torch.zeros(B, dtype=torch.int32, device=DEV), torch.zeros(B, dtype=torch.int32, device=DEV)
    logits = torch.zeros(B * (k + 1), s.vocab, device=DEV)
    p.ctx.sssd_debug_logits(logits)
    p.ctx.sssd_verify_step(tokens.to(DEV), lens.to(DEV), *dev)
    assert p.ctx.sssd_verify_sync() == sv.SSSD_ENOSPACE
    p.ctx.sssd_kv_set_block_table(good)
    logits = logits.cpu().view(B, k + 1, s.vocab)
    for b in (0, 2):
        assert torch.equal(logits[b], healthy[b])
    assert torch.isfinite(logits[1]).all()
    assert all(torch.equal(x, y) for x, y in zip(cache(), before))


@pytest.mark.parametrize("length", [-1, -(1 << 31), (1 << 31) - 1, (1 << 31) - 3, 156])
def test_lengths_that_do_not_fit_are_rejected(length):
    """Negative, one too many and so large that the new rows' count takes them past 2^31: the call reports it, and neither the
    step, the attention entry point nor the commit touches the cache."""
    s = MODEL_SHAPES["tiny"]
    B, k, max_seq = 2, 4, 160
    p = Pair(s, seed=95, max_batch=B, max_k=k, max_seq=max_seq)
    for b in range(B):
        p.prefill_random_kv(96, b, max_seq)
    print(f"length {length}", flush=True)

    def row(b):
        kv = [torch.empty(s.n_kv_heads, max_seq, s.head_dim, dtype=torch.bfloat16, device=DEV) for _ in range(2)]
        p.ctx.sssd_kv_export(0, b, 0, *kv)
        return [x.view(torch.int16) for x in kv]

    before = row(1)
    lens = torch.tensor([20, length], dtype=torch.int32, device=DEV)
    acc, nxt = (torch.zeros(B, dtype=torch.int32, device=DEV) for _ in range(2))
    p.ctx.sssd_verify_step(uniform_int(97, 1, (B, k + 1), 0, s.vocab - 1).to(DEV), lens, acc, nxt)
    assert p.ctx.sssd_verify_sync() == sv.SSSD_ENOSPACE
    q = torch.randn(B, k + 1, s.n_q_heads, s.head_dim, device=DEV)
    p.ctx.sssd_op_attention(0, q, lens, torch.empty(B, k + 1, s.n_q_heads * s.head_dim, device=DEV))
    assert p.ctx.sssd_verify_sync() == sv.SSSD_ENOSPACE
    path = torch.tensor([[0, 2, -1, -1, -1]] * B, dtype=torch.int32, device=DEV)
    p.ctx.sssd_kv_commit_tree(lens, torch.ones(B, dtype=torch.int32, device=DEV), path)
    assert p.ctx.sssd_verify_sync() == sv.SSSD_ENOSPACE
    assert lens.tolist() == [22, length]
    assert all(torch.equal(x, y) for x, y in zip(row(1), before))
