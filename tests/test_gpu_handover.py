"""Partial results handed over between the workgroups of one launch (one die's workgroups share its L2).  In a context created with
SSSD_NO_WAIT nobody waits for the others, so the last workgroup of every group does all of its work: the way taken when workgroups do not
arrive in time.  Both ways must give the reference and the same bits, launch after launch (the words between them are zero again); the
context says which launches hand over and how many groups took the slow way."""
from types import SimpleNamespace

import pytest
import torch

pytestmark = pytest.mark.gpu

from harness import Pair, compare_step, gen_weights
from paper_2411_05894_amd import binding as sv
from sssd_synth import MODEL_SHAPES, global_weight_specs, layer_weight_specs, normal_bf16, uniform_int
from test_gpu_attention_segments import reference

DEV = "cuda:0"
QKV, O, GATE_UP, DOWN, LM, ATTENTION = (1 << i for i in range(6))   # bits of sssd_debug_handover


def attention_context(shape_name, B, k, max_seq, no_wait):
    """A context of which only the cache matters: the matrices are small and zero."""
    s = MODEL_SHAPES[shape_name]
    s = type(s)(**{**s.__dict__, "n_layers": 1, "vocab": 1024, "hidden": 64, "ffn": 64})
    layers = [{n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in layer_weight_specs(s)}]
    g = {n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in global_weight_specs(s)}
    return s, sv.VerifyContext(sv.make_config(s, B, k, max_seq), layers, g, no_wait=no_wait)


@pytest.mark.parametrize("shape_name,k,lens,max_seq", [
    ("8b", 8, [2048], 2057),               # 8 heads, 17 segments of one sequence
    ("8b", 0, [5000], 5001),               # four rows for 32 segments: most have nothing to merge
    ("8b", 17, [700, 12345], 12400),       # five row tiles, two passes
    ("8b", 31, [1500, 40, 3000], 3100),    # a sequence of one segment beside merged ones
    ("8b", 12, [900 + 100 * i for i in range(8)], 4000),    # two passes of two tiles
    ("8b", 31, [900 + 100 * i for i in range(9)], 4000),    # two passes of four tiles, up to two workgroups per compute unit
    ("tiny", 4, [300, 2000, 5, 1000], 2100)])               # two kv heads, head size 64
def test_attention_merged_inside_the_launch(shape_name, k, lens, max_seq):
    B, sq = len(lens), k + 1
    outs, late = [], []
    for no_wait in (False, True):
        s, ctx = attention_context(shape_name, B, k, max_seq, no_wait=no_wait)
        q = (normal_bf16(51, 1, (B, sq, s.n_q_heads, s.head_dim), 1.0, device=DEV).float() * 1.28).contiguous()
        kv = [[normal_bf16(52, 2 * b + i, (s.n_kv_heads, n + sq, s.head_dim), 1.0, device=DEV) for i in range(2)] for b, n in enumerate(lens)]
        for b in range(B):
            ctx.sssd_kv_import(0, b, 0, *kv[b])
        out = torch.empty(B, sq, s.n_q_heads * s.head_dim, dtype=torch.float32, device=DEV)
        print(f"hand-over attention {shape_name} k={k} B={B} no_wait={no_wait}", flush=True)
        for i in range(12):
            out.fill_(-1.0)
            ctx.sssd_op_attention(0, q, torch.tensor(lens, dtype=torch.int32, device=DEV), out)
            assert ctx.sssd_verify_sync() == 0
            outs.append(out.clone())
            launches, n = ctx.sssd_debug_handover(B, k)
            assert launches & ATTENTION, "merged by a second launch"
            if i == 0: groups = n        # of sequences of more than one segment
            if no_wait: assert n == (i + 1) * groups > 0
        late.append(n)
    assert late[0] < late[1]
    got = outs[0].view(B, sq, s.n_q_heads, s.head_dim)
    for b in range(B):   # as test_gpu_attention_segments: operands in bf16 pairs, ~2^-17 relative
        assert (got[b] - reference(q[b], *kv[b], lens[b], s.n_q_heads // s.n_kv_heads)).abs().max().item() <= 1e-4, b
    for o in outs[1:]:
        assert torch.equal(o, outs[0])


# K in two slices and more everywhere but in the O projection of the smaller model: 17 to 65 k-tiles (slices of unequal
# length), units of one to ten row tiles shared out over as few as two and as many as eight slices, blocks of eight and six row tiles, column groups
# that end inside the matrix, more slices than units; an LM head of few columns
@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,vocab", [(768, 6, 2, 128, 2064, 1040), (528, 4, 4, 64, 1120, 4112)])
@pytest.mark.parametrize("B,k", [(3, 10), (6, 7), (5, 12), (7, 13), (9, 12), (9, 15), (5, 31), (7, 25), (11, 28), (16, 31)])   # 33 .. 512 rows
def test_split_gemms_summed_inside_the_launch(hidden, nq, nkv, d, ffn, vocab, B, k):
    s = SimpleNamespace(name="edge", n_layers=2, hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=ffn, vocab=vocab, rms_eps=1e-5,
                        rope_base=10000.0)
    p = Pair(s, seed=61, max_batch=B, max_k=k, max_seq=96, unit_gains=False)
    late = Pair(s, seed=61, max_batch=B, max_k=k, max_seq=96, unit_gains=False, oracle_batch=1)
    late.ctx.sssd_verify_destroy()
    layers, g = gen_weights(s, 61, late.dev, False)
    late.ctx = sv.VerifyContext(late.cfg, layers, g, no_wait=True)
    late.ctx.sssd_debug_outputs(late.logits, late.hidden)
    late.ctx.sssd_debug_argmax(late.that)
    lens = uniform_int(62, B * 64 + k, (B,), 0, 96 - k - 1).to(torch.int32)
    for b in range(B):
        p.prefill_random_kv(63, b, int(lens[b]), oracle_slot=b)
        late.prefill_random_kv(63, b, int(lens[b]))
    tokens = uniform_int(64, B * 64 + k, (B, k + 1), 0, s.vocab - 1)
    ref = p.oracle.verify_step(tokens, lens, return_hidden=True)
    first, slow = None, []
    for pair in (p, late):
        print(f"hand-over step h={hidden} ffn={ffn} B={B} k={k} no_wait={pair is late}", flush=True)
        for i in range(4):
            pair.logits.fill_(-1.0)
            got = pair.step(tokens, lens)
            if first is None:
                first = got
                compare_step(got, ref, tokens)
                herr = (got["hidden"] - ref["hidden"]).abs().max().item() / ref["hidden"].abs().max().item()
                assert herr < 5e-3   # a bf16 rounding of a new K or V element may fall the other way: 2^-9 of it
            for name in ("logits", "hidden", "that", "accepted_len", "next_token"):
                assert torch.equal(got[name], first[name]), (name, i, pair is late)
            launches, n = pair.ctx.sssd_debug_handover(B, k)
            assert launches == QKV | GATE_UP | DOWN | LM | (O if hidden == 768 else 0)
            if i == 0: groups = n
            if pair is late: assert n == (i + 1) * groups > 0
        slow.append(n)
        pair.ctx.sssd_verify_destroy()
    assert slow[0] < slow[1]


# One column tile, so one arg-max partial or sum of squares per row, in row blocks whose waves hold two pairs of tiles
@pytest.mark.parametrize("hidden,ffn,vocab", [(512, 48, 16), (16, 512, 528)])
@pytest.mark.parametrize("B,k", [(11, 15), (16, 31)])   # 176 and 512 rows
def test_a_single_column_tile(hidden, ffn, vocab, B, k):
    s = SimpleNamespace(name="edge", n_layers=2, hidden=hidden, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=ffn, vocab=vocab, rms_eps=1e-5,
                        rope_base=10000.0)
    print(f"single column tile h={hidden} ffn={ffn} vocab={vocab} B={B} k={k}", flush=True)
    p = Pair(s, seed=81, max_batch=B, max_k=k, max_seq=96, unit_gains=False)
    lens = uniform_int(82, B * 64 + k, (B,), 0, 96 - k - 1).to(torch.int32)
    for b in range(B):
        p.prefill_random_kv(83, b, int(lens[b]), oracle_slot=b)
    tokens = uniform_int(84, B * 64 + k, (B, k + 1), 0, s.vocab - 1)
    ref = p.oracle.verify_step(tokens, lens, return_hidden=True)
    got = p.step(tokens, lens)
    compare_step(got, ref, tokens)
    herr = (got["hidden"] - ref["hidden"]).abs().max().item() / ref["hidden"].abs().max().item()
    assert herr < 5e-3   # a bf16 rounding of a new K or V element may fall the other way: 2^-9 of it
    p.ctx.sssd_verify_destroy()


def edge_pair(seed, B, k, max_seq=700):
    s = SimpleNamespace(name="edge", n_layers=2, hidden=768, n_q_heads=6, n_kv_heads=2, head_dim=128, ffn=2064, vocab=1040, rms_eps=1e-5,
                        rope_base=10000.0)
    p = Pair(s, seed=seed, max_batch=B, max_k=k, max_seq=max_seq, unit_gains=False, oracle_batch=1)
    lens = uniform_int(seed + 1, B * 64 + k, (B,), max_seq // 2, max_seq - k - 1).to(torch.int32)
    for b in range(B):
        p.prefill_random_kv(seed + 2, b, int(lens[b]))
    tokens = uniform_int(seed + 3, B * 64 + k, (B, k + 1), 0, s.vocab - 1)
    assert p.ctx.sssd_debug_handover(B, k)[0] == QKV | O | GATE_UP | DOWN | LM | ATTENTION
    return p, tokens.to(DEV, torch.int32), lens.to(DEV), [torch.empty(B, dtype=torch.int32, device=DEV) for _ in range(2)]


# Every product and the attention of a step hand over: 36, 144 and 512 rows, segments of sequences of 350..700 positions
ROWS = pytest.mark.parametrize("B,k", [(4, 8), (16, 8), (16, 31)])


@ROWS
def test_replayed_hand_over(B, k):
    """Under graph capture, with the program's own steps and synchronisations between the replays."""
    p, tokens, lens, ints = edge_pair(91, B, k)
    print(f"replayed hand-over B={B} k={k}", flush=True)

    def outputs():
        assert p.ctx.sssd_verify_sync() == 0
        return [p.logits.clone(), p.hidden.clone(), p.that.clone()] + [t.clone() for t in ints]

    def eager(t):
        p.ctx.sssd_verify_step(t, lens, *ints)
        return outputs()

    want, other = eager(tokens), (tokens + 1) % 1040
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            p.ctx.sssd_verify_step(tokens, lens, *ints)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(4):
        for t in (p.logits, p.hidden, p.that, *ints):
            t.fill_(-5)
        g.replay()
        assert all(torch.equal(a, b) for a, b in zip(outputs(), want)), rep
        eager(other)
        assert all(torch.equal(a, b) for a, b in zip(eager(tokens), want)), rep
    p.ctx.sssd_verify_destroy()


@ROWS
def test_two_contexts_at_once(B, k):
    """Two contexts on two streams: workgroups of one hold compute units that the other's wait for.  Each gives what it gives alone."""
    both = [edge_pair(seed, B, k) for seed in (101, 111)]
    streams = [torch.cuda.Stream() for _ in both]
    want = []
    for p, tokens, lens, ints in both:
        p.ctx.sssd_verify_step(tokens, lens, *ints)
        assert p.ctx.sssd_verify_sync() == 0
        want.append([t.clone() for t in (p.logits, p.hidden, p.that, *ints)])
    for turn in range(4):
        print(f"two contexts B={B} k={k} turn {turn}", flush=True)
        for p, _, _, ints in both:
            for t in (p.logits, p.hidden, p.that, *ints):
                t.fill_(-5)
        torch.cuda.synchronize()
        for _ in range(12):
            for s, (p, tokens, lens, ints) in zip(streams, both):
                with torch.cuda.stream(s):
                    p.ctx.sssd_verify_step(tokens, lens, *ints)
        torch.cuda.synchronize()
        for (p, _, _, ints), w in zip(both, want):
            assert all(torch.equal(a, b) for a, b in zip((p.logits, p.hidden, p.that, *ints), w)), turn
    print("groups that did not wait:", [p.ctx.sssd_debug_handover(B, k)[1] for p, _, _, _ in both], flush=True)
    for p, _, _, _ in both:
        assert p.ctx.sssd_verify_sync() == 0
        p.ctx.sssd_verify_destroy()


def test_on_every_stream():
    """The dies that take a launch's workgroups depend on the stream's hardware queue; contexts made and steps run on any of them hand over."""
    B, k = 4, 8
    streams = [torch.cuda.Stream() for _ in range(9)]
    for s in streams:
        with torch.cuda.stream(s):
            torch.zeros(64, device=DEV)
    torch.cuda.synchronize()
    p, tokens, lens, ints = edge_pair(121, B, k)
    p.ctx.sssd_verify_step(tokens, lens, *ints)
    assert p.ctx.sssd_verify_sync() == 0
    want = [t.clone() for t in (p.logits, p.hidden, p.that, *ints)]
    groups = 2 * (8 + 4 * 2)     # of a step, at least: 8 of attention and the column groups of four products in two layers
    for i, s in enumerate(streams):
        print(f"hand-over on stream {i}", flush=True)
        with torch.cuda.stream(s):
            before = p.ctx.sssd_debug_handover(B, k)[1]
            for _ in range(8):
                p.ctx.sssd_verify_step(tokens, lens, *ints)
            late = p.ctx.sssd_debug_handover(B, k)[1] - before
            assert p.ctx.sssd_verify_sync() == 0
        assert late < groups, "workgroups that found themselves on other dies than expected"   # of 8 steps: most groups waited for each other
        assert all(torch.equal(a, b) for a, b in zip((p.logits, p.hidden, p.that, *ints), want)), i
    p.ctx.sssd_verify_destroy()


# Nine groups of 256 columns: one die gets two, so a launch that sums its 256 k-tiles inside has half the slices of one that does not.
# Sixteen share out evenly.
@pytest.mark.parametrize("hidden,inside", [(2304, False), (4096, True)])
def test_row_blocks_whose_column_groups_do_not_share_out_evenly(hidden, inside):
    s = SimpleNamespace(name="edge", n_layers=1, hidden=hidden, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=8192, vocab=16, rms_eps=1e-5, rope_base=10000.0)
    layers = [{n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in layer_weight_specs(s)}]
    g = {n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in global_weight_specs(s)}
    ctx = sv.VerifyContext(sv.make_config(s, 16, 31, 64), layers, g)
    for B, k in ((11, 28), (16, 31)):   # 319 and 512 rows
        assert bool(ctx.sssd_debug_handover(B, k)[0] & DOWN) == inside, (B, k)
    assert ctx.sssd_debug_handover(16, 8)[0] & DOWN   # one row block: the weights' stream bounds it
    ctx.sssd_verify_destroy()
