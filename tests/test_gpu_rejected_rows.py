"""Sequences that a step of more than 32 rows rejects: too long, negative, or with a page outside the pool, beside healthy ones.
The QKV epilogue of the pipelined kernel writes the cache inside the launch where K is whole (hidden 256) and in a launch of its
own where K is split (1024); either way a rejected sequence writes nothing, and the others get the oracle's logits."""
from types import SimpleNamespace

import pytest
import torch

pytestmark = pytest.mark.gpu

from harness import LOGIT_TOL, Pair
from paper_2411_05894_amd import binding as sv
from sssd_synth import uniform_int

DEV = "cuda:0"
MAX_SEQ = 96


def cache(p, B):
    s, out = p.shape, []
    for l in range(s.n_layers):
        for b in range(B):
            K = torch.empty(s.n_kv_heads, MAX_SEQ, s.head_dim, dtype=torch.bfloat16, device=DEV)
            V = torch.empty_like(K)
            p.ctx.sssd_kv_export(l, b, 0, K, V)
            out.append(torch.stack([K, V]).view(torch.int16).cpu())
    return out


@pytest.mark.parametrize("hidden,B,k", [(256, 8, 8), (256, 7, 25), (1024, 8, 8), (1024, 7, 25)])
def test_rejected_sequences_of_large_steps(hidden, B, k):
    s = SimpleNamespace(name="edge", n_layers=2, hidden=hidden, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=432, vocab=1040, rms_eps=1e-5,
                        rope_base=10000.0)
    p = Pair(s, seed=41, max_batch=B, max_k=k, max_seq=MAX_SEQ)
    lens = [40, 50, 33, 20, 64, 7, 31, 60][:B - 1] + [45]
    for b in range(B):
        p.prefill_random_kv(42, b, MAX_SEQ if b in (1, 2, 3) else lens[b], oracle_slot={0: 0, B - 1: 1}.get(b))
    tokens = uniform_int(43, B * 64 + k, (B, k + 1), 0, s.vocab - 1)
    ref = p.oracle.verify_step(tokens[[0, B - 1]].contiguous(), torch.tensor([lens[0], lens[B - 1]], dtype=torch.int32))
    _, bps, n_pages = sv.sssd_kv_geometry(p.cfg)
    bad = torch.arange(B * bps, dtype=torch.int32).view(B, bps)
    bad[2, 1] = n_pages + 5                                             # rows 32..63 of sequence 2
    too_long, negative = list(lens), list(lens)
    too_long[1], negative[3] = MAX_SEQ - k, -3                          # one row too many
    for name, ls, table, out in (("too long", too_long, None, 1), ("negative", negative, None, 3), ("bad page", lens, bad, 2)):
        before = cache(p, B)
        if table is not None:
            p.ctx.sssd_kv_set_block_table(table.to(DEV))
        acc, nxt = (torch.empty(B, dtype=torch.int32, device=DEV) for _ in range(2))
        print(f"rejected rows h={hidden} B={B} k={k}: {name}", flush=True)
        p.ctx.sssd_verify_step(tokens.to(DEV, torch.int32), torch.tensor(ls, dtype=torch.int32, device=DEV), acc, nxt)
        assert p.ctx.sssd_verify_sync() == sv.SSSD_ENOSPACE, name
        p.ctx.sssd_kv_set_block_table(None)
        for i, (x, y) in enumerate(zip(before, cache(p, B))):
            b = i % B
            kept = MAX_SEQ if b == out else lens[b]                     # new rows of the accepted ones lie behind
            assert torch.equal(x[:, :, :kept], y[:, :, :kept]), (name, i // B, b)
            if b != out:
                assert torch.equal(x[:, :, lens[b] + k + 1:], y[:, :, lens[b] + k + 1:]), (name, i // B, b)
        logits = p.logits.cpu().view(B, k + 1, -1)
        for i, b in enumerate((0, B - 1)):
            assert (logits[b] - ref["logits"][i]).abs().max().item() <= LOGIT_TOL, (name, b)
    p.ctx.sssd_verify_destroy()
