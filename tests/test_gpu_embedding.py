"""The embedding launch: row tiles that end inside the step, chunks of channels that end inside a chunk or an operand tile, embedding
and gains at odd addresses; against the oracle."""
from types import SimpleNamespace

import pytest
import torch

pytestmark = pytest.mark.gpu

from harness import Pair, compare_step, gen_weights
from paper_2411_05894_amd import binding as sv
from sssd_synth import uniform_int


def moved(t):
    """The same values two bytes further on."""
    room = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    return room[1:].view(t.shape).copy_(t)


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("hidden,B,k", [(16, 1, 0), (240, 2, 7), (272, 3, 10), (784, 5, 9), (1040, 13, 4)])   # 1, 16, 33, 50 and 65 rows
def test_embedding(hidden, B, k, odd):
    s = SimpleNamespace(name="edge", n_layers=1, hidden=hidden, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=48, vocab=528, rms_eps=1e-5,
                        rope_base=10000.0)
    print(f"embedding h={hidden} B={B} k={k} odd={odd}", flush=True)
    p = Pair(s, seed=71, max_batch=B, max_k=k, max_seq=64, unit_gains=False)
    if odd:
        p.ctx.sssd_verify_destroy()
        layers, g = gen_weights(s, 71, p.dev, False)
        g["embed"] = moved(g["embed"])
        layers[0]["attn_norm"] = moved(layers[0]["attn_norm"])
        assert g["embed"].data_ptr() % 4 == 2
        p.ctx = sv.VerifyContext(p.cfg, layers, g)
        p.ctx.sssd_debug_outputs(p.logits, p.hidden)
        p.ctx.sssd_debug_argmax(p.that)
    lens = uniform_int(72, B, (B,), 0, 64 - k - 1).to(torch.int32)
    for b in range(B):
        p.prefill_random_kv(73, b, int(lens[b]), oracle_slot=b)
    tokens = uniform_int(74, B, (B, k + 1), 0, s.vocab - 1)
    ref = p.oracle.verify_step(tokens, lens, return_hidden=True)
    gpu = p.step(tokens, lens)
    compare_step(gpu, ref, tokens)
    herr = (gpu["hidden"] - ref["hidden"]).abs().max().item() / ref["hidden"].abs().max().item()
    assert herr < 5e-3      # a bf16 rounding of a new K or V element may fall the other way: 2^-9 of it
    p.ctx.sssd_verify_destroy()
