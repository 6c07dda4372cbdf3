"""The LM head's arg-max over its three levels (a thread's columns, a workgroup's, the row's) on every form of the GEMM that
carries it: equal maxima in different column groups go to the lowest token, logits that are no number never win, and a row
without any number above -inf gives token 0, never an id outside the vocabulary."""
from types import SimpleNamespace

import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2411_05894_amd import binding as sv
from sssd_synth import TensorId, global_weight_specs, layer_weight_specs, make_weight, uniform_int

DEV = "cuda:0"
VOCAB = 4112                                   # 257 tiles of 16: column groups end inside every 32-column block
TIED, OTHER = [5, 700, 4100], [300, 2048, 4111]
FORMS = [(256, 1, 4), (256, 2, 9),             # small-step kernel, whole K: one and two row tiles
         (4224, 3, 4),                         # ... K split, summed by the last workgroup
         (256, 5, 8), (256, 7, 25),            # pipelined kernel, whole K: one block of rows, several
         (1024, 5, 8), (1024, 7, 25)]          # ... K split, an epilogue launch


def head(kind, g, hidden):
    """The LM head and final norm that make the wanted logits."""
    w = g["lm_head"]
    if kind == "ties":                         # the rows' sign decides which of the two sets is the maximum
        v = torch.randn(hidden, generator=torch.Generator().manual_seed(hidden)).to(torch.bfloat16).to(DEV)
        w[TIED] = v
        w[OTHER] = -v
    elif kind == "some nan":
        w[::3] = float("nan")
        w[4096:] = float("nan")                # whole tiles without a number
    elif kind == "all nan":
        g["final_norm"][7] = float("nan")
    else:                                      # -inf: an overflowing product in every column
        w.zero_()
        w[:, 0] = -3.3e38
        g["embed"][:, 0] = 4.0


@pytest.mark.parametrize("kind", ["ties", "some nan", "all nan", "minus infinity"])
@pytest.mark.parametrize("hidden,B,k", FORMS)
def test_argmax_of_unusual_rows(hidden, B, k, kind):
    s = SimpleNamespace(name="edge", n_layers=1, hidden=hidden, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=64, vocab=VOCAB, rms_eps=1e-5,
                        rope_base=10000.0)
    layers = [{n: make_weight(3, n, TensorId.layer(0, slot), shp, device=DEV) for n, slot, shp in layer_weight_specs(s)}]
    g = {n: make_weight(3, n, tid, shp, device=DEV) for n, tid, shp in global_weight_specs(s)}
    head(kind, g, hidden)
    ctx = sv.VerifyContext(sv.make_config(s, B, k, 64), layers, g)
    M = B * (k + 1)
    logits = torch.zeros(M, VOCAB, device=DEV)
    that = torch.full((M,), -1, dtype=torch.int32, device=DEV)
    ctx.sssd_debug_outputs(logits, None)
    ctx.sssd_debug_argmax(that)
    tokens = uniform_int(5, M, (B, k + 1), 0, VOCAB - 1).to(DEV, torch.int32)
    acc, nxt = (torch.full((B,), -1, dtype=torch.int32, device=DEV) for _ in range(2))
    print(f"lm arg-max {kind} h={hidden} B={B} k={k}", flush=True)
    ctx.sssd_verify_step(tokens, torch.zeros(B, dtype=torch.int32, device=DEV), acc, nxt)
    assert ctx.sssd_verify_sync() == 0
    if kind == "ties":
        assert all(torch.equal(logits[:, TIED[0]], logits[:, c]) for c in TIED)
        tied = (that == TIED[0]) | (that == OTHER[0])      # all but rows at a right angle to v
        assert tied.float().mean().item() > 0.75
    elif kind == "some nan":
        assert torch.isnan(logits[:, ::3]).all() and torch.isnan(logits[:, 4096:]).all() and not torch.isnan(logits[:, 1:4096:3]).any()
    elif kind == "all nan":
        assert torch.isnan(logits).all()
    else:
        assert torch.isneginf(logits).all()
    z = torch.where(torch.isnan(logits), -torch.inf, logits)
    first = (z == z.max(-1, keepdim=True).values).int().argmax(-1).to(torch.int32)
    assert torch.equal(that, first)
    walk = that.view(B, k + 1)
    n = (tokens[:, 1:] == walk[:, :-1]).int().cumprod(-1).sum(-1).to(torch.int32)
    assert torch.equal(acc, n) and torch.equal(nxt, walk.gather(1, n[:, None].long())[:, 0])
    ctx.sssd_verify_destroy()
