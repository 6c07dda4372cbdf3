"""Attention over segments cut from the device's own lens: ragged batches in caches with room to grow, more sequences than a
wave has lanes, sequences of one segment (finished without a merge) beside long ones, several passes over the row tiles, and
sequences that the step rejects.  Reference: softmax in 64 bits."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2411_05894_amd import binding as sv
from sssd_synth import MODEL_SHAPES, global_weight_specs, layer_weight_specs, normal_bf16

DEV = "cuda:0"
CASES = [  # shape, k, lens, max_seq
    ("8b", 8, [5000, 17, 1200], 20000),            # three row tiles
    ("8b", 4, [9000], 9100),                       # one sequence, segments of an odd number of blocks
    ("8b", 31, [479] * 16, 1024),                  # eight row tiles in two passes, one segment per sequence
    ("8b", 12, [0, 700, 31, 32, 1500], 4096),      # four row tiles
    ("70b", 8, [2048, 40], 8192),                  # five row tiles
    ("70b", 10, [700, 3000], 3100),                # six row tiles
    ("70b", 12, [64, 640], 1000),                  # seven row tiles: two passes, the second with a wave to spare
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


@pytest.mark.parametrize("shape_name,k,lens,max_seq", CASES)
def test_ragged_batches(shape_name, k, lens, max_seq):
    s = MODEL_SHAPES[shape_name]
    s = type(s)(**{**s.__dict__, "n_layers": 1, "vocab": 1024, "hidden": 64, "ffn": 64})
    layers = [{n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in layer_weight_specs(s)}]
    g = {n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in global_weight_specs(s)}
    B, sq, d, grp = len(lens), k + 1, s.head_dim, s.n_q_heads // s.n_kv_heads
    ctx = sv.VerifyContext(sv.make_config(s, B, k, max_seq), layers, g)
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
