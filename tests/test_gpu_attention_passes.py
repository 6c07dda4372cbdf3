"""How many row tiles an attention workgroup takes in a pass: four tiles as one pass of four and two of two, ten to fifteen in
passes of four, three and two, on both sides of each line between them (B x kv heads decides), short and long sequences, lengths
around a block and a segment.  Reference: softmax in 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2411_05894_amd import binding as sv
from sssd_synth import normal_bf16
from test_gpu_attention_segments import DEV, attention_context, reference

CASES = [  # shape, k, lens, max_seq
    ("8b", 12, [2047], 4096),                                                   # four tiles, the last one of four rows: two of two
    ("8b", 15, [0, 33, 255, 1100, 3000], 3100),                                 # B = 5: two of two
    ("8b", 15, [0, 33, 255, 256, 1100, 3000], 3100),                            # B = 6: one of four
    ("8b", 12, [90 * i for i in range(16)], 1500),                              # B = 16: two of two
    ("8b", 13, [60 * i for i in range(17)], 1100),                              # B = 17: one of four
    ("70b", 7, [31, 700], 2000),                                                # eight query rows per node
    ("tiny", 31, [5, 300, 1200], 1300),                                         # head size 64
    ("70b", 18, [1500], 1600),                                                  # ten tiles: four of three, two tiles to spare
    ("70b", 18, [17, 400, 900], 1000),                                          # B = 3: five of two
    ("70b", 20, [17, 400, 900], 1000),                                          # eleven: three of four
    ("70b", 23, [0, 31, 64, 200, 288, 300, 511, 640], 700),                     # twelve, B = 8: four of three
    ("70b", 23, [40 * i for i in range(10)], 500),                              # B = 10: three of four
    ("70b", 18, [40 * i for i in range(11)], 500),                              # B = 11: four of three, two workgroups per compute unit
    ("70b", 28, [300, 700], 800),                                               # fifteen: five of three
]


@pytest.mark.parametrize("shape_name,k,lens,max_seq", CASES)
def test_tiles_of_a_pass(shape_name, k, lens, max_seq):
    B, sq = len(lens), k + 1
    s, ctx = attention_context(shape_name, B, k, max_seq)
    grp = s.n_q_heads // s.n_kv_heads
    q = (normal_bf16(61, k + 1, (B, sq, s.n_q_heads, s.head_dim), 1.0, device=DEV).float() * 1.28).contiguous()
    kv = []
    for b, n in enumerate(lens):
        kv.append([normal_bf16(62, 2 * b + i, (s.n_kv_heads, n + sq, s.head_dim), 1.0, device=DEV) for i in range(2)])
        ctx.sssd_kv_import(0, b, 0, *kv[b])
    out = torch.empty(B, sq, s.n_q_heads * s.head_dim, dtype=torch.float32, device=DEV)
    print(f"attention passes {shape_name} k={k} B={B}", flush=True)
    ctx.sssd_op_attention(0, q, torch.tensor(lens, dtype=torch.int32, device=DEV), out)
    assert ctx.sssd_verify_sync() == 0
    got = out.view(B, sq, s.n_q_heads, s.head_dim)
    for b in range(B):
        # q and the probabilities enter the MFMAs as bf16 hi+lo pairs (~2^-17 relative); outputs are O(1)
        assert (got[b] - reference(q[b], *kv[b], lens[b], grp)).abs().max().item() <= 1e-4, b
