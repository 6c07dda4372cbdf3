"""The attention kernel's division of work: waves with no block, one block and more than 64 (the pages of the next chunk are read
ahead), whole and partial rounds of the four waves, every count of row tiles and passes with tiles to spare, new rows that
straddle a block, maxima that outgrow the running reference in later blocks; plain runs of pages and shuffled tables.
Reference: softmax in 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2411_05894_amd import binding as sv
from sssd_synth import normal_bf16
from test_gpu_attention_segments import DEV, attention_context, reference

CASES = [  # shape, k, lens, max_seq
    ("tiny", 4, [9100, 20, 300] + [40] * 125, 9200),                    # one segment of 285 blocks
    ("8b", 3, [8170 + 2 * i for i in range(32)], 8300),                 # 256 and 257 blocks, 64 and 65 for the first wave
    ("8b", 7, [0, 1, 31, 32, 33, 60, 64, 95, 96, 100, 127, 128, 129], 160),
    ("8b", 8, [240, 255, 256, 257, 288, 511, 512, 513, 700], 800),      # around one segment of eight blocks, three row tiles
    ("8b", 17, [20, 700, 2047], 2100),                                  # five row tiles: two passes of three
    ("8b", 22, [33, 1000], 1100),                                       # six
    ("70b", 13, [90, 1500], 1600),                                      # seven: two passes of four
    ("70b", 17, [500], 600),                                            # nine: three passes of three
    ("70b", 31, [300, 2000], 2100),                                     # sixteen: four passes of four
    ("tiny", 31, [5, 200, 1200], 1300),                                 # head size 64
]


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("shape_name,k,lens,max_seq", CASES)
def test_waves_and_passes(shape_name, k, lens, max_seq, paged):
    B, sq = len(lens), k + 1
    s, ctx = attention_context(shape_name, B, k, max_seq)
    grp = s.n_q_heads // s.n_kv_heads
    if paged:
        _, bps, n_pages = sv.sssd_kv_geometry(ctx.cfg)
        g = torch.Generator().manual_seed(B * 64 + k)
        ctx.sssd_kv_set_block_table(torch.randperm(n_pages, generator=g).to(torch.int32).view(B, bps).to(DEV))
    # whole bf16 values (no lo part), four times as large as usual: scores of up to 20 whose maximum keeps moving
    q = (normal_bf16(51, k + 1, (B, sq, s.n_q_heads, s.head_dim), 1.0, device=DEV).float() * 4.0).contiguous()
    kv = []
    for b, n in enumerate(lens):
        kv.append([normal_bf16(52, 2 * b + i, (s.n_kv_heads, n + sq, s.head_dim), 1.0, device=DEV) for i in range(2)])
        if n > 64:
            kv[b][0][:, n // 2:] *= 2.0                                 # later rows score twice as high
        ctx.sssd_kv_import(0, b, 0, *kv[b])
    out = torch.empty(B, sq, s.n_q_heads * s.head_dim, dtype=torch.float32, device=DEV)
    print(f"attention waves {shape_name} k={k} B={B} paged={paged}", flush=True)
    ctx.sssd_op_attention(0, q, torch.tensor(lens, dtype=torch.int32, device=DEV), out)
    assert ctx.sssd_verify_sync() == 0
    got = out.view(B, sq, s.n_q_heads, s.head_dim)
    for b in range(B):
        # probabilities and results are bf16 hi + lo (2^-17 of values of up to 5), scores are fp32 sums of 64 or 128 products of
        # up to 40 in all (2^-21 absolute, as much in a probability): 4e-5 + 5e-6, twice that
        assert (got[b] - reference(q[b], *kv[b], lens[b], grp)).abs().max().item() <= 1e-4, b
