"""The epilogues of the pipelined GEMM kernel where K is not split: QKV, residual, SwiGLU and LM head inside the kernel, at odd
and whole row tiles, one and several row blocks, column groups that end inside the matrix (an odd count of 16-column tiles in
the vocabulary and of gate/up pairs), few and many sums of squares per row, chains and both head dimensions."""
from types import SimpleNamespace

import pytest
import torch

pytestmark = pytest.mark.gpu

from harness import Pair, compare_step
from sssd_synth import uniform_int


# hidden, heads and widths so small that every K has one slice (fewer than 16 k-tiles), but for `ffn` 1104 (35 k-tiles: the
# down projection and its sums go through memory)
@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,vocab", [(256, 4, 2, 64, 432, 1040), (272, 6, 2, 64, 1104, 528), (384, 3, 1, 128, 48, 4112)])
@pytest.mark.parametrize("B,k", [(3, 10), (7, 6), (8, 9), (9, 15), (5, 31), (7, 25), (20, 24)])     # 33 .. 500 rows
def test_unsplit_epilogues_vs_oracle(hidden, nq, nkv, d, ffn, vocab, B, k):
    print(f"epilogues h={hidden} ffn={ffn} vocab={vocab} B={B} k={k}", flush=True)
    s = SimpleNamespace(name="edge", n_layers=2, hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=ffn, vocab=vocab,
                        rms_eps=1e-5, rope_base=10000.0)
    p = Pair(s, seed=31, max_batch=B, max_k=k, max_seq=96, unit_gains=False)
    lens = uniform_int(32, B * 64 + k, (B,), 0, 96 - k - 1)
    for b in range(B):
        p.prefill_random_kv(33, b, int(lens[b]), oracle_slot=b)
    tokens = uniform_int(34, B * 64 + k, (B, k + 1), 0, s.vocab - 1)
    ref = p.oracle.verify_step(tokens, lens.to(torch.int32), return_hidden=True)
    gpu = p.step(tokens, lens.to(torch.int32))
    compare_step(gpu, ref, tokens)
    herr = (gpu["hidden"] - ref["hidden"]).abs().max().item() / ref["hidden"].abs().max().item()
    assert herr < 5e-3      # a bf16 rounding of a new K or V element may fall the other way: 2^-9 of it
    p.ctx.sssd_verify_destroy()
