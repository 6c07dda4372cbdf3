"""Steps of up to 32 rows with a short K: one, two and four k-tiles per wave, on both sides of every line between them, K that ends
inside a k-tile, and waves with nothing but padding; the plain store and the fused epilogues."""
from types import SimpleNamespace

import pytest
import torch

pytestmark = pytest.mark.gpu

from harness import Pair, compare_step
from paper_2411_05894_amd import binding as sv
from sssd_synth import uniform_int
from test_gpu_gemm_pipeline import check


@pytest.mark.parametrize("K", [8, 32, 488, 512, 520, 1024, 1032, 1504, 2048, 2056, 4096])
@pytest.mark.parametrize("N,M", [(16, 1), (272, 5), (4128, 16), (96, 17), (528, 32)])
def test_short_k(N, K, M):
    assert sv.sssd_op_gemm_kernel_of(M, N, K) == "pgemm_kernel"
    check(N, K, M)


# QKV and LM head, residual and SwiGLU with two k-tiles per wave (17, 20 and 17 k-tiles; the down projection's 33 take four) and with
# four (33, 36, 33 and 47), one and two row tiles
@pytest.mark.parametrize("hidden,nq,ffn", [(528, 10, 1040), (1040, 18, 1504)])
@pytest.mark.parametrize("B,k", [(1, 4), (2, 7), (1, 16), (4, 7)])     # 5, 16, 17 and 32 rows
def test_fused_short_k(hidden, nq, ffn, B, k):
    print(f"fused short K h={hidden} ffn={ffn} B={B} k={k}", flush=True)
    s = SimpleNamespace(name="edge", n_layers=2, hidden=hidden, n_q_heads=nq, n_kv_heads=2, head_dim=64, ffn=ffn, vocab=1040, rms_eps=1e-5,
                        rope_base=10000.0)
    p = Pair(s, seed=35, max_batch=B, max_k=k, max_seq=96, unit_gains=False)
    lens = uniform_int(36, B * 64 + k, (B,), 0, 96 - k - 1)
    for b in range(B):
        p.prefill_random_kv(37, b, int(lens[b]), oracle_slot=b)
    tokens = uniform_int(38, B * 64 + k, (B, k + 1), 0, s.vocab - 1)
    ref = p.oracle.verify_step(tokens, lens.to(torch.int32), return_hidden=True)
    gpu = p.step(tokens, lens.to(torch.int32))
    compare_step(gpu, ref, tokens)
    herr = (gpu["hidden"] - ref["hidden"]).abs().max().item() / ref["hidden"].abs().max().item()
    assert herr < 5e-3      # a bf16 rounding of a new K or V element may fall the other way: 2^-9 of it
    p.ctx.sssd_verify_destroy()


# Workgroups with two tiles beside those with one, three beside two, one each and none to spare; whole and split K, one and two row tiles
@pytest.mark.parametrize("tiles,K", [(256, 64), (257, 1024), (259, 1000), (515, 2048), (129, 4128), (131, 2056)])
@pytest.mark.parametrize("M", [5, 16, 20])
def test_uneven_tiles(tiles, K, M):
    N = 16 * tiles
    assert sv.sssd_op_gemm_kernel_of(M, N, K) == "pgemm_kernel"
    check(N, K, M)


# The largest unsplit K of one, two, four, seven and eight k-tiles per wave, and K just past it (1040, the two-tile form's, above; past 4096
# K is split): the row scales of the second layer add up a sum of squares per 16 columns, as many as a row of these widths has.  3568
# ends inside its last k-tile.
@pytest.mark.parametrize("hidden", [512, 528, 1024, 2048, 2064, 3568, 3584, 3600, 4096, 4112])
@pytest.mark.parametrize("B,k", [(1, 4), (2, 7), (2, 12)])     # 5, 16 and 26 rows
def test_row_scales_of_the_widest_rows(hidden, B, k):
    print(f"row scales h={hidden} B={B} k={k}", flush=True)
    s = SimpleNamespace(name="edge", n_layers=2, hidden=hidden, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=144, vocab=528, rms_eps=1e-5,
                        rope_base=10000.0)
    p = Pair(s, seed=75, max_batch=B, max_k=k, max_seq=64, unit_gains=False)
    lens = uniform_int(76, B * 64 + k, (B,), 0, 64 - k - 1)
    for b in range(B):
        p.prefill_random_kv(77, b, int(lens[b]), oracle_slot=b)
    tokens = uniform_int(78, B * 64 + k, (B, k + 1), 0, s.vocab - 1)
    ref = p.oracle.verify_step(tokens, lens.to(torch.int32), return_hidden=True)
    gpu = p.step(tokens, lens.to(torch.int32))
    compare_step(gpu, ref, tokens)
    herr = (gpu["hidden"] - ref["hidden"]).abs().max().item() / ref["hidden"].abs().max().item()
    assert herr < 5e-3      # a bf16 rounding of a new K or V element may fall the other way: 2^-9 of it
    p.ctx.sssd_verify_destroy()
