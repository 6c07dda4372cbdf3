"""Parity at the full sizes of the benchmark configurations (Llama-3-8B and 70B shapes),
in the launch configuration bench.py times.  The oracle cannot run whole batches of
these in seconds, so it recomputes SAMPLED sequences completely (every layer, every
logit of their k+1 rows); sequences are independent, so a sampled sequence of the
batched GPU step must match the oracle run on that sequence alone."""
import os
import sys
import time

import pytest
import torch

pytestmark = pytest.mark.gpu

import oracle
from paper_2411_05894_amd import binding as sv
from sssd_synth import (MODEL_SHAPES, TensorId, global_weight_specs, layer_weight_specs, make_kv_prefill,
                        make_weight, uniform_int)

sys.path.insert(0, os.path.dirname(__file__))
from harness import LOGIT_TOL, Pair, check_exempt, compare_step, compare_tree_step, step_tree  # noqa: E402

DEV = "cuda:0"
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def progress(msg):
    """Progress lines for long tests: printed, and appended to a file the harness can watch."""
    print(msg, flush=True)
    try:
        os.makedirs(os.path.join(ROOT, "gpurun_out"), exist_ok=True)
        with open(os.path.join(ROOT, "gpurun_out", "progress.log"), "a") as f:
            f.write(f"{time.strftime('%H:%M:%S')} {msg}\n")
    except OSError:
        pass


@pytest.fixture(scope="module")
def pair_8b():
    """8B-shaped weights (seed 3) once per module: capacity B=32, k<=16, 4128 rows per sequence."""
    progress("8b: generating weights")
    p = Pair(MODEL_SHAPES["8b"], seed=3, max_batch=32, max_k=16, max_seq=4096 + 17, oracle_batch=2)
    progress("8b: ready")
    yield p
    p.ctx.sssd_verify_destroy()


@pytest.mark.timeout(300)
def test_cfg2_8b_b1_ctx2048_k_sweep(pair_8b):
    """Config 2: B=1, KV context 2048 (random N(0,1) prefill), uniform-random drafts.  The oracle
    runs k=16 once; rows 0..k of that pass are the reference for every smaller k (row j never
    depends on later rows)."""
    p, s = pair_8b, pair_8b.shape
    p.prefill_random_kv(4, 0, 2048, oracle_slot=0)
    tokens = uniform_int(4, TensorId.TOKENS, (1, 17), 0, s.vocab - 1)
    lens = torch.tensor([2048], dtype=torch.int32)
    t = time.time()
    ref = p.oracle.verify_step(tokens, lens)
    progress(f"cfg2: oracle k=16 took {time.time() - t:.1f}s")
    ex_all, rows_all = 0, 0
    for k in (16, 8, 3, 0):
        tk = tokens[:, : k + 1].contiguous()
        sub = {"logits": ref["logits"][:, : k + 1], "that": ref["that"][:, : k + 1]}
        a, n = oracle.accept(tk[0].tolist(), sub["that"][0].tolist())
        sub["accepted_len"], sub["next_token"] = torch.tensor([a]), torch.tensor([n])
        gpu = p.step(tk, lens)
        err, ex, rows = compare_step(gpu, sub, tk)
        progress(f"cfg2 k={k}: max logit err {err:.2e}, exempt rows {ex}/{rows}")
        ex_all, rows_all = ex_all + ex, rows_all + rows
    check_exempt(ex_all, rows_all)


@pytest.mark.timeout(300)
def test_cfg2_shape_draft_tree_k16(pair_8b):
    """The 8B shape at B=1, context 2048, with the 16 drafts arranged as a seeded random TREE
    (Sec. 3.1: the candidates are verified as a tree under its attention mask) instead of a chain."""
    p, s = pair_8b, pair_8b.shape
    k = 16
    p.prefill_random_kv(4, 0, 2048, oracle_slot=0)
    tokens = uniform_int(4, TensorId.TOKENS, (1, k + 1), 0, s.vocab - 1)
    raw = uniform_int(4, TensorId.LENS, (k + 1,), 0, 1 << 20).tolist()
    parents = torch.tensor([[0] + [raw[i] % i for i in range(1, k + 1)]], dtype=torch.int32)
    lens = torch.tensor([2048], dtype=torch.int32)
    t = time.time()
    ref = p.oracle.verify_step_tree(tokens, parents, lens, compact=False)
    # plant the oracle's own choice after the root in one child of the root: that child's row is unchanged
    # (its token was not an input of the root row), but the walk now accepts at least one draft
    kid = max(c for c in range(1, k + 1) if int(parents[0, c]) == 0)
    tokens[0, kid] = int(ref["that"][0, 0])
    ref = p.oracle.verify_step_tree(tokens, parents, lens, compact=False)
    progress(f"cfg2-tree: two oracle passes took {time.time() - t:.1f}s, tree {parents[0].tolist()}")
    gpu = step_tree(p, tokens, parents, lens)
    err, ex, rows = compare_tree_step(gpu, ref, tokens, parents)
    progress(f"cfg2-tree k={k}: max logit err {err:.2e}, exempt rows {ex}/{rows}, accepted {int(ref['accepted_len'][0])}")
    check_exempt(ex, rows)
    assert int(ref["accepted_len"][0]) >= 1


@pytest.mark.timeout(300)
def test_cfg2_shape_paged_cache_is_bit_identical(pair_8b):
    """The 8B shape at B=1, context 2048, k=8 with the sequence's 65 blocks scattered over the pool by a
    block table: the logits must equal the contiguous run's bit for bit (same kernels, same launch
    configuration; only the page addresses differ)."""
    p, s = pair_8b, pair_8b.shape
    k = 8
    tokens = uniform_int(4, TensorId.TOKENS, (1, k + 1), 0, s.vocab - 1)
    lens = torch.tensor([2048], dtype=torch.int32)
    p.prefill_random_kv(4, 0, 2048)
    a = p.step(tokens, lens)["logits"].clone()
    rows, bps, n_pages = sv.sssd_kv_geometry(p.cfg)
    keys = uniform_int(7, 1, (n_pages,), 0, 1 << 30).tolist()
    perm = sorted(range(n_pages), key=lambda i: (keys[i], i))
    table = torch.tensor(perm[: 32 * bps], dtype=torch.int32).view(32, bps).to(DEV)
    try:
        p.ctx.sssd_kv_set_block_table(table)
        p.prefill_random_kv(4, 0, 2048)                   # the same rows, imported through the table
        b = p.step(tokens, lens)["logits"]
        assert torch.equal(a, b)
        progress(f"cfg2-paged: {bps} blocks of sequence 0 scattered over {n_pages} pages, logits bit-identical")
    finally:
        p.ctx.sssd_kv_set_block_table(None)
        p.prefill_random_kv(4, 0, 2048)                   # pages of other sequences were overwritten: restore slot 0


@pytest.mark.timeout(300)
def test_8b_shape_split_k_sums_repeat_bit_for_bit(pair_8b):
    """Steps whose GEMMs split K over workgroups (k=8: the down projection; k=16: every GEMM) hand the
    slices from one workgroup to another inside a launch.  200 repetitions of the same step must give
    the same logits bit for bit: a slice read before it was complete would show up as a difference."""
    p, s = pair_8b, pair_8b.shape
    p.prefill_random_kv(4, 0, 2048)
    lens = torch.tensor([2048], dtype=torch.int32)
    for k in (8, 16):
        tokens = uniform_int(76, 1 + k, (1, k + 1), 0, s.vocab - 1)
        t = tokens.to(p.dev, torch.int32).contiguous()
        ln = lens.to(p.dev, torch.int32)
        acc = torch.empty(1, dtype=torch.int32, device=p.dev)
        nxt = torch.empty(1, dtype=torch.int32, device=p.dev)
        first, bad = None, 0
        for rep in range(200):
            p.ctx.sssd_verify_step(t, ln, acc, nxt)
            cur = p.logits[: k + 1]
            if first is None:
                first = cur.clone()
            else:
                bad += int(not torch.equal(first, cur))
        assert p.ctx.sssd_verify_sync() == 0
        assert bad == 0, (k, bad)
        progress(f"split-K repeat k={k}: 200 steps, logits identical every time")


@pytest.mark.timeout(300)
def test_cfg3_8b_b32_ragged_k4(pair_8b):
    """Config 3: B=32, context lengths uniform in [1024, 4096], k=4.  Sequences 5 and 31 are
    recomputed by the oracle."""
    p, s = pair_8b, pair_8b.shape
    B, k = 32, 4
    lens = uniform_int(5, TensorId.LENS, (B,), 1024, 4096)
    sample = [5, 31]
    for b in range(B):
        p.prefill_random_kv(5, b, int(lens[b]), oracle_slot=sample.index(b) if b in sample else None)
    progress(f"cfg3: prefilled, lens[sample]={[int(lens[b]) for b in sample]}")
    tokens = uniform_int(5, TensorId.TOKENS, (B, k + 1), 0, s.vocab - 1)
    gpu = p.step(tokens, lens)
    t = time.time()
    ref = p.oracle.verify_step(tokens[sample].contiguous(), lens[sample].contiguous())
    progress(f"cfg3: oracle on 2 sequences took {time.time() - t:.1f}s")
    err, ex, rows = compare_step(gpu, ref, tokens, seqs=sample)
    progress(f"cfg3: max logit err {err:.2e}, exempt rows {ex}/{rows}")
    check_exempt(ex, rows)


@pytest.mark.timeout(300)
def test_cfg4_8b_b4_ctx32768_k8():
    """Config 4: B=4, KV context 32768, k=8 (attention-dominated).  Sequence 2 is recomputed."""
    s = MODEL_SHAPES["8b"]
    B, k, ctx = 4, 8, 32768
    progress("cfg4: generating weights")
    p = Pair(s, seed=3, max_batch=B, max_k=k, max_seq=ctx + k + 1, oracle_batch=1)
    for b in range(B):
        p.prefill_random_kv(6, b, ctx, oracle_slot=0 if b == 2 else None)
    progress("cfg4: prefilled")
    tokens = uniform_int(6, TensorId.TOKENS, (B, k + 1), 0, s.vocab - 1)
    lens = torch.full((B,), ctx, dtype=torch.int32)
    gpu = p.step(tokens, lens)
    t = time.time()
    ref = p.oracle.verify_step(tokens[2:3].contiguous(), lens[2:3].contiguous())
    progress(f"cfg4: oracle on 1 sequence took {time.time() - t:.1f}s")
    err, ex, rows = compare_step(gpu, ref, tokens, seqs=[2])
    progress(f"cfg4: max logit err {err:.2e}, exempt rows {ex}/{rows}")
    check_exempt(ex, rows)
    p.ctx.sssd_verify_destroy()


@pytest.mark.timeout(900)
def test_cfg5_70b_b16_ctx2048_k8():
    """Config 5: Llama-3-70B shape (141 GB of bf16 weights, reordered in place), B=16, context
    2048, k=8.  The oracle recomputes rows 0..4 of sequence 7 (row j never depends on later
    rows), streaming the weights layer by layer from the device copy before the library
    reorders it."""
    s = MODEL_SHAPES["70b"]
    B, k, ctx, seed, sample, k_ref = 16, 8, 2048, 6, 7, 4
    dev = torch.device(DEV)
    free, _ = torch.cuda.mem_get_info()
    if free < 170e9:
        pytest.skip("needs ~165 GB of free device memory")
    max_seq = ctx + k + 1
    tokens = uniform_int(seed, TensorId.TOKENS, (B, k + 1), 0, s.vocab - 1)
    lens = torch.full((B,), ctx, dtype=torch.int32)
    g = {n: make_weight(seed, n, tid, shp, device=dev) for n, tid, shp in global_weight_specs(s)}
    om = oracle.OracleModel(s, [None] * s.n_layers, {n: t.cpu() for n, t in g.items()}, 1, max_seq)
    tok_ref = tokens[sample: sample + 1, : k_ref + 1].contiguous()
    x = om.embed(tok_ref)
    layers = []
    t0 = time.time()
    for l in range(s.n_layers):
        lw = {n: make_weight(seed, n, TensorId.layer(l, slot), shp, device=dev) for n, slot, shp in layer_weight_specs(s)}
        layers.append(lw)
        K, V = make_kv_prefill(seed * 1000 + sample, l, (s.n_kv_heads, ctx, s.head_dim), device=dev)
        om.K[l, 0, :, :ctx] = K.cpu()
        om.V[l, 0, :, :ctx] = V.cpu()
        om.layers[l] = {n: t.cpu() for n, t in lw.items()}
        om.layer_verify(l, x, lens[sample: sample + 1], 1, k_ref)
        om.layers[l] = None
        if l % 8 == 7:
            progress(f"cfg5: oracle through layer {l} ({time.time() - t0:.0f}s)")
    ref_logits = om.lm_head(x).view(1, k_ref + 1, -1)
    that = torch.tensor([[oracle.argmax(ref_logits[0, j]) for j in range(k_ref + 1)]], dtype=torch.int32)
    a, n = oracle.accept(tok_ref[0].tolist(), that[0].tolist())
    ref = {"logits": ref_logits, "that": that, "accepted_len": torch.tensor([a]), "next_token": torch.tensor([n])}
    del om
    progress("cfg5: oracle done; initialising the library in place")
    ctx_ = sv.VerifyContext(sv.make_config(s, B, k, max_seq), layers, g, in_place=True)
    for b in range(B):
        for l in range(s.n_layers):
            K, V = make_kv_prefill(seed * 1000 + b, l, (s.n_kv_heads, ctx, s.head_dim), device=dev)
            ctx_.sssd_kv_import(l, b, 0, K, V)
        torch.cuda.synchronize()
    progress("cfg5: prefilled")
    logits = torch.zeros(B * (k + 1), s.vocab, dtype=torch.float32, device=dev)
    fused = torch.full((B * (k + 1),), -1, dtype=torch.int32, device=dev)
    ctx_.sssd_debug_logits(logits)
    ctx_.sssd_debug_argmax(fused)
    acc = torch.empty(B, dtype=torch.int32, device=dev)
    nxt = torch.empty(B, dtype=torch.int32, device=dev)
    # every k the benchmark sweeps at this configuration beyond 0 (k = 0 follows): M = 144, 80 and 48 rows
    for kk in (8, 4, 2):
        tk = tokens[:, : kk + 1].contiguous()
        n_ref = min(kk, k_ref) + 1
        sub = {"logits": ref_logits[:, :n_ref], "that": that[:, :n_ref]}
        a, n = oracle.accept(tk[sample, :n_ref].tolist(), that[0, :n_ref].tolist())
        sub["accepted_len"], sub["next_token"] = torch.tensor([a]), torch.tensor([n])
        ctx_.sssd_verify_step(tk.to(dev), lens.to(dev), acc, nxt)
        assert ctx_.sssd_verify_sync() == 0
        M = B * (kk + 1)
        gpu = {"logits": logits[:M].cpu().view(B, kk + 1, -1), "that": fused[:M].cpu().view(B, kk + 1),
               "accepted_len": acc.cpu(), "next_token": nxt.cpu()}
        err, ex, rows = compare_step(gpu, sub, tk, seqs=[sample])
        progress(f"cfg5 k={kk}: max logit err {err:.2e}, exempt rows {ex}/{rows}")
        check_exempt(ex, rows)
        # every sequence, not only the sampled one: the fused arg-max must be the arg-max of the step's logits
        assert torch.equal(gpu["that"], gpu["logits"].argmax(-1).to(torch.int32))
    # k = 0 (16 rows: QKV and O on the small-step kernel with K split over workgroups and summed by the last
    # of them to arrive, the larger matrices on the pipelined one): 30 repetitions must give the same logits bit for bit
    t1 = tokens[:, :1].contiguous().to(dev)
    first, bad = None, 0
    for rep in range(30):
        ctx_.sssd_verify_step(t1, lens.to(dev), acc, nxt)
        cur = logits[:B]
        if first is None:
            first = cur.clone()
        else:
            bad += int(not torch.equal(first, cur))
    assert ctx_.sssd_verify_sync() == 0
    assert bad == 0, bad
    e0 = float((first[sample].cpu() - ref_logits[0, 0]).abs().max())
    progress(f"cfg5 k=0: 30 steps identical, row 0 of sequence {sample} within {e0:.2e} of the oracle")
    assert e0 < 2e-2
    ctx_.sssd_verify_destroy()
