"""GPU parity of target-only speculative sampling (Sec. 4.4) against the fp64 oracle: the row sampler
on its own (same logits on both sides, so only the fp32 arithmetic of the weights differs), its tie
rules, its sampling frequencies, and the sampled tree step of the tiny model."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from harness import LOGIT_TOL, Pair
from paper_2411_05894_amd import binding as sv
from sssd_synth import MODEL_SHAPES, normal_bf16, uniform_int

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# A decision whose relative distance to its threshold is below this is exempt: the kernel sums fp32
# weights (relative error of a few 1e-7 each: exp2 of a product rounded twice; then accumulated exactly
# in 32.32 fixed point, 2.3e-10 resolution).
MARGIN_SAME_LOGITS = 1e-6


def say(msg):
    print(msg, flush=True)


def uniforms(seed, n):
    return (uniform_int(seed, 1, (n,), 0, (1 << 24) - 1).float() / float(1 << 24)).contiguous()


def check_rows(logits, params, u, min_checked):
    """Kernel vs oracle on every row; returns (checked, exempt)."""
    got = sv.sssd_op_sample(logits.to(DEV), params, u.to(DEV)).cpu().tolist()
    wide = sv.sssd_op_sample_wide(logits.to(DEV), params, u.to(DEV)).cpu().tolist()
    assert wide == got, "several workgroups per row must draw exactly the tokens of one workgroup per row"
    checked = exempt = 0
    for r in range(logits.shape[0]):
        want, margin = oracle.sample_row(logits[r], params.temperature, params.top_k, params.top_p, float(u[r]),
                                         w_noise=MARGIN_SAME_LOGITS)
        if margin < MARGIN_SAME_LOGITS:
            exempt += 1
            continue
        assert got[r] == want, f"row {r}: sampled {got[r]}, oracle {want} (margin {margin:.2e})"
        checked += 1
    assert checked >= min_checked
    return checked, exempt


@pytest.mark.parametrize("V,rows", [(1024, 48), (128256, 12), (1000, 16), (77, 8)])
def test_row_sampler_vs_oracle(V, rows):
    logits = (normal_bf16(101, V, (rows, V), 1.0).float() * 2.5 +
              2.0 ** -9 * normal_bf16(102, V, (rows, V), 1.0).float()).contiguous()
    u = uniforms(103, rows)
    for T, k, p in ((1.0, 0, 1.0), (0.6, 0, 0.95), (0.7, 20, 0.8), (1.5, 50, 1.0), (0.9, 1, 1.0), (1.0, 0, 0.05),
                    (1.2, 0, 0.9), (0.3, 5, 0.5)):
        params = sv.SamplingParams(T, k, p)
        # with 128256 tokens a flat distribution has inverse-CDF steps of ~8e-6: more rows land within the exemption
        c, e = check_rows(logits, params, u, rows - 2 if V <= 4096 else rows // 3)
        say(f"sampler V={V} T={T} top_k={k} top_p={p}: {c} rows equal, {e} exempt")


def test_ties_are_resolved_by_token_id():
    """Quantised logits: thousands of exact ties at every threshold."""
    V, rows = 4096, 32
    logits = (uniform_int(104, 1, (rows, V), 0, 7).float() * 0.5).contiguous()      # 8 distinct values
    u = uniforms(105, rows)
    for T, k, p in ((1.0, 100, 1.0), (1.0, 0, 0.3), (0.8, 700, 0.6), (1.0, 513, 0.999), (1.0, 4095, 1.0)):
        check_rows(logits, sv.SamplingParams(T, k, p), u, rows - 2)
    # all logits equal: uniform over the first top_k ids
    flat = torch.zeros(4, 1024)
    got = sv.sssd_op_sample(flat.to(DEV), sv.SamplingParams(1.0, 10, 1.0), torch.tensor([0.0, 0.35, 0.95, 0.999]).to(DEV))
    assert got.cpu().tolist() == [0, 3, 9, 9]


def test_sampling_frequencies_match_the_target_distribution():
    V, N = 1024, 8192
    z = normal_bf16(106, 1, (V,), 1.0).float() * 2.0
    logits = z.repeat(N, 1).contiguous()
    u = ((torch.arange(N, dtype=torch.float64) + 0.5) / N).float()
    for T, k, p in ((1.0, 0, 1.0), (0.7, 20, 0.8), (0.6, 0, 0.95)):
        got = sv.sssd_op_sample(logits.to(DEV), sv.SamplingParams(T, k, p), u.to(DEV)).cpu().numpy()
        d = oracle.target_distribution(z, T, k, p)
        counts = np.bincount(got, minlength=V)
        assert set(np.nonzero(counts)[0]) <= set(np.nonzero(d)[0])                  # nothing outside S
        assert np.abs(counts / N - d).max() <= 2.0 / N + 1e-6
        again = sv.sssd_op_sample(logits.to(DEV), sv.SamplingParams(T, k, p), u.to(DEV)).cpu().numpy()
        assert np.array_equal(got, again)                                            # deterministic


def test_sampled_tree_step_vs_oracle():
    s = MODEL_SHAPES["tiny"]
    B, k = 3, 7
    p = Pair(s, seed=51, max_batch=B, max_k=k, max_seq=96, unit_gains=False)
    ctxs = [3, 20, 60]
    for b in range(B):
        p.prefill_random_kv(52, b, ctxs[b], oracle_slot=b)
    lens = torch.tensor(ctxs, dtype=torch.int32)
    raw = uniform_int(53, 1, (B, k + 1), 0, 1 << 20).tolist()
    parents = torch.tensor([[0] + [raw[b][i] % i for i in range(1, k + 1)] for b in range(B)], dtype=torch.int32)
    T, top_k, top_p = 0.7, 20, 0.8
    u = uniforms(54, B * (k + 1)).view(B, k + 1)
    tokens = uniform_int(55, 1, (B, k + 1), 0, s.vocab - 1)
    # plant, level by level, the oracle's own sampled token in one child so that the walk accepts drafts
    cur = [0] * B
    for _ in range(3):
        ref = p.oracle.verify_step_tree_sampled(tokens, parents, lens, T, top_k, top_p, u, compact=False)
        for b in range(B):
            kids = [c for c in range(1, k + 1) if int(parents[b, c]) == cur[b]]
            if kids:
                tokens[b, kids[-1]] = int(ref["sampled"][b, cur[b]])
                cur[b] = kids[-1]
    ref = p.oracle.verify_step_tree_sampled(tokens, parents, lens, T, top_k, top_p, u, compact=False)
    scratch = torch.empty(B * (k + 1), s.vocab, dtype=torch.float32, device=DEV)
    acc = torch.empty(B, dtype=torch.int32, device=DEV)
    nxt = torch.empty(B, dtype=torch.int32, device=DEV)
    path = torch.empty(B, k + 1, dtype=torch.int32, device=DEV)
    p.ctx.sssd_verify_step_tree_sampled(tokens.to(DEV), parents.to(DEV), lens.to(DEV), sv.SamplingParams(T, top_k, top_p),
                                        u.to(DEV), scratch, acc, nxt, path)
    assert p.ctx.sssd_verify_sync() == 0
    logits = scratch.cpu().view(B, k + 1, -1)
    err = (logits - ref["logits"]).abs().max().item()
    assert err <= LOGIT_TOL
    assert torch.equal(p.logits[: B * (k + 1)].cpu().view(B, k + 1, -1), logits)      # the parity aid sees the same logits
    # The library's logits differ from the oracle's by `err`, which moves every weight by up to err / T
    # relative: decisions closer than that to a threshold are exempt.
    noise = 4 * err / T + 1e-5
    accepted = 0
    for b in range(B):
        n = int(acc[b])
        g_path = path[b].cpu().tolist()
        # the library's own walk is consistent with its own samples
        mine = [oracle.sample_row(logits[b, j], T, top_k, top_p, float(u[b, j]), w_noise=MARGIN_SAME_LOGITS)
                for j in range(k + 1)]
        drawn = p.that[b * (k + 1): (b + 1) * (k + 1)].cpu().tolist()      # the step's own per-row draws
        for j in range(k + 1):
            if mine[j][1] > MARGIN_SAME_LOGITS:
                assert drawn[j] == mine[j][0], f"row ({b},{j}): step drew {drawn[j]}, oracle on the same logits {mine[j][0]}"
        robust = [oracle.sample_row(ref["logits"][b, i], T, top_k, top_p, float(u[b, i]), w_noise=noise, logit_noise=2 * err)[1]
                  for i in ref["path"][b]]
        decided = all(m > noise for m in robust)
        if decided:
            assert g_path[: n + 1] == ref["path"][b] and int(nxt[b]) == int(ref["next_token"][b])
            accepted += n
        own_safe = all(mine[i][1] > MARGIN_SAME_LOGITS for i in g_path[: n + 1])
        if own_safe:
            cur_node = 0
            for i in range(1, n + 1):
                assert int(parents[b, g_path[i]]) == cur_node and int(tokens[b, g_path[i]]) == mine[cur_node][0]
                cur_node = g_path[i]
            assert int(nxt[b]) == mine[cur_node][0]
        assert all(x == -1 for x in g_path[n + 1:])
    # the same step again: the sampler's workgroup clusters must find their counters as the first call left them
    acc2, nxt2, path2 = torch.empty_like(acc), torch.empty_like(nxt), torch.empty_like(path)
    for _ in range(3):
        p.ctx.sssd_verify_step_tree_sampled(tokens.to(DEV), parents.to(DEV), lens.to(DEV), sv.SamplingParams(T, top_k, top_p),
                                            u.to(DEV), scratch, acc2, nxt2, path2)
        assert p.ctx.sssd_verify_sync() == 0
        assert torch.equal(acc, acc2) and torch.equal(nxt, nxt2) and torch.equal(path, path2)
    say(f"sampled tree step: logit err {err:.2e}, accepted {ref['accepted_len'].tolist()}")
    assert int(ref["accepted_len"].sum()) >= B


@pytest.mark.parametrize("V,rows", [(128256, 1), (128256, 9), (128256, 33), (128256, 128), (128256, 200), (4100, 5), (52, 3)])
def test_clustered_sampler_equals_the_single_workgroup_sampler(V, rows):
    """Row counts from one (16 workgroups per row) to more rows than compute units/2 (one each), vocabularies
    from fewer tokens than workgroups to the full size, logits with many exact ties (values on a coarse grid)
    and without; every parameter combination must give identical tokens from both forms, twice in a row
    (the second call finds the first call's scratch contents)."""
    grid = (uniform_int(71, V + rows, (rows, V), -40, 40).float() / 8.0)            # ties everywhere
    smooth = normal_bf16(72, V + rows, (rows, V), 1.0).float() * 2.5
    u = uniforms(73, rows)
    for logits in (grid, smooth):
        z = logits.to(DEV).contiguous()
        for T, k, p in ((0.6, 0, 0.95), (0.7, 20, 0.8), (1.0, 50, 1.0), (1.0, 0, 1.0), (1.5, 3, 0.3), (0.3, 0, 0.05)):
            sp = sv.SamplingParams(T, k, p)
            one = sv.sssd_op_sample(z, sp, u.to(DEV)).cpu()
            for _ in range(2):
                many = sv.sssd_op_sample_wide(z, sp, u.to(DEV)).cpu()
                assert torch.equal(one, many), (V, rows, T, k, p)
            assert int(one.min()) >= 0 and int(one.max()) < V
    say(f"clustered sampler V={V} rows={rows}: identical tokens in 12 settings")


def test_sampling_argument_checks():
    z = torch.zeros(2, 64, device=DEV)
    u = torch.zeros(2, device=DEV)
    # the clustered form wants its scratch: too little of it is refused before anything is launched
    need = sv.lib().sssd_op_sample_scratch_bytes(2)
    assert need > 0 and sv.lib().sssd_op_sample_scratch_bytes(100000) == 0
    small = torch.empty(16, dtype=torch.uint8, device=DEV)
    out = torch.empty(2, dtype=torch.int32, device=DEV)
    import ctypes as C
    ok = sv.SamplingParams(1.0, 0, 1.0)
    assert sv.lib().sssd_op_sample_wide(z.data_ptr(), 2, 64, C.byref(ok), u.data_ptr(), out.data_ptr(), small.data_ptr(), 16, None) == sv.SSSD_ECAPACITY
    assert sv.lib().sssd_op_sample_wide(z.data_ptr(), 2, 64, C.byref(ok), u.data_ptr(), out.data_ptr(), None, 0, None) == sv.SSSD_ECAPACITY
    for bad in (sv.SamplingParams(0.0, 0, 1.0), sv.SamplingParams(1.0, -1, 1.0), sv.SamplingParams(1.0, 0, 0.0),
                sv.SamplingParams(1.0, 0, 1.5)):
        with pytest.raises(sv.SssdError):
            sv.sssd_op_sample(z, bad, u)


@pytest.mark.parametrize("V,rows", [(4099, 1), (4099, 17), (8192, 129), (32004, 9)])   # clusters of 16, 8, 1 and 16 workgroups
def test_list_selections_at_their_edges(V, rows):
    """The largest top_k of either bound search and one more, ties taken in part by both selections, rows whose length
    is no multiple of four."""
    smooth = (normal_bf16(111, V, (rows, V), 1.0).float() * 2.0 + 2.0 ** -9 * normal_bf16(112, V, (rows, V), 1.0).float()).contiguous()
    coarse = (smooth * 4).round() / 4                                # hundreds of equal logits at every threshold
    u = uniforms(113, rows)
    for T, k, p in ((0.8, 64, 0.9), (0.8, 65, 0.9), (1.0, 256, 0.99), (1.0, 257, 0.99), (0.9, 2, 0.5), (1.0, 0, 1e-6), (0.7, 0, 0.97)):
        params = sv.SamplingParams(T, k, p)
        for logits in (smooth, coarse):
            say(f"V={V} rows={rows} T={T} top_k={k} top_p={p}")
            check_rows(logits, params, u, rows // 2)


def test_lists_that_overflow_take_the_general_path():
    """Flat rows, and likely tokens that all lie in one workgroup's share of the row: closed-form answers."""
    u = torch.tensor([0.0, 0.3, 0.999])
    for V, top_k, top_p, n in ((16384, 0, 0.5, 8192), (16384, 100, 1.0, 100)):
        flat = torch.zeros(3, V)
        for call in (sv.sssd_op_sample, sv.sssd_op_sample_wide):
            assert call(flat.to(DEV), sv.SamplingParams(1.0, top_k, top_p), u.to(DEV)).cpu().tolist() == [int(x * n) for x in u.tolist()]
    V = 128256
    heap = torch.full((1, V), -10.0)
    heap[0, 300:1100] = 5.0
    for x in u.tolist():
        got = sv.sssd_op_sample_wide(heap.to(DEV), sv.SamplingParams(1.0, 50, 1.0), torch.tensor([x]).to(DEV))
        assert got.cpu().tolist() == [300 + int(x * 50)]


@pytest.mark.parametrize("V,rows", [(8192, 3), (4099, 129)])     # clusters of 16 workgroups and of one
@pytest.mark.parametrize("T", [1e-40, 4e-39])                    # 1 / T overflows; only its product with log2(e) does
def test_temperatures_without_any_mass_give_the_argmax(V, rows, T):
    """The limit of T towards 0 is the arg-max, also where no weight can be represented any more.  Every token is written:
    the outputs hold a sentinel before the call."""
    z = (normal_bf16(121, V, (rows, V), 1.0).float() * 2.0).contiguous()
    z[torch.arange(rows), (torch.arange(rows) * 997) % V] = 20.0
    z, u = z.to(DEV), uniforms(122, rows).to(DEV)
    need = sv.lib().sssd_op_sample_scratch_bytes(rows)
    scratch = torch.empty(max(need, 16), dtype=torch.uint8, device=DEV)
    for k, p in ((5, 1.0), (5, 0.9), (0, 0.95), (0, 1.0)):
        say(f"V={V} rows={rows} T={T} top_k={k} top_p={p}")
        params = sv.SamplingParams(T, k, p)
        one, wide = (torch.full((rows,), -7, dtype=torch.int32, device=DEV) for _ in range(2))
        at = (z.data_ptr(), rows, V, C.byref(params), u.data_ptr())
        assert sv.lib().sssd_op_sample(*at, one.data_ptr(), None) == 0
        assert sv.lib().sssd_op_sample_wide(*at, wide.data_ptr(), scratch.data_ptr() if need else None, need, None) == 0
        assert torch.equal(one, z.argmax(-1).to(torch.int32)) and torch.equal(wide, one)


@pytest.mark.parametrize("V,rows", [(128256, 3), (32003, 130)])    # clusters of 16 and of one; rows of 16-byte loads and not
@pytest.mark.parametrize("kind", ["equal", "narrow", "narrow_high", "narrow_low", "quarters", "two_values"])
def test_rows_that_the_lists_leave_to_the_general_path(V, rows, kind):
    """The general path starts from what the lists' passes found: the maximum, the digits that the keys between a bound and
    the maximum or within one bin share, the mass above that bin.  Logits whose keys share one to three digits or none, ties
    cut by either selection; every token against the sort that the definition states."""
    z = (normal_bf16(131, V, (rows, V), 1.0).float() + 2.0 ** -9 * normal_bf16(132, V, (rows, V), 1.0).float())
    z = {"equal": torch.full_like(z, 1.7), "narrow": z * 0.1, "narrow_high": z * 0.05 + 900.0, "narrow_low": z * 0.02 - 37.0,
         "quarters": (z * 8).round() / 4, "two_values": (z > 0).float() * 3 - 1}[kind].contiguous()
    u = uniforms(133, rows)
    checked = 0
    for T, k, p in ((1.0, 0, 0.9), (1.0, 0, 0.3), (0.3, 0, 0.99), (1.0, 50, 1.0), (1.0, 256, 0.9), (1.0, 257, 0.9)):
        params = sv.SamplingParams(T, k, p)
        say(f"{kind} V={V} rows={rows} T={T} top_k={k} top_p={p}")
        n = min(rows, 3)                                            # the oracle sorts the whole row on the host
        checked += check_rows(z[:n].contiguous(), params, u[:n].contiguous(), 0)[0]
        one = sv.sssd_op_sample(z.to(DEV), params, u.to(DEV))
        assert torch.equal(one, sv.sssd_op_sample_wide(z.to(DEV), params, u.to(DEV)))
        if k:                                                       # order O on the host: by logit, then by id
            order = torch.sort(z[0], descending=True, stable=True).indices[:k]
            assert int(one[0]) in set(order.tolist())
    assert checked >= 10    # of 18; a flat distribution over 128256 tokens has steps of 8e-6, so several rows lie within the exemption
