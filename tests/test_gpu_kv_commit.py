"""Tree commit against a plain tensor: paths of up to 31 rows (the kernel moves eight at a time), rows that are each other's
destinations, rows that cross a block of 32 positions, both head sizes, sequences that commit nothing, a shuffled block table,
and a path that stops increasing on the way."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2411_05894_amd import binding as sv
from sssd_synth import MODEL_SHAPES, global_weight_specs, layer_weight_specs, normal_bf16

DEV = "cuda:0"
PATHS = [list(range(1, 32)),                            # a chain: nothing moves
         [2, 3, 4, 5, 6, 7, 8, 9, 10, 11],              # every destination is the source before
         [1, 2, 3, 30, 31], [31], [],
         [2 * i for i in range(1, 16)],
         [i + (i > 5) + (i > 9) + (i > 17) for i in range(1, 28)]]


@pytest.mark.parametrize("shape_name", ["tiny", "8b"])   # head sizes 64 and 128
@pytest.mark.parametrize("paged", [False, True])
def test_commit_moves_the_path(shape_name, paged):
    k, max_seq, L = 31, 160, 2
    s = MODEL_SHAPES[shape_name]
    s = type(s)(**{**s.__dict__, "n_layers": L, "vocab": 1024, "hidden": 64, "ffn": 64})
    layers = [{n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in layer_weight_specs(s)} for _ in range(L)]
    g = {n: torch.zeros(shp, dtype=torch.bfloat16, device=DEV) for n, _, shp in global_weight_specs(s)}
    paths = PATHS + [[2, 5, 9, 12, 15, 18, 20, 22, 25, 24, 30]]      # the tenth row goes back: nine move, the length stays
    B = len(paths)
    ctx = sv.VerifyContext(sv.make_config(s, B, k, max_seq), layers, g)
    if paged:
        _, bps, n_pages = sv.sssd_kv_geometry(ctx.cfg)
        ctx.sssd_kv_set_block_table(torch.randperm(n_pages, generator=torch.Generator().manual_seed(9)).to(torch.int32).view(B, bps).to(DEV))
    lens = [0, 1, 31, 20, 64, 100, 90, 33][:B]
    want = []
    for l in range(L):
        for b in range(B):
            kv = [normal_bf16(81, (l * B + b) * 2 + i, (s.n_kv_heads, max_seq, s.head_dim), 1.0, device=DEV) for i in range(2)]
            ctx.sssd_kv_import(l, b, 0, *kv)
            moved = paths[b] if b < len(PATHS) else paths[b][:9]
            for x in kv:
                new = x[:, [lens[b] + node for node in moved]].clone()
                x[:, lens[b] + 1:lens[b] + 1 + len(moved)] = new
            want.append(kv)
    path = torch.full((B, k + 1), -1, dtype=torch.int32)
    for b, p in enumerate(paths):
        path[b, 0] = 0
        path[b, 1:len(p) + 1] = torch.tensor(p, dtype=torch.int32)
    dlens = torch.tensor(lens, dtype=torch.int32, device=DEV)
    acc = torch.tensor([len(p) for p in paths], dtype=torch.int32, device=DEV)
    print(f"kv commit {shape_name} paged={paged}", flush=True)
    ctx.sssd_kv_commit_tree(dlens, acc, path.to(DEV))
    assert ctx.sssd_verify_sync() == sv.SSSD_ENOSPACE                # the bad path
    assert dlens.tolist() == [n + len(p) + 1 for n, p in zip(lens, PATHS)] + [lens[-1]]
    for l in range(L):
        for b in range(B):
            got = [torch.empty_like(x) for x in want[l * B + b]]
            ctx.sssd_kv_export(l, b, 0, *got)
            for x, y in zip(got, want[l * B + b]):
                assert torch.equal(x.view(torch.int16), y.view(torch.int16)), (l, b)
