"""The C-ABI library loads without a GPU and exports every function include/*.h declares;
argument validation that needs no device is exercised too."""
import ctypes as C
import glob
import os
import re

import pytest

from paper_2411_05894_amd import binding as sv
from sssd_synth import MODEL_SHAPES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    names = []
    for path in sorted(glob.glob(os.path.join(ROOT, "include", "*.h"))):
        text = re.sub(r"/\*.*?\*/", "", open(path).read(), flags=re.S)
        names += re.findall(r"\b(sssd_[a-z_0-9]+)\s*\(", text)
    return sorted(set(names))


def test_every_declared_symbol_is_exported():
    names = declared_functions()
    assert len(names) >= 15
    lib = sv.lib()
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in include/ but not exported"


def test_sizes_and_config_validation_without_gpu():
    cfg = sv.make_config(MODEL_SHAPES["8b"], 1, 16, 2048 + 17)
    kv, ws, pk = sv.sssd_verify_sizes(cfg)
    assert kv == 2 * 32 * 8 * 2080 * 128 * 2            # K and V, 32 layers, rows padded to 32
    assert pk == 15009316864                            # every 8B matrix, bf16, no padding needed
    assert ws > 0
    bad = sv.make_config(MODEL_SHAPES["8b"], 1, 16, 2048 + 17)
    bad.head_dim = 96
    assert sv.lib().sssd_verify_sizes(C.byref(bad), None, None, None) == sv.SSSD_EINVAL
    bad = sv.make_config(MODEL_SHAPES["8b"], 1, 40, 4096)
    assert sv.lib().sssd_verify_sizes(C.byref(bad), None, None, None) == sv.SSSD_EINVAL
    assert sv.lib().sssd_verify_sizes(None, None, None, None) == sv.SSSD_EINVAL
    tiny = sv.make_config(MODEL_SHAPES["tiny"], 1, 4, 512)
    _, _, pk = sv.sssd_verify_sizes(tiny)
    assert pk > 3424256                                 # ffn = 688 is padded to 704 columns


def test_null_handles_are_rejected():
    lib = sv.lib()
    assert lib.sssd_verify_step(None, 1, 0, None, None, None, None, None) == sv.SSSD_EINVAL
    assert lib.sssd_kv_rollback(None, 1, None, None, None, None) == sv.SSSD_EINVAL
    assert lib.sssd_verify_destroy(None) == sv.SSSD_EINVAL
    assert lib.sssd_verify_sync(None, None) == sv.SSSD_EINVAL
    assert "capacity" in sv.strerror(sv.SSSD_ECAPACITY)
    assert lib.sssd_op_packed_weight_bytes(4096, 4096) == 4096 * 4096 * 2
    assert lib.sssd_op_packed_weight_bytes(256, 688) == 256 * 704 * 2


def test_plan_check_covers_every_step_of_a_configuration_without_gpu():
    """sssd_verify_plan_check (host only): every (B, k) inside the configuration fits the buffers
    sssd_verify_sizes asks for; anything beyond the configuration is a capacity error."""
    lib = sv.lib()
    for shape, mb, mk, ms in (("tiny", 8, 31, 260), ("8b", 32, 16, 4113), ("70b", 16, 8, 2057)):
        cfg = sv.make_config(MODEL_SHAPES[shape], mb, mk, ms)
        for B in range(1, mb + 1):
            for k in range(mk + 1):
                assert lib.sssd_verify_plan_check(C.byref(cfg), B, k) == sv.SSSD_OK, (shape, B, k)
        assert lib.sssd_verify_plan_check(C.byref(cfg), mb + 1, 0) == sv.SSSD_ECAPACITY
        assert lib.sssd_verify_plan_check(C.byref(cfg), 1, mk + 1) == sv.SSSD_ECAPACITY
        assert lib.sssd_verify_plan_check(C.byref(cfg), 0, 0) == sv.SSSD_EINVAL
    assert lib.sssd_verify_plan_check(None, 1, 0) == sv.SSSD_EINVAL


def test_the_gemm_kernel_of_a_matrix_follows_from_its_size_without_gpu():
    """Up to 32 rows the matrix decides which kernel a GEMM takes: 64 MB at 17..32 rows; below, 256 MB and a K beyond what
    one workgroup covers.  pgemm_kernel with an unsplit K is the one form that needs no scratch."""
    of = sv.sssd_op_gemm_kernel_of
    for M, N, K, want in ((9, 28672, 4096, "pgemm_kernel"), (16, 57344, 8192, "qgemm16_kernel"), (16, 8192, 28672, "qgemm16_kernel"),
                          (16, 10240, 8192, "pgemm_kernel"), (1, 128256, 4096, "pgemm_kernel"), (32, 6144, 4096, "pgemm_kernel"),
                          (17, 28672, 4096, "qgemm16_kernel"), (32, 4096, 14336, "qgemm16_kernel"), (33, 16, 32, "qgemm16_kernel")):
        assert of(M, N, K) == want, (M, N, K)
        if K <= 4096:
            assert (sv.lib().sssd_op_gemm_scratch_bytes(M, N, K) == 0) == (want == "pgemm_kernel")
    assert of(0, 16, 32) == of(1, 8, 32) == of(1, 16, 0) == ""
    for M in (1, 16, 17, 32, 33, 160, 512):
        assert sv.sssd_op_gemm_kernel_name(M) == of(M, 28672, 4096)


def test_workspace_holds_no_copy_of_logits_that_no_launch_splits_without_gpu():
    """An LM head whose K is never split over workgroups adds its arg-max partials to the workspace (a value and an index per
    16 columns and row, rows in whole blocks of 160), not the fp32 copy of its output that only split sums pass through."""
    from types import SimpleNamespace
    base = MODEL_SHAPES["8b"].__dict__
    ws = [sv.sssd_verify_sizes(sv.make_config(SimpleNamespace(**{**base, "vocab": v}), 16, 31, 512))[1] for v in (1024, 128256)]
    rows = 640                                    # 16 * 32 in blocks of 160
    assert ws[1] - ws[0] <= 8 * rows * (128256 - 1024) // 16 + 1024


def test_plans_fit_models_of_a_single_column_tile_without_gpu():
    """A hidden size or a vocabulary of 16 leaves one sum of squares or arg-max partial per row, and the buffers hold no more: with row
    blocks (more than 160 rows) and a K split over workgroups, too."""
    from types import SimpleNamespace
    for hidden, ffn, vocab in ((512, 48, 16), (1040, 48, 16), (16, 512, 528), (16, 4096, 16), (32, 1024, 32), (272, 512, 272)):
        s = SimpleNamespace(n_layers=1, hidden=hidden, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=ffn, vocab=vocab, rms_eps=1e-5,
                            rope_base=10000.0)
        cfg = sv.make_config(s, 16, 31, 64)
        for B in range(1, 17):
            for k in range(32):
                assert sv.lib().sssd_verify_plan_check(C.byref(cfg), B, k) == sv.SSSD_OK, (hidden, ffn, vocab, B, k)
