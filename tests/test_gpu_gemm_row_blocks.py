"""GEMMs of more than 160 rows: two to eight row blocks of six or eight tiles in one launch, whole and partial last blocks,
grids that do and do not divide into sets of eight, split and unsplit K, a last column group partly inside the matrix."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import oracle
from paper_2411_05894_amd import binding as sv
from sssd_synth import normal_bf16

DEV = "cuda:0"


@pytest.mark.parametrize("N,K", [(96, 4096), (272, 352), (2064, 1024), (24592, 64)])
@pytest.mark.parametrize("M", [161, 176, 177, 192, 256, 320, 321, 352, 481, 512, 1000])
def test_row_blocks_vs_oracle(N, K, M):
    print(f"gemm N={N} K={K} M={M}", flush=True)
    w = normal_bf16(61, N * 3 + K, (N, K), 0.02, device=DEV)
    x = normal_bf16(62, M * 7 + K, (M, K), 1.0, device=DEV).float() * 1.25
    x += 2.0 ** -10 * normal_bf16(63, M + K, (M, K), 1.0, device=DEV).float()     # not bf16-representable
    hi, lo = sv.sssd_op_pack_activation(x)
    y = sv.sssd_op_gemm(hi, lo, sv.sssd_op_pack_weight(w), M, N, K)
    rows = sorted(set(range(0, M, 37)) | {15, 16, 159, 160, M - 17, M - 2, M - 1})  # the oracle runs on the host
    ref = oracle.linear(x[rows].cpu(), w.cpu())
    assert (y[rows].cpu() - ref).abs().max().item() <= 3e-5 * ref.abs().max().item() + 1e-6
    full = x.double() @ w.double().t().contiguous()
    assert (y - full).abs().max().item() <= 3e-5 * full.abs().max().item() + 1e-6
