"""The pipelined GEMM kernel at every row-tile count up to ten: slices of one, two and three k-tiles (fewer than are in
flight), odd k-tile counts, split and unsplit K, four and eight waves (up to 64 rows eight from 512 MB on, a test of its own),
a last column group partly inside the matrix."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import oracle
from paper_2411_05894_amd import binding as sv
from sssd_synth import normal_bf16

DEV = "cuda:0"


def check(N, K, M):
    print(f"gemm N={N} K={K} M={M}", flush=True)
    w = normal_bf16(71, N * 3 + K, (N, K), 0.02, device=DEV)
    x = normal_bf16(72, M * 7 + K, (M, K), 1.0, device=DEV).float() * 1.25
    x += 2.0 ** -10 * normal_bf16(73, M + K, (M, K), 1.0, device=DEV).float()     # not bf16-representable
    hi, lo = sv.sssd_op_pack_activation(x)
    y = sv.sssd_op_gemm(hi, lo, sv.sssd_op_pack_weight(w), M, N, K)
    full = x.double() @ w.double().t().contiguous()
    # x = hi + lo to 2^-17 of x, products and sums in fp32: the bound of the other GEMM parity tests
    assert (y - full).abs().max().item() <= 3e-5 * full.abs().max().item() + 1e-6
    cols = slice(max(0, N - 96), N)                                                # the oracle runs on the host
    ref = oracle.linear(x[[0, M - 1]].cpu(), w[cols].cpu())
    assert (y[[0, M - 1]][:, cols].cpu() - ref).abs().max().item() <= 3e-5 * ref.abs().max().item() + 1e-6


@pytest.mark.parametrize("N,K", [(16, 32), (96, 64), (144, 96), (272, 352), (2064, 1056), (8208, 4128)])
@pytest.mark.parametrize("M", [33, 47, 48, 49, 64, 80, 81, 112, 113, 128, 144, 145, 160])
def test_row_tiles(N, K, M):
    check(N, K, M)


# either side of the lines between the kernels: 64 MB at 17..32 rows, 256 MB and a K split at up to 16 rows, and results
# whose partial sums would not fit the library's own scratch array
@pytest.mark.parametrize("N,K,M", [(8192, 4064, 17), (8192, 4096, 17), (8208, 4128, 31), (3888, 8640, 32), (127104, 288, 18),
                                   (270000, 128, 32), (16368, 8192, 16), (16384, 8192, 1), (16400, 8224, 16), (9616, 14336, 5),
                                   (32800, 4096, 9)])
def test_small_steps_of_large_matrices(N, K, M):
    check(N, K, M)


# 514 MB: eight waves also at up to four row tiles, each count with its own staging, read-ahead and wait counts; the matrix
# ends inside a column group of 256, and K, 257 k-tiles in seven slices, in a shorter slice
@pytest.mark.parametrize("N,K", [(32784, 8224)])
@pytest.mark.parametrize("M", [5, 16, 17, 32, 33, 48, 49, 64])
def test_eight_waves_at_few_rows(N, K, M):
    assert sv.sssd_op_gemm_kernel_of(M, N, K) == "qgemm16_kernel" and N * K * 2 >= 512 << 20
    check(N, K, M)


# up to 32 rows either kernel may serve a matrix, so neither may round worse than the other
@pytest.mark.parametrize("N,K", [(28672, 4096), (4096, 14336), (57344, 8192), (8192, 28672)])
@pytest.mark.parametrize("M", [5, 16, 17, 32])
def test_rounding_of_small_steps(N, K, M):
    """Against 64 bits on the operands as they are stored.  A chain of n fp32 additions of like terms has a relative error
    of sqrt(n / 2) * 2^-24 / sqrt(3) (every sum rounds once, and is sqrt(i / n) of the last).  The small-step kernel adds 8
    k-tiles, 16 waves and J slices of 128 k-tiles: sqrt(4 + 8 + J / 2).  The error averages over M * N >= 20480 elements."""
    print(f"gemm rounding N={N} K={K} M={M}", flush=True)
    w = normal_bf16(74, N * 3 + K, (N, K), 0.02, device=DEV)
    x = normal_bf16(75, M * 7 + K, (M, K), 1.0, device=DEV).float() * 1.25
    hi, lo = sv.sssd_op_pack_activation(x)
    y = sv.sssd_op_gemm(hi, lo, sv.sssd_op_pack_weight(w), M, N, K)
    xh = x.to(torch.bfloat16)
    stored = xh.double() + (x - xh.float()).to(torch.bfloat16).double()
    err = size = 0.0
    for n in range(0, N, 8192):
        full = stored @ w[n:n + 8192].double().t().contiguous()
        err += (y[:, n:n + 8192] - full).square().sum().item()
        size += full.square().sum().item()
    J = -(-K // 4096)
    bound = (12 + J / 2) ** 0.5 * 2.0 ** -24 / 3 ** 0.5
    rel = (err / size) ** 0.5
    print(f"relative error {rel:.3e}, bound {bound:.3e}", flush=True)
    assert rel <= bound
