"""Steps of up to 32 rows with a short K: one, two and four k-tiles per wave, on both sides of every line between them, K that ends
inside a k-tile, and waves with nothing but padding."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2411_05894_amd import binding as sv
from test_gpu_gemm_pipeline import check


@pytest.mark.parametrize("K", [8, 32, 488, 512, 520, 1024, 1032, 1504, 2048, 2056, 4096])
@pytest.mark.parametrize("N,M", [(16, 1), (272, 5), (4128, 16), (96, 17), (528, 32)])
def test_short_k(N, K, M):
    assert sv.sssd_op_gemm_kernel_of(M, N, K) == "pgemm_kernel"
    check(N, K, M)
